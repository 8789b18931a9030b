#pragma once
// Heads per workgroup of the ring attention kernels (k_nat_tile.hip), chosen on
// the host.

namespace wm {

enum NatRows : int { NAT_HEAD_MAJOR = 0, NAT_TOKEN_MAJOR = 1, NAT_E4M3 = 2 };

// Heads that a workgroup walks one after the other over the same tile, of
// `tiles` (query tiles of all states) and H heads.  The fewer workgroups are
// left, the more CUs idle in the last round; so a number is taken where it
// leaves 4096 workgroups (e4m3, four heads: 8192), 5 rounds or more of those that
// run at once.  us with 1 / 2 / 4 heads, by tiles x heads, 8 levels and window
// 5x7x7 unless said:
//   bf16 from token-major q and k (wm_nat_forward): two heads share K's cache lines
//       4232   78 /  83 /  93     16928 (16 heads) 398 / 371 / 364     33856 713 / 671 / 698
//   bf16 from head-major ones (the blocks): nothing is shared, and the halo rows
//   that the next tiles share have left L2 by the next head (1.02 GB fetched with 4
//   heads, 0.73 with 2, 0.47 with 1, per block of 129600 tokens).  A walk of 5 to 8
//   levels covers what a workgroup does around it; one of 3 to 5 gains by two heads
//       8832  140 / 144 / 150     12512  209 / 213 / 218     16928 282 / 282 / 284
//     3x5x5:  9216  111 / 106 / 107     16928  204 / 195 / 197     36864 440 / 413 / 401
//             4608   59 /  58 /  64      1152   21 /  22 /  34
//   e4m3
//       4608   74 /  73 /  84      8832  122 / 120 / 121     12288  185 / 177 / 179
//      23040  331 / 312 / 320     36864  515 / 491 / 487     67712 1010 / 970 / 960
//     3x5x5:  4608   56 /  58 /  63      9216  106 / 102 / 107     36864  385 / 361 / 354
inline int nat_heads(long tiles, int H, int Kz, NatRows rows) {
    const int most = rows == NAT_HEAD_MAJOR ? (Kz > 3 ? 1 : 2) : 4;
    for (int n = most; n > 1; n >>= 1)
        if (H % n == 0 && tiles * (H / n) >= (rows == NAT_E4M3 ? 2048 * n : 4096)) return n;
    return 1;
}

}  // namespace wm
