#pragma once
// The tile of the LDS-ring GEMMs (k_gemm_lds.hip), chosen on the host.
#include <algorithm>

namespace wm {

// Tile choice.  Three tiles give the same bits (every accumulator adds the
// same k-steps in the same order), so the choice is by time alone:
//   256 x 256 (gemm_pp_kernel)   fewest LDS and L2 bytes per FLOP, but one
//                                 workgroup per CU: 1.0 to 1.9 rounds over the
//                                 256 CUs cost two;
//   128 x 128 (gemm_lds_kernel)  two workgroups per CU, finer rounds;
//   64 x 64                      four per CU, for outputs too small to give
//                                 every CU a larger tile.
// The estimates below (us) are fits to times measured over M = 100 .. 129600
// at (N, K) = (1536, 512), (2048, 512), (512, 2048), (512, 512), (3072, 1024),
// (1024, 4096), (768, 256), (256, 1024), in bf16 and e4m3; nk: stages of 128
// bytes per row.  They place the lines between the tiles; measured, bf16, us,
// (M, N, K): 256 x 256 / 128 x 128 / 64 x 64
//   (129600, 2048, 512) 347 / 467 / 589     (32000, 512, 2048)  70 /  75 / 101
//   ( 40000, 512, 2048) 105 /  96 / 127     (20250,  512, 512)  31 /  28 /  26
//   (  8640, 2048, 512)  41 /  30 /  33     ( 2880, 512, 2048)  51 /  25 /  19
//   (  1200, 512, 512)   18 /  10 /   7     (  405, 1024, 4096) 85 /  41 /  31
struct TilePlan {
    int bm;        // 256, 128 or 64
    int tpw;       // 256: tiles per workgroup
    int rw;        // 256: walk row blocks (1) or feature tiles (0)
};
// n256: whether 256-wide feature tiles are possible; wmax: most feature tiles
// a 256 x 256 workgroup may walk (a QKV workgroup's are all V or none).
// resid: the float32 residual update (reads and writes 8 bytes per element).
inline TilePlan plan_tiles(int M, int N, int nk, bool n256, int wmax, bool resid) {
    auto cdiv = [](long a, long b) { return (a + b - 1) / b; };
    const long t64 = cdiv(M, 64) * (N / 64), t128 = cdiv(M, 128) * (N / 128);
    // (past some 7500 tiles of 128 x 128 the bf16 output no longer fits the 256
    // MB cache behind the L2s, and the smaller tiles' extra reads cost a third)
    const double far = t128 > 7500 ? 1.3 : 1.0;
    // us per round of 64 x 64, and of 128 x 128, tiles, and per 256 x 256 tile
    double r64 = 0.35 + 0.22 * nk, r128 = 4.5 + 1.1 * nk, r256 = 11.0 + 1.15 * nk;
    // One and two stages: past a few rounds the output counts and not the main
    // loop.  bf16, us, (M, N, K, residual): 256 x 256 / 128 x 128 / 64 x 64
    //   (130000, 2048,  64, no) 151 / 195 / 232    (130000, 1536, 128, no) 149 / 194 / 223
    //   (130000,  384,  64, no)  -  /  33 /  36    (520000,  768, 128, no) 331 / 392 / 463
    // The lines above, fitted from four stages on, gave all of these 64 x 64.
    // The residual update is bound by its bytes, which 128 x 128 tiles move fastest:
    //   (130000, 4096,  64, yes) 843 / 825 / 918   (130000, 1536, 192, yes) 384 / 366 / 398
    if (nk <= 4 && resid) {
        if (t128 > 4000 && (nk <= 2 || N != 512)) return TilePlan{128, 1, 0};
    } else if (nk <= 2 && t128 > 2048) {
        r64 = std::max(r64, 0.69);
        r128 = 3.2 + 1.55 * nk;
        r256 = 6.5 + 2.1 * nk;
    }
    const double c64 = 4.0 + r64 * cdiv(t64, 256) * far;
    const double c128 = t128 <= 256 ? 5.5 + 0.65 * nk : r128 * (t128 <= 512 ? 1.0 : std::max(2.0, t128 / 512.0)) * far;
    TilePlan best{c64 <= c128 ? 64 : 128, 1, 0};
    double c = std::min(c64, c128);
    if (!n256) return best;
    // 256 x 256: a workgroup that walks w tiles overlaps each next tile's
    // loads with the previous epilogue (one tile alone: 3 us more), unless
    // that leaves a round of workgroups short.  N = 512 walks row blocks (the
    // workgroups that share a row block are neighbours on one XCD), wider N
    // feature tiles; the block's MLP1 (N = 2048) runs fastest with 4.
    const long ntm = cdiv(M, 256), ntn = N / 256;
    const int rw = N == 512 && wmax > 1;
    for (int w = 1; w <= wmax; ++w) {
        const long groups = rw ? cdiv(ntm, w) * ntn : ntm * cdiv(ntn, w);
        const double t = 4.0 + cdiv(groups, 256) * (3.0 + w * r256);
        if (t < c) {
            c = t;
            best = TilePlan{256, w, rw};
        }
    }
    return best;
}
// Most tiles a 256 x 256 workgroup walks.
inline int wide_max(int N) { return N >= 2048 ? 4 : (N >= 1536 ? 3 : (N == 512 ? 2 : 1)); }

}  // namespace wm
