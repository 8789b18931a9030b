// MFMA GEMM (bf16 or e4m3 operands, or float32 ones split into bf16 parts;
// float32 accumulation) fed by an LDS ring that direct buffer->LDS loads fill.
//
//   D[m][n] = sum_k A[m][k] * W[n][k]      (A: tokens x K, W: [out][in])
//
// K advances in stages of 128 bytes per row (64 bf16, 128 e4m3 or 32 float32 values),
// written straight from global memory into LDS by buffer_load_dwordx4 ... lds
// (no register staging).  Rows of A past M come back as zeros from the buffer
// range check, which handles the ragged last token tile.  16-byte chunks of an
// LDS row are XOR-swizzled so that fragment reads have no bank conflicts.  The
// MFMA "A" operand is the weight tile and "B" the activation tile, so every
// lane ends up with four consecutive output features of one token for the
// epilogue (V tiles of the QKV projection swap them).  Tiles go out in an
// XCD-aware order (consecutive ids on one XCD share an activation tile in its
// L2).  gemm_pp_kernel computes wide tiles (256 x 256, or 128 x 512 with the
// LayerNorm epilogue) in two groups of waves half a phase apart,
// gemm_lds_kernel the narrow ones; plan_tiles chooses.
#include <algorithm>
#include <type_traits>

#include "gemm_plan.hpp"
#include "kernels.hpp"

namespace wm {
namespace glds {

typedef __attribute__((address_space(3))) void lds_void;

// EPI_RESID and EPI_RESID_LN on states in separate buffers whose token count
// is not a multiple of 64: the 64 rows of a wave may lie in several states.
constexpr int EPI_RESID_SPLIT = 6, EPI_RESID_LN_SPLIT = 7;
// EPI_GELU of bf16 maps whose N is not a multiple of 128 (no processor's): erf
// by 7.1.28, as these maps have always had it.
constexpr int EPI_GELU_28 = 8;
constexpr bool epi_resid(int e) { return e == EPI_RESID || e == EPI_RESID_SPLIT; }
constexpr bool epi_resid_ln(int e) { return e == EPI_RESID_LN || e == EPI_RESID_LN_SPLIT; }
inline bool splits(const EpiArgs &ep) { return ep.resid_ptrs && ep.T % 64 != 0; }

// XOR swizzle of the 16-byte chunks of a 128-byte LDS row, so that a fragment
// read (ds_read_b128) has no bank conflict.  Its 64 lanes (row r16 = l % 16,
// chunk by g = l / 16) go through LDS 16 at a time: in the lower half of the
// wave rows 0-3 and 12-15 of g = 0 with rows 4-11 of g = 1, then the others;
// the upper half alike with g = 2, 3.  bf16 lanes of neighbouring g read
// neighbouring chunks (4 o + g): (row >> 1) & 7.  e4m3 lanes read chunks 2 g
// and 2 g + 1, two apart: with t = (row >> 1) & 7 rows 0-3 and 12-15 get the
// even and rows 4-11 the odd values (with the bf16 swizzle half of the LDS
// cycles of the e4m3 GEMM were conflicts).
template <bool FP8>
__device__ __forceinline__ int swz(int row) {
    const int t = (row >> 1) & 7;
    return FP8 ? (t & 4) | ((t & 1) << 1) | (((t >> 1) ^ (t >> 2)) & 1) : t;
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *p, unsigned bytes) {
    const unsigned long long v = (unsigned long long)p;
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
    return __builtin_amdgcn_make_buffer_rsrc((void *)(((unsigned long long)hi << 32) | lo), 0, bytes,
                                             0x00020000);
}

// Epilogue stores (and residual loads) go through buffer resources whose base
// is the wave's first row, so that a lane's 32-bit offsets are the same for
// every tile and rows past M fail the range check: a store there is dropped,
// a load reads zero.
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// An offset that fails every range check.
constexpr unsigned DROP = 0xfffff000u;

// A wave's rows of an output: `bytes` from `p` on; at(n): the same n bytes on.
// Constant byte offsets of stores go into the resource's base and not into the
// instruction's scalar offset: after a 16-byte store with a scalar offset
// register the compiler may overwrite the data registers in the very next
// instruction, and such stores then wrote some of the new values (single rows
// of MLP1's output at N = 1024); without that register it keeps the two
// instructions between that the hardware needs.
struct RowSpan {
    unsigned long long p;
    unsigned bytes;
    __device__ __forceinline__ RowSpan(const void *q, unsigned n) {
        const unsigned long long v = (unsigned long long)q;
        p = ((unsigned long long)__builtin_amdgcn_readfirstlane((unsigned)(v >> 32)) << 32) |
            (unsigned)__builtin_amdgcn_readfirstlane((unsigned)v);
        bytes = __builtin_amdgcn_readfirstlane(n);
    }
    __device__ __forceinline__ __amdgpu_buffer_rsrc_t at(unsigned n) const {
        return __builtin_amdgcn_make_buffer_rsrc((void *)(p + n), 0, bytes > n ? bytes - n : 0u, 0x00020000);
    }
};

__device__ __forceinline__ u32x2 pack4_bf16(const float *v) { return u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])}; }
__device__ __forceinline__ u32x4 pack8_bf16(const float *v) {
    return u32x4{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7])};
}

// One MFMA k-step: acc of the tile of W rows wf by activation rows af, from
// zero if FIRST.  SWAP: the activation tile is the MFMA "A" operand, so a lane
// holds four consecutive tokens of one output feature (the blocked V layout).
template <bool FIRST, bool SWAP>
__device__ __forceinline__ f32x4 mma_bf16(i32x4 wf, i32x4 af, f32x4 c) {
    const bf16x8 w = __builtin_bit_cast(bf16x8, wf), a = __builtin_bit_cast(bf16x8, af);
    const f32x4 z = {0.f, 0.f, 0.f, 0.f};
    return SWAP ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, w, FIRST ? z : c, 0, 0, 0)
                : __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, a, FIRST ? z : c, 0, 0, 0);
}
// gfx950 16x16x128 f8f6f4 MFMA (e4m3 x e4m3): a lane holds 32 k-values of its
// row for both operands, the k chunk 32 g .. 32 g + 31 of the stage as two
// 16-byte pieces; both operands use the same k assignment, which is all a
// contraction over k needs.
template <bool FIRST, bool SWAP>
__device__ __forceinline__ f32x4 mma_fp8(const i32x4 (&wf)[2], const i32x4 (&af)[2], f32x4 c) {
    const i32x8 w = __builtin_shufflevector(wf[0], wf[1], 0, 1, 2, 3, 4, 5, 6, 7);
    const i32x8 a = __builtin_shufflevector(af[0], af[1], 0, 1, 2, 3, 4, 5, 6, 7);
    const f32x4 z = {0.f, 0.f, 0.f, 0.f};
    return SWAP ? __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, w, FIRST ? z : c, 0, 0, 0, 0, 0, 0)
                : __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(w, a, FIRST ? z : c, 0, 0, 0, 0, 0, 0);
}

// Float32 operands on the bf16 matrix cores: SPLIT_SCALE x = x1 + x2 + x3
// exactly, each part the remainder rounded to nearest bf16 (8 significant bits;
// so |x2| <= 2^-9 |x1|, |x3| <= 2^-18 |x1|).  The last bit of x is 2^-149 or
// more: times 2^24 it is 2^-125, a normal bf16, so no part is lost however small
// x is (without the factor the parts of x < 2^-110 fell under bf16's smallest
// values: errors of 2^-22 of x at 2^-112, 2^-8 at 2^-126).  Values of 2^104 and
// more and sums of 2^80 and more overflow and are done again (f32_finish).
// A product is the sum of the six partial products x_i w_j with i + j <= 4,
// smallest first; the three left out are below 2^-26 of it, with either sign.
// The products of bf16 values are exact and the sum takes 6 roundings per 32 k
// where 16x16x4 f32 MFMAs take 8, at six bf16 MFMAs of 16 cycles instead of eight
// of 32.  Measured (N(0,1) rows, N(0,0.02) weights) the relative error against
// float64 is 1.54e-7, 3.36e-7, 4.9e-7 and 1.00e-6 at K = 128, 512, 1024 and 4096,
// against 2.04e-7, 4.06e-7, 5.7e-7 and 1.15e-6 with f32 MFMAs.  M = 129600,
// N = 1536, K = 512: 2141 us with those, 1165 so (1110 without the factor); K =
// 2048, N = 512: 2714, 1461 (1382).  Lane and k layout are those of one 16x16x32
// operand (8 consecutive k).
constexpr float SPLIT_SCALE = 0x1p24f, UNSPLIT = 0x1p-48f;
struct Split3 {
    i32x4 p[3];
};
__device__ __forceinline__ Split3 split3(const i32x4 (&raw)[2]) {
    Split3 s;
    // remainders by the bf16 dot product, a - part as part * -1 + other * 0 + a: one
    // instruction where unpacking and subtracting take two (products and differences
    // are exact; 4e9 random pairs of all exponents gave the bits of the subtraction).
    // It pays for the scaling: a float32 block at 8x90x180, C = 512, takes 6.10 ms
    // without the factor, 6.30 with it and subtractions, 6.19 with it and this.
    // The constants stay in registers.
    unsigned lo = 0x0000bf80u, hi = 0xbf800000u;
    asm("" : "+s"(lo), "+s"(hi));
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float a = __int_as_float(raw[q >> 1][2 * (q & 1)]) * SPLIT_SCALE, b = __int_as_float(raw[q >> 1][2 * (q & 1) + 1]) * SPLIT_SCALE;
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const unsigned u = pack_bf16x2(a, b);
            s.p[t][q] = (int)u;
            if (t == 2) break;
            a = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, u), __builtin_bit_cast(bf16x2_t, lo), a, false);
            b = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, u), __builtin_bit_cast(bf16x2_t, hi), b, false);
        }
    }
    return s;
}

// Sums of split products to their own scale; those that are not finite are done
// again with f32 MFMAs, operands straight from global memory: an operand is not
// finite, or the scaled sum overflows, and this gives what float32 arithmetic
// gives.  The finite sums of a tile are kept, so that a row's result does not
// depend on its neighbours.  A NaN in a row of A makes all its sums NaN: where one
// is among the first 32 (in a row that a LayerNorm or a map wrote all are), no
// products are needed, so that a state which has diverged costs little more than
// another (a float32 block at 8x90x180, C = 512: 6.1 to 6.5 ms, all NaN 18.1 with
// the products and 5.8 without).  Values and sums past the split's range cost
// both routes: M = 129600, N = 1536, K = 512 of 1e32 4.2 ms, 1.4 in range.
template <int TM, int TN>
__device__ void f32_finish(const float *A, const float *W, int M, int K, int r0, int n0, int g, int r16, f32x4 (&acc)[TN][TM]) {
    const float *ar[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) ar[i] = A + (size_t)min(r0 + 16 * i + r16, M - 1) * K + 8 * g;
    unsigned anan = 0;                                     // bit i: row 16 i + r16 has a NaN
    bool scanned = false;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        bool bad = false;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int c = 0; c < 4; ++c) bad |= !__builtin_isfinite(acc[j][i][c]);
        if (!__builtin_amdgcn_ballot_w64(bad)) {
#pragma unroll
            for (int i = 0; i < TM; ++i) acc[j][i] *= UNSPLIT;
            continue;
        }
        const float *wr = W + (size_t)(n0 + 16 * j + r16) * K + 8 * g;
        if (!scanned) {
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const f32x4 lo = *(const f32x4 *)ar[i], hi = *(const f32x4 *)(ar[i] + 4);
                bool nan = false;
#pragma unroll
                for (int c = 0; c < 4; ++c) nan |= __builtin_isnan(lo[c]) || __builtin_isnan(hi[c]);
                const unsigned long long m = __builtin_amdgcn_ballot_w64(nan) >> r16;      // the row's lanes: every 16th
                anan |= (m & 0x0001000100010001ull ? 1u : 0u) << i;
            }
            scanned = true;
        }
        bool todo = false;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int c = 0; c < 4; ++c) todo |= !__builtin_isfinite(acc[j][i][c]) && !(anan >> i & 1u);
        f32x4 t[TM];
#pragma unroll
        for (int i = 0; i < TM; ++i) t[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (__builtin_amdgcn_ballot_w64(todo))
            // lane group g contracts k = 8 g + s over the 8 steps s
            for (int k = 0; k < K; k += 32)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const f32x4 w = *(const f32x4 *)(wr + k + 4 * h);
#pragma unroll
                    for (int i = 0; i < TM; ++i) {
                        const f32x4 a = *(const f32x4 *)(ar[i] + k + 4 * h);
#pragma unroll
                        for (int s = 0; s < 4; ++s) t[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[s], a[s], t[i], 0, 0, 0);
                    }
                }
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                acc[j][i][c] = __builtin_isfinite(acc[j][i][c]) ? acc[j][i][c] * UNSPLIT
                                                                : (anan >> i & 1u ? __builtin_nanf("") : t[i][c]);
    }
}

// Epilogue of a V tile of the QKV projection (swapped operands): acc[j][i]
// holds tokens r0 + 16 i + 4 g + (0..3) (chunk rows) of V feature
// f0 + 16 j + r16 (head f >> 5, channel f & 31; V bias `bias`); each lane
// stores its four tokens' values in the blocked layout (plus the wrapped
// copies near lon 0 and X): 8 bytes of bf16, or (FP8) 4 e4m3 codes of
// value * out_mul[2] after the dequantization acc * a_dequant * w_dequant.
// Rows whose four tokens leave a lat row (X or the state size not a
// multiple of 4) are stored one by one.
template <int TM, int TN, bool FP8, typename F>
__device__ __forceinline__ void vt_epilogue(const EpiArgs &ep, const float *bias, int M, int r0, int f0,
                                            const f32x4 (&acc)[TN][TM], int g, int r16, F pre_store) {
    constexpr unsigned ES = FP8 ? 1 : 2;
    float bv[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) bv[j] = bias[f0 + 16 * j + r16];
    const float dq = FP8 ? ep.a_dequant * ep.w_dequant : 1.0f;
    const float om = FP8 ? ep.out_mul[2] : 1.0f;
    const int X = ep.vX, xp = ep.vxp, YX = ep.vY * ep.vX;
    pre_store();
    // element 0 of (head f0 / 32, state of the wave's first row); a head's plane, and a state's in it
    const unsigned b0 = udiv((unsigned)__builtin_amdgcn_readfirstlane(min(r0, M - 1) + ep.row0), ep.dT);
    const size_t state = (size_t)ep.vZ * ep.vY * xp * 32 * ES, plane = state * ep.vB;
    const unsigned char *vbase = (const unsigned char *)ep.vt + (size_t)__builtin_amdgcn_readfirstlane(f0 >> 5) * plane + b0 * state;
    // byte offset from vbase of position i of token row mg's (state, level, lat) row, channel r16
    auto row_off = [&](unsigned mg, int &x) -> unsigned {
        const unsigned b = udiv(mg, ep.dT), tt = mg - b * (unsigned)ep.T;
        const unsigned z = udiv(tt, ep.dYX), rr = tt - z * (unsigned)YX;
        const unsigned y = udiv(rr, ep.dX);
        x = (int)(rr - y * (unsigned)X);
        return (((b - b0) * (unsigned)ep.vZ + z) * (unsigned)ep.vY + y) * (unsigned)xp * (32 * ES) + (unsigned)r16 * 4 * ES;
    };
    if ((X & 3) == 0 && (ep.T & 3) == 0) {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int m4 = r0 + 16 * i + 4 * g;
            int x;
            const unsigned row = row_off((unsigned)(min(m4, M - 1) + ep.row0), x);
            const int i0 = x + 4;
            const bool in = m4 < M;
            const unsigned o0 = in ? row + (unsigned)(i0 >> 2) * 128 * ES : DROP;
            const unsigned o1 = in && i0 >= X ? row + (unsigned)((i0 - X) >> 2) * 128 * ES
                                              : (in && i0 + X < xp ? row + (unsigned)((i0 + X) >> 2) * 128 * ES : DROP);
            const unsigned o2 = in && i0 >= X && i0 + X < xp ? row + (unsigned)((i0 + X) >> 2) * 128 * ES : DROP;
            const bool wrap = __builtin_amdgcn_ballot_w64(o1 != DROP) != 0;
            const bool wrap2 = __builtin_amdgcn_ballot_w64(o2 != DROP) != 0;
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const RowSpan head(vbase + (j >> 1) * plane, DROP);
                const __amdgpu_buffer_rsrc_t rs = head.at((j & 1) * 64 * ES);      // from channel 16 (j & 1) of the head
                float e[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) e[k] = fmaf(acc[j][i][k], dq, bv[j]);
                if constexpr (FP8) {
                    const unsigned u = e4m3x4(e[0] * om, e[1] * om, e[2] * om, e[3] * om);
                    __builtin_amdgcn_raw_buffer_store_b32(u, rs, o0, 0, 0);
                    if (wrap) __builtin_amdgcn_raw_buffer_store_b32(u, rs, o1, 0, 0);
                    if (wrap2) __builtin_amdgcn_raw_buffer_store_b32(u, rs, o2, 0, 0);
                } else {
                    const u32x2 u = pack4_bf16(e);
                    __builtin_amdgcn_raw_buffer_store_b64(u, rs, o0, 0, 0);
                    if (wrap) __builtin_amdgcn_raw_buffer_store_b64(u, rs, o1, 0, 0);
                    if (wrap2) __builtin_amdgcn_raw_buffer_store_b64(u, rs, o2, 0, 0);
                }
            }
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int m4 = r0 + 16 * i + 4 * g;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (m4 + e >= M) break;
            int x;
            const unsigned row = row_off((unsigned)(m4 + e + ep.row0), x);
            const int i0 = x + 4;
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const float val = fmaf(acc[j][i][e], dq, bv[j]);
                unsigned char *vt = const_cast<unsigned char *>(vbase) + (j >> 1) * plane + row + (j & 1) * 64 * ES;
                auto put = [&](int p) {
                    const size_t o = ((size_t)(p >> 2) * 128 + (p & 3)) * ES;
                    if constexpr (FP8) vt[o] = (unsigned char)(e4m3x4(val * om, 0.f, 0.f, 0.f) & 0xffu);
                    else *(bf16 *)(vt + o) = (bf16)val;
                };
                put(i0);
                if (i0 - X >= 0) put(i0 - X);
                if (i0 + X < xp) put(i0 + X);
            }
        }
    }
}

// Workgroup barrier ordering LDS accesses only: the vector-memory loads and
// stores in flight (the next stage's loads) stay in flight.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Residual update of a wave's tiles: rows r0 + 16 i + r16, features
// n + 16 j + 4 g .. +3 of the float32 rows += acc * dq + bias; use(j, i, v)
// receives the updated values.  Two feature tiles at a time; with AHEAD the
// next pair's rows and bias are loaded before this pair's stores (a wait for a
// load also waits for the stores issued before it).  The wave's rows lie in
// one buffer, or in one state's; SPLIT: they may straddle states.
template <int TM, int TN, bool AHEAD, bool SPLIT, typename F>
__device__ __forceinline__ void resid_update(const EpiArgs &ep, int M, int N, int r0, int n, int g, int r16, float dq,
                                             const f32x4 (&acc)[TN][TM], F use) {
    const int rows = min(max(M - r0, 0), 16 * TM);
    RowSpan span(nullptr, 0);
    unsigned off[TM];
    float *xr[TM];
    if constexpr (SPLIT) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
            xr[i] = state_row(ep.resid, ep.resid_ptrs, (unsigned)ep.T, ep.dT, (unsigned)(min(r0 + 16 * i + r16, M - 1) + ep.row0), N) +
                    n + 4 * g;
    } else {
        const unsigned mg = (unsigned)__builtin_amdgcn_readfirstlane(min(r0, M - 1) + ep.row0);
        span = RowSpan(state_row(ep.resid, ep.resid_ptrs, (unsigned)ep.T, ep.dT, mg, N) + n, rows ? (unsigned)(rows * N - n) * 4u : 0u);
#pragma unroll
        for (int i = 0; i < TM; ++i) off[i] = (unsigned)((16 * i + r16) * N + 4 * g) * 4u;
    }
    f32x4 rz[1 + AHEAD][TM][2], bz[1 + AHEAD][2];
    auto load = [&](int j) {
        const int s = AHEAD ? (j >> 1) & 1 : 0;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            bz[s][h] = *(const f32x4 *)(ep.bias + n + 16 * (j + h) + 4 * g);
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                if constexpr (SPLIT) rz[s][i][h] = *(const f32x4 *)(xr[i] + 16 * (j + h));
                else rz[s][i][h] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(span.at(64 * (j + h)), off[i], 0, 0));
            }
        }
    };
    if (AHEAD) load(0);
#pragma unroll
    for (int j = 0; j < TN; j += 2) {
        if (!AHEAD) load(j);
        else if (j + 2 < TN) load(j + 2);
        const int s = AHEAD ? (j >> 1) & 1 : 0;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                f32x4 v;
                // explicit FMAs: the rounding of every element must not
                // depend on how the compiler contracts each unrolled copy
#pragma unroll
                for (int c = 0; c < 4; ++c) v[c] = rz[s][i][h][c] + fmaf(acc[j + h][i][c], dq, bz[s][h][c]);
                if constexpr (!SPLIT) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), span.at(64 * (j + h)), off[i], 0, 0);
                else if (r0 + 16 * i + r16 < M) *(f32x4 *)(xr[i] + 16 * (j + h)) = v;
                use(j + h, i, v);
            }
    }
}

// Epilogue of EPI_RESID_LN (LayerNorm fused into the residual update, WM3
// Sec. 2.1: a block's second LayerNorm reads the residual stream its
// out-projection has just updated).  The tile spans all N features
// of its rows.  A lane holds features ncol + 16 j + 4 g .. +3 of token
// row0w + 16 i + r16 (tile j, row tile i): the residual update of
// EPI_RESID, kept in acc, then the row statistics, summed in the lane (the
// tiles in order, each tile's 4 values pairwise), over the 4 lanes g
// (xsum16_32) and over the WGN waves of the row block through LDS, the
// same steps for every row, so a row's result does not depend on its
// position in the batch.  Two passes, as the LayerNorm kernel: the mean,
// then the mean square of the deviations.
// On gfx9 a wait for a load also waits for the stores issued before it:
// ln_g and ln_b are loaded before the first store and go through LDS, so
// that the normalized rows' stores wait for nothing (the updated rows are
// stored a pair of feature tiles at a time, as in the EPI_RESID epilogue:
// holding them to the end spills registers).
// `red` (LDS, 2 WGN BM + 2 N floats): row sums, then ln_g and ln_b.
template <int TM, int TN, int WGN, int BM, bool FP8, bool SPLIT>
__device__ __forceinline__ void resid_ln_epilogue(const EpiArgs &ep, int M, int N, int mt, int row0w, int wn, int ncol,
                                                  int g, int r16, int tid, int nth, f32x4 (&acc)[TN][TM], float *red) {
    const float dq = FP8 ? ep.a_dequant * ep.w_dequant : 1.0f;
    // this thread's share of ln_g and ln_b (N <= 2 nth)
    float lg[2], lb[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int c = tid + u * nth;
        lg[u] = c < N ? ep.ln_g[c] : 0.f;
        lb[u] = c < N ? ep.ln_b[c] : 0.f;
    }
    float s[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) s[i] = 0.f;
    resid_update<TM, TN, !SPLIT, SPLIT>(ep, M, N, mt + row0w, ncol, g, r16, dq, acc, [&](int j, int i, f32x4 v) {
        acc[j][i] = v;
        s[i] += (v[0] + v[1]) + (v[2] + v[3]);
    });
    // row sums across the lanes g and the waves: red[w][row], then
    // red[WGN + w][row]; ln_g and ln_b at red + 2 WGN BM
    const float invN = 1.0f / (float)N;
    float *const lgb = red + 2 * WGN * BM;
    float mean[TM], rstd[TM];
    lds_barrier();    // every wave is done with the stage slot that `red` lies in
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int c = tid + u * nth;
        if (c < N) {
            lgb[c] = lg[u];
            lgb[N + c] = lb[u];
        }
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        s[i] = xsum16_32(s[i]);
        if (g == 0) red[wn * BM + row0w + 16 * i + r16] = s[i];
    }
    lds_barrier();
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        float t = red[row0w + 16 * i + r16];
#pragma unroll
        for (int w = 1; w < WGN; ++w) t += red[w * BM + row0w + 16 * i + r16];
        mean[i] = t * invN;
        float q = 0.f;
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const float d = acc[j][i][c] - mean[i];
                q = fmaf(d, d, q);
            }
        q = xsum16_32(q);
        if (g == 0) red[(WGN + wn) * BM + row0w + 16 * i + r16] = q;
    }
    lds_barrier();
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        float t = red[WGN * BM + row0w + 16 * i + r16];
#pragma unroll
        for (int w = 1; w < WGN; ++w) t += red[(WGN + w) * BM + row0w + 16 * i + r16];
        rstd[i] = 1.0f / sqrtf(t * invN + ep.ln_eps);
    }
    // normalized rows: bf16, or e4m3 codes at the static scale *ln_amax / 448
    const float inv = FP8 ? (*ep.ln_amax > 0.f ? 448.0f / *ep.ln_amax : 1.0f) : 1.0f;
    constexpr unsigned ES = FP8 ? 1 : 2;
    const int r0 = mt + row0w, rows = min(max(M - r0, 0), 16 * TM);
    const RowSpan span((const unsigned char *)ep.ln_out + ((size_t)(r0 + ep.row0) * N + ncol) * ES,
                       rows ? (unsigned)(rows * N - ncol) * ES : 0u);
    unsigned off[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) off[i] = (unsigned)((16 * i + r16) * N + 4 * g) * ES;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int n = ncol + 16 * j + 4 * g;
        const float4 gm = *(const float4 *)(lgb + n), bt = *(const float4 *)(lgb + N + n);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const f32x4 a = acc[j][i];
            // explicit FMAs, as in the LayerNorm kernel
            float y[4];
            y[0] = fmaf((a[0] - mean[i]) * rstd[i], gm.x, bt.x) * inv;
            y[1] = fmaf((a[1] - mean[i]) * rstd[i], gm.y, bt.y) * inv;
            y[2] = fmaf((a[2] - mean[i]) * rstd[i], gm.z, bt.z) * inv;
            y[3] = fmaf((a[3] - mean[i]) * rstd[i], gm.w, bt.w) * inv;
            if constexpr (FP8) __builtin_amdgcn_raw_buffer_store_b32(e4m3x4(y[0], y[1], y[2], y[3]), span.at(16 * j * ES), off[i], 0, 0);
            else __builtin_amdgcn_raw_buffer_store_b64(pack4_bf16(y), span.at(16 * j * ES), off[i], 0, 0);
        }
    }
}

// Epilogue of a wave's TM x TN tiles of every kind but EPI_RESID_LN and the
// swapped V tiles: rows r0 + 16 i + r16 (of the chunk), features
// n0 + ncol + 16 j + .. (n0: first feature of the workgroup's tile).  PERM
// (permuted W rows, EpiArgs.perm): the pair of tiles j, j + 1 covers features
// 16 j + 8 g .. +7 of each lane, stored at once (16 bytes of bf16, or 8 e4m3
// codes in the FP8 kernels, whose permuted outputs are codes); else tile j
// covers 16 j + 4 g .. +3.  The bias is loaded before the first store (on
// gfx9 a wait for a load also waits for every store issued before it).
// `pre_store` runs once before the first store.  All arithmetic is explicit
// FMAs: the rounding of an element must not depend on how the compiler
// contracts each unrolled copy (a token's result must not depend on its
// position in the tile, i.e. on the batch).
template <int EPI, bool FP8, bool PERM, int TM, int TN, typename F>
__device__ __forceinline__ void tile_epilogue(const EpiArgs &ep, int M, int N, int r0, int n0, int ncol, int g, int r16,
                                              const f32x4 (&acc)[TN][TM], F pre_store) {
    const float dq = FP8 ? ep.a_dequant * ep.w_dequant : 1.0f;
    if constexpr (epi_resid(EPI)) {
        pre_store();
        resid_update<TM, TN, EPI == EPI_RESID, EPI == EPI_RESID_SPLIT>(ep, M, N, r0, n0 + ncol, g, r16, dq, acc, [](int, int, f32x4) {});
        return;
    } else {
    constexpr bool OUT8 = FP8 && PERM;
    constexpr unsigned ES = OUT8 ? 1 : 2;
    constexpr int NP = PERM ? 8 : 4;          // consecutive features per lane
    // a feature tile never straddles Q/K/V (C is a multiple of BN)
    const int part = epi_qkv(EPI) ? ep.part0 + n0 / ep.C : 0;
    const int rows = min(max(M - r0, 0), 16 * TM);
    const int rs_len = epi_qkv(EPI) ? 32 : N;              // elements per row of the output
    float om = 1.0f;
    if constexpr (epi_qkv(EPI)) om = (part == 0 ? ep.qscale : 1.0f) * (OUT8 ? ep.out_mul[part] : 1.0f);
    else if constexpr (OUT8) om = ep.out_mul[0];
    // the wave's first row, and (QKV) its first head's plane in [3][H][M][32]
    const unsigned char *base = (const unsigned char *)ep.out;
    size_t pair = 32 * ES;                                 // bytes from a pair of feature tiles to the next
    unsigned bytes;
    if constexpr (epi_qkv(EPI)) {
        const int hc = n0 + ncol - (part - ep.part0) * ep.C;
        base += (((size_t)part * ep.H + (hc >> 5)) * ep.Mtot + r0 + ep.row0) * 32 * ES;
        pair = (size_t)ep.Mtot * 32 * ES;
        bytes = (unsigned)(rows * 32) * ES;
    } else {
        base += ((size_t)(r0 + ep.row0) * N + n0 + ncol) * ES;
        bytes = rows ? (unsigned)(rows * N - n0 - ncol) * ES : 0u;
    }
    unsigned off[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) off[i] = (unsigned)((16 * i + r16) * rs_len + NP * g) * ES;
    // rotary (cos, sin) of each row's channel pairs 4g .. 4g+3 (the same
    // pairs in every head this lane stores), loaded once per tile
    float2 rc[TM][4];
    if constexpr (EPI == EPI_QKV_ROPE) {
        if (part < 2) {
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const long mg = (long)min(r0 + 16 * i + r16, M - 1) + ep.row0;
                const unsigned tt = (unsigned)(mg % ep.T);
                const unsigned yx = (unsigned)(ep.rY * ep.rX);
                const int z = (int)(tt / yx), y = (int)((tt / (unsigned)ep.rX) % (unsigned)ep.rY),
                          x = (int)(tt % (unsigned)ep.rX);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int pr = 4 * g + q;
                    const int row = pr < 4 ? z : (pr < 10 ? ep.rZ + y : ep.rZ + ep.rY + x);
                    rc[i][q] = *(const float2 *)(ep.rope + 2 * (row * 16 + pr));
                }
            }
        }
    }
    f32x4 bz[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j)
        bz[j] = *(const f32x4 *)(ep.bias + n0 + ncol + 16 * (j & ~1) + (PERM ? 8 * g + 4 * (j & 1) : 4 * g + 16 * (j & 1)));
    pre_store();
#pragma unroll
    for (int j = 0; j < TN; j += 2) {
        const RowSpan span(base + (epi_qkv(EPI) ? (j >> 1) * pair : 0), bytes);
        const __amdgpu_buffer_rsrc_t rs = span.at(epi_qkv(EPI) ? 0 : 16 * j * ES);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            float v[8];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                v[c] = fmaf(acc[j][i][c], dq, bz[j][c]);
                v[4 + c] = fmaf(acc[j + 1][i][c], dq, bz[j + 1][c]);
            }
            if constexpr (EPI == EPI_QKV_ROPE) {
                if (part < 2) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const float a0 = v[2 * q], a1 = v[2 * q + 1];
                        v[2 * q] = fmaf(a0, rc[i][q].x, -(a1 * rc[i][q].y));
                        v[2 * q + 1] = fmaf(a0, rc[i][q].y, a1 * rc[i][q].x);
                    }
                }
            }
            if constexpr (EPI == EPI_GELU) {
#pragma unroll
                for (int c = 0; c < 8; ++c) v[c] = gelu_as4(v[c]);
            }
            if constexpr (EPI == EPI_GELU_28) {
#pragma unroll
                for (int c = 0; c < 8; ++c) v[c] = gelu_as(v[c]);
            }
            if constexpr (epi_qkv(EPI) || OUT8) {
#pragma unroll
                for (int c = 0; c < 8; ++c) v[c] *= om;
            }
            if constexpr (OUT8)
                __builtin_amdgcn_raw_buffer_store_b64(u32x2{e4m3x4(v[0], v[1], v[2], v[3]), e4m3x4(v[4], v[5], v[6], v[7])}, rs, off[i], 0, 0);
            else if constexpr (PERM)
                __builtin_amdgcn_raw_buffer_store_b128(pack8_bf16(v), rs, off[i], 0, 0);
            else {
                __builtin_amdgcn_raw_buffer_store_b64(pack4_bf16(v), rs, off[i], 0, 0);
                __builtin_amdgcn_raw_buffer_store_b64(pack4_bf16(v + 4), span.at((epi_qkv(EPI) ? 0 : 16 * j * ES) + 32), off[i], 0, 0);
            }
        }
    }
    }
}

// tile_epilogue of the float32 kernels: every kind but EPI_RESID stores
// float32 (16 bytes per lane, row and feature tile); W rows in natural order.
template <int EPI, int TM, int TN>
__device__ __forceinline__ void tile_epilogue_f32(const EpiArgs &ep, int M, int N, int r0, int n0, int ncol, int g, int r16,
                                                  const f32x4 (&acc)[TN][TM]) {
    if constexpr (epi_resid(EPI)) {
        resid_update<TM, TN, false, EPI == EPI_RESID_SPLIT>(ep, M, N, r0, n0 + ncol, g, r16, 1.0f, acc, [](int, int, f32x4) {});
        return;
    } else {
    const int part = epi_qkv(EPI) ? ep.part0 + n0 / ep.C : 0;
    const int rows = min(max(M - r0, 0), 16 * TM);
    const int rs_len = epi_qkv(EPI) ? 32 : N;
    const float om = epi_qkv(EPI) && part == 0 ? ep.qscale : 1.0f;
    const float *base = (const float *)ep.out;
    size_t pair = 0;
    unsigned bytes;
    if constexpr (epi_qkv(EPI)) {
        const int hc = n0 + ncol - (part - ep.part0) * ep.C;
        base += (((size_t)part * ep.H + (hc >> 5)) * ep.Mtot + r0 + ep.row0) * 32;
        pair = (size_t)ep.Mtot * 32;
        bytes = (unsigned)(rows * 32) * 4u;
    } else {
        base += (size_t)(r0 + ep.row0) * N + n0 + ncol;
        bytes = rows ? (unsigned)(rows * N - n0 - ncol) * 4u : 0u;
    }
    unsigned off[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) off[i] = (unsigned)((16 * i + r16) * rs_len + 4 * g) * 4u;
    // rotary (cos, sin) of each row's channel pairs 2g, 2g+1 and 8 + 2g, 9 + 2g
    float2 rc[TM][4];
    if constexpr (EPI == EPI_QKV_ROPE) {
        if (part < 2) {
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const long mg = (long)min(r0 + 16 * i + r16, M - 1) + ep.row0;
                const unsigned tt = (unsigned)(mg % ep.T);
                const unsigned yx = (unsigned)(ep.rY * ep.rX);
                const int z = (int)(tt / yx), y = (int)((tt / (unsigned)ep.rX) % (unsigned)ep.rY),
                          x = (int)(tt % (unsigned)ep.rX);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int pr = 8 * (q >> 1) + 2 * g + (q & 1);
                    const int row = pr < 4 ? z : (pr < 10 ? ep.rZ + y : ep.rZ + ep.rY + x);
                    rc[i][q] = *(const float2 *)(ep.rope + 2 * (row * 16 + pr));
                }
            }
        }
    }
    f32x4 bz[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) bz[j] = *(const f32x4 *)(ep.bias + n0 + ncol + 16 * j + 4 * g);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const RowSpan span(base + (epi_qkv(EPI) ? (j >> 1) * pair : 0), bytes);
        const __amdgpu_buffer_rsrc_t rs = span.at(epi_qkv(EPI) ? 64 * (j & 1) : 64 * j);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            f32x4 v;
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] = acc[j][i][c] + bz[j][c];
            if constexpr (EPI == EPI_QKV_ROPE) {
                if (part < 2) {
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        const float2 cs = rc[i][2 * (j & 1) + q];
                        const float a = v[2 * q], b = v[2 * q + 1];
                        v[2 * q] = fmaf(a, cs.x, -(b * cs.y));
                        v[2 * q + 1] = fmaf(a, cs.y, b * cs.x);
                    }
                }
            }
            if constexpr (epi_qkv(EPI)) {
                if (part == 0) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) v[c] *= om;
                }
            }
            if constexpr (EPI == EPI_GELU) {
#pragma unroll
                for (int c = 0; c < 4; ++c) v[c] = gelu_as(v[c]);
            }
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rs, off[i], 0, 0);
        }
    }
    }
}

// The narrow tiles: WGM x WGN waves compute one BM x BN tile, OCC workgroups
// share a CU, and the activation and weight tiles of each K stage stream
// through two slots, one stage ahead of the MFMAs.
enum OperandType : int { T_BF16 = 0, T_E4M3 = 1, T_F32 = 2 };
template <int BM, int BN, int WGM, int WGN, int OCC, int EPI, int TY, bool PERM>
__global__ __launch_bounds__(64 * WGM * WGN, OCC) void gemm_lds_kernel(const void *__restrict__ A, const void *__restrict__ W,
                                                         int M, int N, int K, EpiArgs ep, int, int) {
#if defined(__HIP_DEVICE_COMPILE__)   // LDS-address-space builtins exist only in the device pass
    constexpr int BKB = 128;
    constexpr bool FP8 = TY == T_E4M3, F32 = TY == T_F32;
    constexpr bool HALVES = FP8 || F32;            // a lane's 32 bytes of a row: chunks 2 g and 2 g + 1
    constexpr int NW = WGM * WGN;
    constexpr int WM = BM / WGM, WN = BN / WGN;
    constexpr int TM = WM / 16, TN = WN / 16;
    constexpr int SLOT = (BM + BN) * BKB;          // one stage: the activation rows, then the weight rows
    constexpr int LPA = BM / 8 / NW;               // load instructions (8 rows) per wave and stage
    constexpr int LPB = BN / 8 / NW;
    static_assert(BM % (8 * NW) == 0 && BN % (8 * NW) == 0, "rows per stage must split over the waves");
    static_assert(WM % 16 == 0 && WN % 32 == 0, "wave tile");
    extern __shared__ __align__(16) unsigned char smem[];

    const int ntn = N / BN, ntm = (M + BM - 1) / BM;
    const int total = ntn * ntm;
    const int per = (total + 7) >> 3;
    const int L = blockIdx.x;
    const int id = (L & 7) * per + (L >> 3);
    if (id >= total) return;
    const int m0 = (id / ntn) * BM, n0 = (id % ntn) * BN;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WGM, wn = wave / WGM;
    const int g = lane >> 4, r16 = lane & 15;
    const unsigned Kb = (unsigned)K * (F32 ? 4 : (FP8 ? 1 : 2));
    const __amdgpu_buffer_rsrc_t ars = make_rsrc(A, (unsigned)M * Kb);
    const __amdgpu_buffer_rsrc_t wrs = make_rsrc(W, (unsigned)N * Kb);

    // per-lane global byte offsets: instruction i of wave w fills rows
    // 8 (w + NW i) .. +7 of a slot's part
    unsigned voa[LPA], vob[LPB];
#pragma unroll
    for (int i = 0; i < LPA; ++i) {
        const int row = 8 * (wave + NW * i) + (lane >> 3);
        voa[i] = (unsigned)(m0 + row) * Kb + (((lane & 7) ^ swz<HALVES>(row)) << 4);
    }
#pragma unroll
    for (int i = 0; i < LPB; ++i) {
        const int row = 8 * (wave + NW * i) + (lane >> 3);
        vob[i] = (unsigned)(n0 + row) * Kb + (((lane & 7) ^ swz<HALVES>(row)) << 4);
    }
    const int nk = (int)(Kb / BKB);
    int lslot = 0;
    unsigned lk = 0;
    auto load = [&]() {
        unsigned char *dst = smem + lslot * SLOT;
#pragma unroll
        for (int i = 0; i < LPA; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(ars, (lds_void *)(dst + 1024 * (wave + NW * i)), 16, voa[i], lk, 0, 0);
#pragma unroll
        for (int i = 0; i < LPB; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wrs, (lds_void *)(dst + BM * BKB + 1024 * (wave + NW * i)), 16, vob[i], lk, 0, 0);
        lk += BKB;
        lslot ^= 1;
    };

    // fragment chunks of a row: as in gemm_pp_kernel
    int aoff[2], woff[2];
#pragma unroll
    for (int o = 0; o < 2; ++o) {
        const int pc = (HALVES ? 2 * g + o : 4 * o + g) ^ swz<HALVES>(r16);
        aoff[o] = (wm * WM + r16) * BKB + (pc << 4);
        woff[o] = BM * BKB + (wn * WN + r16) * BKB + (pc << 4);
    }

    load();

    // SWAP (the V tiles of a QKV projection with ep.vt set): swapped MFMA
    // operands and the blocked-layout epilogue.
    auto body = [&](auto swap_tag) {
    constexpr bool SWAP = decltype(swap_tag)::value;
    f32x4 acc[TN][TM];
    int slot = 0;
    auto stage = [&](auto first_tag, int kt) {
        constexpr bool FIRST = decltype(first_tag)::value;
        // This wave's loads of stage kt have landed; the barrier then makes all
        // waves' parts of it visible and frees the slot read in stage kt - 1.
        wait_vmcnt<0>();
        __builtin_amdgcn_s_barrier();
        if (kt + 1 < nk) load();
        const unsigned char *sl = smem + slot * SLOT;
        slot ^= 1;
        // (typed reads: see gemm_pp_kernel)
        i32x4 a[TM][2], w[TN][2];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int o = 0; o < 2; ++o) a[i][o] = *(const i32x4 *)(sl + aoff[o] + 16 * i * BKB);
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int o = 0; o < 2; ++o) w[j][o] = *(const i32x4 *)(sl + woff[o] + 16 * j * BKB);
        __builtin_amdgcn_s_setprio(1);
        if constexpr (FP8) {
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int i = 0; i < TM; ++i) acc[j][i] = mma_fp8<FIRST, SWAP>(w[j], a[i], acc[j][i]);
        } else if constexpr (F32) {
            Split3 as[TM];
#pragma unroll
            for (int i = 0; i < TM; ++i) as[i] = split3(a[i]);
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const Split3 ws = split3(w[j]);
                // (part of W, part of A), smallest products first
                constexpr int pw[6] = {2, 0, 1, 1, 0, 0}, pa[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
                for (int t = 0; t < 6; ++t)
#pragma unroll
                    for (int i = 0; i < TM; ++i)
                        acc[j][i] = t == 0 ? mma_bf16<FIRST, false>(ws.p[pw[t]], as[i].p[pa[t]], acc[j][i])
                                           : mma_bf16<false, false>(ws.p[pw[t]], as[i].p[pa[t]], acc[j][i]);
            }
        } else {
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int i = 0; i < TM; ++i) acc[j][i] = mma_bf16<FIRST, SWAP>(w[j][0], a[i][0], acc[j][i]);
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int i = 0; i < TM; ++i) acc[j][i] = mma_bf16<false, SWAP>(w[j][1], a[i][1], acc[j][i]);
        }
        __builtin_amdgcn_s_setprio(0);
    };
    stage(std::true_type{}, 0);
    for (int kt = 1; kt < nk; ++kt) stage(std::false_type{}, kt);
    if constexpr (F32) {
        f32_finish<TM, TN>((const float *)A, (const float *)W, M, K, m0 + wm * WM, n0 + wn * WN, g, r16, acc);
        tile_epilogue_f32<EPI, TM, TN>(ep, M, N, m0 + wm * WM, n0, wn * WN, g, r16, acc);
    } else if constexpr (epi_resid_ln(EPI)) {
        static_assert((2 * WGN * BM + 2 * BN) * 4 <= SLOT && BN <= 2 * NW * 64, "row sums and ln_g, ln_b fit a slot");
        resid_ln_epilogue<TM, TN, WGN, BM, FP8, EPI == EPI_RESID_LN_SPLIT>(ep, M, N, m0, wm * WM, wn, wn * WN, g, r16, tid, NW * 64,
                                                                           acc, (float *)smem);
    } else if constexpr (SWAP) {
        vt_epilogue<TM, TN, FP8>(ep, ep.bias + 2 * ep.C, M, m0 + wm * WM, n0 - 2 * ep.C + wn * WN, acc, g, r16, [] {});
    } else {
        tile_epilogue<EPI, FP8, PERM, TM, TN>(ep, M, N, m0 + wm * WM, n0, wn * WN, g, r16, acc, [] {});
    }
    };
    if constexpr (epi_qkv(EPI) && !F32) {
        if (ep.vt && n0 >= 2 * ep.C) {
            body(std::true_type{});
            return;
        }
    }
    body(std::false_type{});
#endif
}

// ---------------------------------------------------------------------------
// Ping-pong kernel: the main loop of the wide tiles.  8 waves, wave tile
// 64 x 128 (TM = 4, TN = 8), two per SIMD: waves 0-3 (group 0) and 4-7
// (group 1).  A K stage (128 bytes per row) is two phases; in each a wave
// first reads fragments from LDS and issues loads (memory part), then runs
// 32 bf16 (or 16 f8f6f4) MFMAs on registers (matrix part), with a workgroup
// barrier after each part.  Group 1 runs one part behind group 0, so on every
// SIMD one wave's MFMAs cover the other wave's LDS reads.
//
// An LDS slot holds one stage in three sub-tiles that are read, and refilled,
// one after the other: A, W03 and W47 (feature tiles 0..3 and 4..7 of every
// wave).  Stage st:
//   phase 0: reads A(st), W03(st)   A x W03   loads W47(st + 1)
//   phase 1: reads W47(st)          A x W47   loads A(st + 2), W03(st + 2)
// so the sub-tiles read in one phase are free (both groups are past it) in
// the next, where the loads that refill them are issued: those have five to
// six parts (about 2800 MFMA cycles) to land.  A wave waits, one barrier ahead
// of group 0's read, until at most the loads issued after those it needs are
// outstanding (loads return in order).
// Every accumulator sees its k-steps in the order of gemm_lds_kernel, so the
// two kernels agree bit for bit.
template <int BM, int BN, int EPI, bool FP8, bool PERM>
__global__ __launch_bounds__(512, 1) void gemm_pp_kernel(const void *__restrict__ A, const void *__restrict__ W,
                                                         int M, int N, int K, EpiArgs ep, int tpw, int rw) {
#if defined(__HIP_DEVICE_COMPILE__)   // LDS-address-space builtins exist only in the device pass
    constexpr int TM = 4, TN = 8, BKB = 128;
    constexpr int WGM = BM / 64, WGN = BN / 128;
    static_assert(WGM * WGN == 8, "8 waves of 64 x 128");
    constexpr int AB = BM * BKB, WH = BN / 2 * BKB;          // bytes of sub-tile A, and of W03 or W47
    constexpr int SLOT = AB + 2 * WH;
    constexpr int LA = BM / 64, LW = BN / 2 / 64;            // load instructions (8 rows) per wave and sub-tile
    extern __shared__ __align__(16) unsigned char smem[];

    const int ntn = N / BN, ntm = (M + BM - 1) / BM;
    const int ngrp = rw ? (ntm + tpw - 1) / tpw : (ntn + tpw - 1) / tpw;
    const int total = rw ? ngrp * ntn : ngrp * ntm;
    const int per = (total + 7) >> 3;
    const int L = blockIdx.x;
    const int id = (L & 7) * per + (L >> 3);
    if (id >= total) return;
    const int m0 = rw ? (id / ntn) * tpw * BM : (id / ngrp) * BM;
    const int tn0 = rw ? id % ntn : (id % ngrp) * tpw;
    // (EPI_RESID_LN: one, see the launcher)
    const int nn = epi_resid_ln(EPI) ? 1 : (rw ? min(tpw, ntm - m0 / BM) : min(tpw, ntn - tn0));

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = wave >> 2;
    const int wm = wave % WGM, wn = wave / WGM;
    const int g = lane >> 4, r16 = lane & 15;
    const unsigned Kb = (unsigned)K * (FP8 ? 1 : 2);
    const unsigned astep = rw ? (unsigned)BM * Kb : 0u, wstep = rw ? 0u : (unsigned)BN * Kb;
    const __amdgpu_buffer_rsrc_t ars = make_rsrc(A, (unsigned)M * Kb);
    const __amdgpu_buffer_rsrc_t wrs = make_rsrc(W, (unsigned)N * Kb);

    // load instruction u of this wave fills sub-tile rows 8 (wave + 8 u) ..;
    // sub-tile row r of W03 is tile row 128 (r / 64) + r % 64 (W47: + 64)
    unsigned voa[LA], vow[LW];
    const int lrow = lane >> 3;
#pragma unroll
    for (int u = 0; u < LA; ++u) {
        const int r = 8 * (wave + 8 * u) + lrow;
        voa[u] = (unsigned)(m0 + r) * Kb + (((lane & 7) ^ swz<FP8>(r)) << 4);
    }
#pragma unroll
    for (int u = 0; u < LW; ++u) {
        const int r = 8 * (wave + 8 * u) + lrow;
        vow[u] = (unsigned)(tn0 * BN + ((r >> 6) << 7) + (r & 63)) * Kb + (((lane & 7) ^ swz<FP8>(r)) << 4);
    }
    const int nk = (int)(Kb / BKB);
    const int S = nn * nk;
    // the next stage of A and W03 (cursor 0) and of W47 (cursor 1): its slot
    // and the byte offsets of its tile and k
    int lkt[2] = {0, 0}, ls[2] = {0, 0};
    unsigned lk[2] = {0, 0}, lslot[2] = {0, 0}, la = 0, lw[2] = {0, 0};
    auto advance = [&](int c) {
        ++ls[c];
        lslot[c] ^= SLOT;
        lk[c] += BKB;
        if (++lkt[c] == nk) {
            lkt[c] = 0;
            lk[c] = 0;
            lw[c] += wstep;
            if (c == 0) la += astep;
        }
    };
    auto load_w = [&](int h) {      // W03 (h = 0) or W47
#pragma unroll
        for (int u = 0; u < LW; ++u)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wrs, (lds_void *)(smem + lslot[h] + AB + h * WH + 1024 * (wave + 8 * u)),
                                                     16, vow[u], lw[h] + lk[h] + (h ? 64u * Kb : 0u), 0, 0);
    };
    auto load_aw = [&]() {          // A and W03 (A's row advance in the vector offset: rows past M must read zero)
#pragma unroll
        for (int u = 0; u < LA; ++u)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(ars, (lds_void *)(smem + lslot[0] + 1024 * (wave + 8 * u)), 16,
                                                     voa[u] + la, lk[0], 0, 0);
        load_w(0);
        advance(0);
    };

    // fragment chunks of a row: bf16 k-step o reads chunk 4 o + g, e4m3 the
    // chunks 2 g and 2 g + 1 of its one k-step
    int aoff[2], woff[2];
#pragma unroll
    for (int o = 0; o < 2; ++o) {
        const int pc = (FP8 ? 2 * g + o : 4 * o + g) ^ swz<FP8>(r16);
        aoff[o] = (wm * 64 + r16) * BKB + (pc << 4);
        woff[o] = AB + (wn * 64 + r16) * BKB + (pc << 4);
    }

    load_aw();
    load_w(1);
    advance(1);
    if (S > 1) load_aw();
    // A and W03 of stage 0 have landed
    if (S > 1) wait_vmcnt<LA + 2 * LW>();
    else wait_vmcnt<LW>();
    __builtin_amdgcn_s_barrier();

    auto body = [&](auto swap_tag) {
    constexpr bool SWAP = decltype(swap_tag)::value;
    f32x4 acc[TN][TM];
    // LDS is read as ext_vector values: before a read of a struct type (uint4)
    // the compiler waits for every LDS load in flight
    i32x4 a[TM][2], w[4][2];      // A and the current half of W: [tile][chunk]
    auto read_a = [&](const unsigned char *sl) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int o = 0; o < 2; ++o) a[i][o] = *(const i32x4 *)(sl + aoff[o] + 16 * i * BKB);
    };
    auto read_w = [&](const unsigned char *sl) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int o = 0; o < 2; ++o) w[j][o] = *(const i32x4 *)(sl + woff[o] + 16 * j * BKB);
    };
    // the matrix part: every row tile by feature tiles j0 .. j0 + 3
    auto mma = [&](auto first_tag, int j0) {
        constexpr bool FIRST = decltype(first_tag)::value;
        __builtin_amdgcn_s_setprio(1);
        if constexpr (FP8) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int i = 0; i < TM; ++i) acc[j0 + j][i] = mma_fp8<FIRST, SWAP>(w[j], a[i], acc[j0 + j][i]);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int i = 0; i < TM; ++i) acc[j0 + j][i] = mma_bf16<FIRST, SWAP>(w[j][0], a[i][0], acc[j0 + j][i]);
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int i = 0; i < TM; ++i) acc[j0 + j][i] = mma_bf16<false, SWAP>(w[j][1], a[i][1], acc[j0 + j][i]);
        }
        __builtin_amdgcn_s_setprio(0);
    };
    int st = 0;                  // global stage
    unsigned slot = 0;
    // wait for the sub-tiles of the phase after phase q of stage st
    auto wait_next = [&](int q) {
        if (st + 1 + q < S) wait_vmcnt<LA + 2 * LW>();
        else if (q) wait_vmcnt<LW>();
        else wait_vmcnt<0>();
    };
    // end of a part (skip: those sub-tiles have landed before the last epilogue)
    auto end_mem = [&](int q, bool skip) {
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0xc07f);      // lgkmcnt(0)
        if (grp == 1 && !skip) wait_next(q);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };
    auto end_mma = [&](int q, bool skip, bool last) {
        __builtin_amdgcn_sched_barrier(0);
        if (grp == 0 && !skip) wait_next(q);
        // (group 1 started the tile one barrier later and ends it without one)
        if (!(last && grp == 1)) __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };
    auto stage = [&](auto first_tag, bool skip, bool last) {
        const unsigned char *sl = smem + slot;
        read_a(sl);
        read_w(sl);                                  // W03
        if (ls[1] < S) {
            load_w(1);
            advance(1);
        }
        end_mem(0, skip);
        mma(first_tag, 0);
        end_mma(0, skip, false);
        read_w(sl + WH);                             // W47
        if (ls[0] < S) load_aw();
        end_mem(1, skip);
        mma(first_tag, 4);
        end_mma(1, skip, last);
        slot ^= SLOT;
        ++st;
    };
    for (int t = 0; t < nn; ++t) {
        if (grp == 1) __builtin_amdgcn_s_barrier();  // one part behind group 0
        stage(std::true_type{}, t > 0, nk == 1);
        for (int kt = 1; kt < nk; ++kt) stage(std::false_type{}, false, kt == nk - 1);
        const int n0 = (rw ? tn0 : tn0 + t) * BN;
        const int mt = rw ? m0 + t * BM : m0;        // first row of this tile
        // The loads in flight belong to the next tile.  They are waited for
        // before the first store, since a later wait for them would also wait
        // for the stores; the first phases of the next tile then wait for none.
        auto pre_store = [] { wait_vmcnt<0>(); };
        if constexpr (epi_resid_ln(EPI)) {
            // one tile per workgroup (the launcher): no load is in flight, and
            // both groups are past their last LDS read
            static_assert((2 * WGN * BM + 2 * BN) * 4 <= SLOT && BN <= 1024, "row sums and ln_g, ln_b fit a slot");
            resid_ln_epilogue<TM, TN, WGN, BM, FP8, EPI == EPI_RESID_LN_SPLIT>(ep, M, N, mt, wm * 64, wn, wn * 128, g, r16, tid, 512, acc, (float *)smem);
        } else if constexpr (SWAP) {
            vt_epilogue<TM, TN, FP8>(ep, ep.bias + 2 * ep.C, M, mt + wm * 64, n0 - 2 * ep.C + wn * 128, acc, g, r16, pre_store);
        } else {
            tile_epilogue<EPI, FP8, PERM, TM, TN>(ep, M, N, mt + wm * 64, n0, wn * 128, g, r16, acc, pre_store);
        }
        if (t + 1 < nn) __builtin_amdgcn_s_barrier();    // every wave's loads for the next phases have landed
    }
    };
    if constexpr (epi_qkv(EPI)) {
        if (ep.vt && tn0 * BN >= 2 * ep.C) {
            body(std::true_type{});
            return;
        }
    }
    body(std::false_type{});
#endif
}

// Launches `kernel` for every row chunk: A is addressed with 32-bit byte
// offsets from the chunk's first row, so M is split into row chunks below
// 2 GiB of A.  tpw_req tiles per workgroup, walking feature tiles (rw = 0)
// or row blocks (rw = 1).
typedef void (*gemm_fn)(const void *, const void *, int, int, int, EpiArgs, int, int);
inline hipError_t launch_chunks(gemm_fn kernel, int BM, int BN, int nth, size_t lds, size_t row_bytes, const void *A,
                                const void *W, int M, int N, int K, const EpiArgs &ep, int tpw_req, int rw,
                                hipStream_t stream) {
    const int ntn = N / BN;
    const int chunk = (int)std::min<size_t>((size_t)M, ((size_t)0x7fffffff / row_bytes) / BM * BM);
    for (int r0 = 0; r0 < M; r0 += chunk) {
        const int Mc = std::min(chunk, M - r0);
        EpiArgs e = ep;
        e.row0 = r0;
        e.Mtot = M;
        const void *Ac = (const unsigned char *)A + (size_t)r0 * row_bytes;
        const int ntm = (Mc + BM - 1) / BM;
        const int tpw = std::max(1, std::min(tpw_req, rw ? ntm : ntn));
        const int total = rw ? ((ntm + tpw - 1) / tpw) * ntn : ((ntn + tpw - 1) / tpw) * ntm;
        const int grid = ((total + 7) >> 3) << 3;
        kernel<<<grid, nth, lds, stream>>>(Ac, W, Mc, N, K, e, tpw, rw);
        const hipError_t err = hipGetLastError();
        if (err != hipSuccess) return err;
    }
    return hipSuccess;
}

// The instantiation of a kernel family F for an epilogue kind: permuted W
// rows (perm) exist for the QKV and GELU epilogues, rotary only with them.
template <typename F>
inline gemm_fn pick_natural(EpiKind epi, const EpiArgs &ep) {
    switch (epi) {
    case EPI_QKV: return F::template get<EPI_QKV, false>();
    case EPI_QKV_ROPE: return F::template get<EPI_QKV_ROPE, false>();
    case EPI_GELU: return F::template get<EPI_GELU, false>();
    case EPI_RESID: return splits(ep) ? F::template get<EPI_RESID_SPLIT, false>() : F::template get<EPI_RESID, false>();
    case EPI_STORE: return F::template get<EPI_STORE, false>();
    default: return nullptr;
    }
}
template <typename F>
inline gemm_fn pick(EpiKind epi, const EpiArgs &ep) {
    const int perm = ep.perm;
    switch (epi) {
    case EPI_QKV: return perm ? F::template get<EPI_QKV, true>() : F::template get<EPI_QKV, false>();
    case EPI_QKV_ROPE: return perm ? F::template get<EPI_QKV_ROPE, true>() : nullptr;
    case EPI_GELU: return perm ? F::template get<EPI_GELU, true>() : F::template get<EPI_GELU, false>();
    case EPI_RESID:
        if (perm) return nullptr;
        return splits(ep) ? F::template get<EPI_RESID_SPLIT, false>() : F::template get<EPI_RESID, false>();
    case EPI_STORE: return perm ? nullptr : F::template get<EPI_STORE, false>();
    default: return nullptr;
    }
}

// LDS limit of a kernel, set once per process and kernel (a local static's
// initialisation is thread-safe; the server thread launches too).
template <size_t LDS, typename K>
inline gemm_fn with_lds(K kernel) {
    return hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS) == hipSuccess
               ? (gemm_fn)kernel : nullptr;
}

template <int BM, int BN, int WGM, int WGN, int OCC, int TY>
struct LdsGemm {
    static constexpr size_t lds = (size_t)2 * (BM + BN) * 128;
    static_assert(lds * OCC <= 160 * 1024, "LDS per CU");
    template <int EPI, bool PERM>
    static gemm_fn get() {
        static const gemm_fn f = with_lds<lds>(gemm_lds_kernel<BM, BN, WGM, WGN, OCC, EPI, TY, PERM>);
        return f;
    }
};

template <int BM, int BN, bool FP8>
struct PpGemm {
    static constexpr size_t lds = (size_t)2 * (BM + BN) * 128;
    template <int EPI, bool PERM>
    static gemm_fn get() {
        static const gemm_fn f = with_lds<lds>(gemm_pp_kernel<BM, BN, EPI, FP8, PERM>);
        return f;
    }
};

template <bool FP8>
hipError_t launch_tiles(const void *A, const void *W, int M, int N, int K, EpiKind epi, const EpiArgs &ep, hipStream_t stream) {
    const size_t row_bytes = (size_t)K * (FP8 ? 1 : 2);
    // a QKV feature tile must not straddle two of Q, K and V (BN divides C),
    // and a workgroup's must be all V or none when V goes to the blocked layout
    const bool n256 = N % 256 == 0 && (!epi_qkv(epi) || ep.C % 256 == 0);
    const int wmax = epi_qkv(epi) && ep.vt ? ((ep.C / 256) % 2 ? 1 : 2) : wide_max(N);
    const TilePlan t = N % 128 == 0 ? plan_tiles(M, N, (int)(row_bytes / 128), n256, wmax, epi == EPI_RESID) : TilePlan{64, 1, 0};
    auto run = [&](auto tag, int BM, int BN, int nth) -> hipError_t {
        typedef decltype(tag) G;
        const gemm_fn f = pick<G>(epi, ep);
        if (!f) return hipErrorInvalidValue;
        return launch_chunks(f, BM, BN, nth, G::lds, row_bytes, A, W, M, N, K, ep, t.tpw, t.rw, stream);
    };
    typedef LdsGemm<64, 64, 2, 2, 4, FP8 ? T_E4M3 : T_BF16> G64;
    if constexpr (!FP8)
        if (epi == EPI_GELU && N % 128 && !ep.perm) {
            const gemm_fn f = G64::template get<EPI_GELU_28, false>();
            if (!f) return hipErrorInvalidValue;
            return launch_chunks(f, 64, 64, 256, G64::lds, row_bytes, A, W, M, N, K, ep, 1, 0, stream);
        }
    if (t.bm == 256) return run(PpGemm<256, 256, FP8>{}, 256, 256, 512);
    if (t.bm == 128) return run(LdsGemm<128, 128, 2, 2, 2, FP8 ? T_E4M3 : T_BF16>{}, 128, 128, 256);
    return run(G64{}, 64, 64, 256);
}

// EPI_RESID_LN: the tile spans N = 512; one row block per workgroup (the row
// sums use the stage slots, which a next tile's loads would be filling).  64
// rows while that gives every workgroup a CU (M = 14400, bf16: 28 us against
// 41 with 128 rows, which fill half the CUs; M = 21600: 49 against 44).  The
// row sums run over the same lanes and waves in both.
template <bool FP8>
hipError_t launch_resid_ln(const void *A, const void *W, int M, int N, int K, const EpiArgs &ep, hipStream_t stream) {
    auto run = [&](auto tag, int BM) -> hipError_t {
        typedef decltype(tag) G;
        const gemm_fn f = splits(ep) ? G::template get<EPI_RESID_LN_SPLIT, false>() : G::template get<EPI_RESID_LN, false>();
        if (!f) return hipErrorInvalidValue;
        return launch_chunks(f, BM, 512, 512, G::lds, (size_t)K * (FP8 ? 1 : 2), A, W, M, N, K, ep, 1, 1, stream);
    };
    if (M <= 64 * 256) return run(LdsGemm<64, 512, 2, 4, 1, FP8 ? T_E4M3 : T_BF16>{}, 64);
    return run(PpGemm<128, 512, FP8>{}, 128);
}

// float32: 128 x 128 tiles once they give every CU one, else 64 x 64 (at 276
// tiles of 128 x 128, M = 2880, N = 1536, K = 512: 52 against 46 us; at 368,
// N = 2048: 54 against 55; at 816, M = 8640, N = 1536: 101 against 111).
inline hipError_t launch_f32(const void *A, const void *W, int M, int N, int K, EpiKind epi, const EpiArgs &ep, hipStream_t stream) {
    auto run = [&](auto tag, int B) -> hipError_t {
        typedef decltype(tag) G;
        const gemm_fn f = pick_natural<G>(epi, ep);
        if (!f) return hipErrorInvalidValue;
        return launch_chunks(f, B, B, 256, G::lds, (size_t)K * 4, A, W, M, N, K, ep, 1, 0, stream);
    };
    const bool n128 = N % 128 == 0 && (!epi_qkv(epi) || ep.C % 128 == 0);
    if (n128 && (long)((M + 127) / 128) * (N / 128) > 300) return run(LdsGemm<128, 128, 2, 2, 2, T_F32>{}, 128);
    return run(LdsGemm<64, 64, 2, 2, 4, T_F32>{}, 64);
}

}  // namespace glds

using namespace glds;

bool gemm_lds_applies(int M, int N, int K) {
    (void)M;
    return N % 64 == 0 && K % 64 == 0 && (unsigned long long)N * K * 2 < (1ull << 31);
}

hipError_t launch_gemm_lds(const void *A, const void *W, int M, int N, int K, EpiKind epi, const EpiArgs &ep,
                           hipStream_t stream) {
    if (ep.out8) return hipErrorInvalidValue;
    if (epi == EPI_RESID_LN) {
        if (!gemm_resid_ln_applies(N) || ep.perm || !ep.ln_g || !ep.ln_b || !ep.ln_out) return hipErrorInvalidValue;
        return launch_resid_ln<false>(A, W, M, N, K, ep, stream);
    }
    return launch_tiles<false>(A, W, M, N, K, epi, ep, stream);
}

hipError_t launch_gemm_f32(const void *A, const void *W, int M, int N, int K, EpiKind epi, const EpiArgs &ep,
                           hipStream_t stream) {
    if (ep.perm || ep.vt || ep.out8) return hipErrorInvalidValue;
    return launch_f32(A, W, M, N, K, epi, ep, stream);
}

hipError_t launch_gemm_fp8(const void *A, const void *W, int M, int N, int K, EpiKind epi, const EpiArgs &ep,
                           hipStream_t stream) {
    if (M <= 0) return hipSuccess;
    if (N % 128 || K % 128 || (unsigned long long)N * K >= (1ull << 31)) return hipErrorInvalidValue;
    if (epi == EPI_RESID_LN) {
        // as in launch_gemm_lds; the LayerNorm output as e4m3 codes (out8) at
        // a given scale
        if (!gemm_resid_ln_applies(N) || !ep.out8 || !ep.ln_amax || ep.perm || !ep.ln_g || !ep.ln_b || !ep.ln_out)
            return hipErrorInvalidValue;
        return launch_resid_ln<true>(A, W, M, N, K, ep, stream);
    }
    if (!ep.out8 != !ep.perm) return hipErrorInvalidValue;   // e4m3 outputs go with permuted W rows
    return launch_tiles<true>(A, W, M, N, K, epi, ep, stream);
}

}  // namespace wm
