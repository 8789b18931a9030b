// 3-D neighborhood attention with relative-position bias on MFMA.
//
// WeatherMesh-3 Sec. 2.1 (NATTEN) and App. A.2: every latent token attends
// to the Kz x Ky x Kx box around it over (level, lat, lon); lon wraps, lat
// and level windows keep their size and shift inward at the borders.
//
// Work split: one wave owns a group of 16 queries -- 4 levels x 2 lats x
// 2 lons -- and one head.  The union of the 16 windows (the group halo) is
// walked in chunks of 32 keys.  Per chunk:
//   S^T[32 keys x 16 queries] = K_chunk . Q^T       (MFMA, d = 32 contracted)
//   mask + bias, online softmax in float32 (base-2 exponent)
//   O^T[32 d x 16 queries] += V^T_chunk . P^T         (MFMA, keys contracted)
// Computing S transposed makes each lane own one query column in both the
// score tile and the output tile, so the softmax state (running max, sum)
// of a query lives in the 4 lanes l, l^16, l^32, l^48.
//
// MFMA lane layouts (16x16 tiles; lane l, g = l/16, r = l%16):
//   bf16 16x16x32: A[r][8g..8g+7], B[8g..8g+7][r], D[4g..4g+3][r]
//   f32  16x16x4 : A[r][g],        B[g][r],        D[4g..4g+3][r]
// A lane's 8 scores in a chunk are keys {4g..4g+3, 16+4g..16+4g+3}; the
// P.V contraction takes its k index in that same order (k-slot 8g + 4j + i
// <-> key 16j + 4g + i), so the score registers feed the second MFMA
// without any data movement.
#include <algorithm>
#include <cmath>

#include "kernels.hpp"

namespace wm {
namespace {

constexpr int GZ = 4, GY = 2, GX = 2;   // query group shape (16 queries)

struct Axis {
    int lo;      // first halo coordinate (may be negative on a periodic axis)
    int n;       // halo length
    int ws;      // this lane's window start, in halo slots
    int boff;    // bias index of halo slot s = s + boff
    int N;       // axis length
    bool per;
};

__device__ __forceinline__ Axis make_axis(int g0, int gsize, int qi, int N, int K, bool per) {
    Axis a;
    a.N = N;
    a.per = per;
    const int r = (K - 1) >> 1;
    if (per) {
        a.lo = g0 - r;
        a.n = gsize + K - 1;
        a.ws = qi - g0;
        a.boff = r - a.ws;
    } else {
        const int last = min(g0 + gsize - 1, N - 1);
        a.lo = win_start(g0, N, K, false);
        a.n = win_start(last, N, K, false) + K - a.lo;
        a.ws = win_start(qi, N, K, false) - a.lo;
        a.boff = a.lo - qi + K - 1;
    }
    return a;
}

__device__ __forceinline__ int coord(const Axis &a, int s) {
    int c = a.lo + s;
    if (a.per) {
        c %= a.N;
        c = c < 0 ? c + a.N : c;
    }
    return c;
}

// Vector loads and stores at the element's own alignment (the caller's tensors
// need no more; the hardware takes any).
template <typename T, int N>
struct Vec {
    typedef T type __attribute__((ext_vector_type(N), aligned(sizeof(T))));
};

constexpr int UB = 512;                 // halo units (level, lat, 4 lons) per pass: whole chunks of 8
constexpr int BIAS_LDS = 8192;          // longest bias table (floats) that is copied to LDS

// A workgroup: nw waves (four, or fewer where lon has fewer groups), groups of
// the same levels and lats that follow each other in lon.  The units of their
// common halo -- 4 lon slots of one (level, lat) -- are listed in LDS, UB at a
// time, with the offset of their row; so are the lon slots of each wave and the
// head's bias table.  A key's address is then
// one addition and a chunk has no divisions or wrap-arounds.  What bounds it:
// the f32 MFMAs (32 of 32 cycles per chunk) and as many cycles of other
// instructions beside them.  K is loaded one chunk ahead.  A lane takes V
// channels 2 r and 2 r + 1 (8 bytes of f32, 4 of bf16), so a key's 32 channels
// are one run per 16 lanes and a lane's output is 8 consecutive channels.
// The softmax reference follows the maximum only when it is passed by 2^SLACK;
// in bf16 at once, so that probabilities are rounded at the same place whatever
// came before.
//   FAR: rows beyond 32-bit byte offsets, or too many lon slots for the table:
//   row and slot hold tokens and the address is computed in 64 bits.
template <typename T, bool FAR>
__global__ __launch_bounds__(256, 4) void nat_generic_kernel(NatArgs p, long first, long count, int ngq, int nw, int nslot, bool bias_lds) {
    __shared__ i32x4 unit[UB + 8];                 // row offset, slots on the level and lat axes, first lon slot
    extern __shared__ __align__(16) float dyn[];                 // [nw][nslot] lon offsets (not FAR), then 4 + table + 8 biases
    const int ngz = (p.Z + GZ - 1) / GZ, ngy = (p.Y + GY - 1) / GY, ngx = (p.X + GX - 1) / GX;
    const int L = blockIdx.x, nth = 64 * nw;
    long t = (long)(L & 7) * (gridDim.x >> 3) + (L >> 3);      // XCD-aware: neighbours share an L2
    if (t >= count) return;
    t += first;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, g = lane >> 4, r16 = lane & 15;
    const int gxw = nw * (int)(t % ngq) + wave; t /= ngq;
    const int gy = (int)(t % ngy); t /= ngy;
    const int gz = (int)(t % ngz); t /= ngz;
    const int h = (int)(t % p.H); t /= p.H;
    const int b = (int)t;
    const int gx = min(gxw, ngx - 1);
    const int z0 = gz * GZ, y0 = gy * GY, x0 = gx * GX;

    const int zq = z0 + (r16 >> 2), yq = y0 + ((r16 >> 1) & 1), xq = x0 + (r16 & 1);
    const bool active = gxw < ngx && zq < p.Z && yq < p.Y && xq < p.X;
    const int zc = min(zq, p.Z - 1), yc = min(yq, p.Y - 1), xc = min(xq, p.X - 1);

    const Axis az = make_axis(z0, GZ, zc, p.Z, p.Kz, p.periodic & 1);
    const Axis ay = make_axis(y0, GY, yc, p.Y, p.Ky, (p.periodic >> 1) & 1);
    const Axis ax = make_axis(x0, GX, xc, p.X, p.Kx, (p.periodic >> 2) & 1);
    const int nx4 = nslot >> 2;                    // units per (level, lat)
    const int nunit = az.n * ay.n * nx4;
    const int By = 2 * p.Ky - 1, Bx = 2 * p.Kx - 1, tbl = (2 * p.Kz - 1) * By * Bx;
    const float *rpb = p.rpb + (size_t)h * tbl;
    const int bias0 = (az.boff * By + ay.boff) * Bx + ax.boff;
    const unsigned tsb = (unsigned)p.ts * (unsigned)sizeof(T);     // (used where offsets fit 32 bits)

    const T *qb = (const T *)p.q + (size_t)b * p.bs + (size_t)h * p.hs;
    const T *kb = (const T *)p.k + (size_t)b * p.bs + (size_t)h * p.hs;
    const T *vb = (const T *)p.v + (size_t)b * p.bs + (size_t)h * p.hs;
    const long qtok = ((long)zc * p.Y + yc) * p.X + xc;

    typedef typename Vec<T, 8>::type T8;
    typedef typename Vec<T, 2>::type T2;
    const T8 qf = *(const T8 *)(qb + qtok * p.ts + 8 * g);    // channels 8g .. of this lane's query

    unsigned *lons = (unsigned *)dyn + wave * nslot;
    float *bias_s = dyn + (FAR ? 0 : nw * nslot) + 4;
    // lon of slot s (a slot past the halo: slot 0's, a key of the halo; its score is masked)
    auto lon = [&](int s) { return coord(ax, s < ax.n ? s : 0); };
    if constexpr (!FAR)
        for (int e = lane; e < nslot; e += 64) lons[e] = (unsigned)lon(e) * tsb;
    if (bias_lds)
        for (int e = (int)threadIdx.x - 4; e < tbl + 8; e += nth)
            bias_s[e] = e >= 0 && e < tbl ? rpb[e] * p.bscale : 0.f;
    auto load_k = [&](unsigned off, int slot) {
        if constexpr (FAR) return *(const T8 *)(kb + (long)((int)off + lon(slot)) * p.ts + 8 * g);
        else return *(const T8 *)((const char *)kb + (off + lons[slot] + 8u * g * (unsigned)sizeof(T)));
    };

    constexpr float SLACK = sizeof(T) == 2 ? 0.f : 8.f;
    const float NEG = -INFINITY;
    float m_run = -1e30f, l_run = 0.f;
    f32x4 o0 = {0.f, 0.f, 0.f, 0.f}, o1 = {0.f, 0.f, 0.f, 0.f};

    for (int ub = 0; ub < nunit; ub += UB) {
        const int nu = min(UB, nunit - ub), nchunk = (nu + 7) >> 3;
        if (ub > 0) __syncthreads();
        for (int e = threadIdx.x; e < 8 * nchunk; e += nth) {
            const int u = min(ub + e, nunit - 1), row = u / nx4;
            const int sz = row / ay.n, sy = row - sz * ay.n;
            const unsigned tok = (unsigned)(coord(az, sz) * p.Y + coord(ay, sy)) * (unsigned)p.X;
            unit[e] = i32x4{(int)(FAR ? tok : tok * tsb), e < nu ? sz : 0x3fffffff, sy, 4 * (u - row * nx4)};
        }
        __syncthreads();
        T8 kn[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const i32x4 u = unit[4 * j + (r16 >> 2)];
            kn[j] = load_k((unsigned)u[0], u[3] + (r16 & 3));
        }
        for (int c = 0; c < nchunk; ++c) {
            const T8 kf[2] = {kn[0], kn[1]};
            // keys f = 32 c + 16 j + 4 g + i of this lane: V, bias and window
            T2 vv[2][4];
            float bias[2][4];
            int xw[2];                             // lon slot in the window; beyond it where level or lat are
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const i32x4 u = unit[8 * c + 4 * j + g];
                const bool zyok = (unsigned)(u[1] - az.ws) < (unsigned)p.Kz && (unsigned)(u[2] - ay.ws) < (unsigned)p.Ky;
                xw[j] = zyok ? u[3] - ax.ws : 0x3fffffff;
                const int bo = zyok ? (u[1] * By + u[2]) * Bx + u[3] + bias0 : 0;
                if constexpr (FAR) {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        vv[j][i] = *(const T2 *)(vb + (long)(u[0] + lon(u[3] + i)) * p.ts + 2 * r16);
                } else {
                    const i32x4 x = *(const i32x4 *)(lons + u[3]);
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        vv[j][i] = *(const T2 *)((const char *)vb +
                                                 ((unsigned)u[0] + (unsigned)x[i] + 2u * r16 * (unsigned)sizeof(T)));
                }
                if (bias_lds) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) bias[j][i] = bias_s[bo + i];
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i) bias[j][i] = rpb[max(0, min(bo + i, tbl - 1))] * p.bscale;
                }
            }
            if (c + 1 < nchunk) {
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const i32x4 u = unit[8 * c + 8 + 4 * j + (r16 >> 2)];
                    kn[j] = load_k((unsigned)u[0], u[3] + (r16 & 3));
                }
            }
            // ---- scores S^T = K . Q^T ----
            f32x4 sacc[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                sacc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
                if constexpr (sizeof(T) == 2) {
                    sacc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf[j]),
                                                                      __builtin_bit_cast(bf16x8, qf), sacc[j], 0, 0, 0);
                } else {
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        sacc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[j][e], qf[e], sacc[j], 0, 0, 0);
                }
            }
            // ---- mask + bias, online softmax ----
            float s[2][4];
            float cmax = NEG;
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const bool ok = (unsigned)(xw[j] + i) < (unsigned)p.Kx;
                    s[j][i] = ok ? fmaf(sacc[j][i], p.qscale, bias[j][i]) : NEG;
                    cmax = fmaxf(cmax, s[j][i]);
                }
            float alpha = 1.f;
            if (__builtin_amdgcn_ballot_w64(cmax > m_run + SLACK)) {
                cmax = fmaxf(cmax, __shfl_xor(cmax, 16, 64));
                cmax = fmaxf(cmax, __shfl_xor(cmax, 32, 64));
                const float m_new = fmaxf(m_run, cmax);
                alpha = __builtin_amdgcn_exp2f(m_run - m_new);
                m_run = m_new;
#pragma unroll
                for (int i = 0; i < 4; ++i) { o0[i] *= alpha; o1[i] *= alpha; }
            }
            float pv[2][4];
            float psum = 0.f;
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    pv[j][i] = __builtin_amdgcn_exp2f(s[j][i] - m_run);
                    psum += pv[j][i];
                }
            l_run = fmaf(l_run, alpha, psum);
            // ---- O^T += V^T . P^T ----
            if constexpr (sizeof(T) == 2) {
                uint4 v0, v1;
                bf16x8 pw;
                unsigned d[8];
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        d[4 * j + i] = __builtin_bit_cast(unsigned, vv[j][i]);
                        pw[4 * j + i] = f2bf(pv[j][i]);
                    }
                v0 = make_uint4(__builtin_amdgcn_perm(d[1], d[0], 0x05040100u), __builtin_amdgcn_perm(d[3], d[2], 0x05040100u),
                                __builtin_amdgcn_perm(d[5], d[4], 0x05040100u), __builtin_amdgcn_perm(d[7], d[6], 0x05040100u));
                v1 = make_uint4(__builtin_amdgcn_perm(d[1], d[0], 0x07060302u), __builtin_amdgcn_perm(d[3], d[2], 0x07060302u),
                                __builtin_amdgcn_perm(d[5], d[4], 0x07060302u), __builtin_amdgcn_perm(d[7], d[6], 0x07060302u));
                o0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, v0), pw, o0, 0, 0, 0);
                o1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, v1), pw, o1, 0, 0, 0);
            } else {
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        o0 = __builtin_amdgcn_mfma_f32_16x16x4f32(vv[j][i][0], pv[j][i], o0, 0, 0, 0);
                        o1 = __builtin_amdgcn_mfma_f32_16x16x4f32(vv[j][i][1], pv[j][i], o1, 0, 0, 0);
                    }
            }
        }
    }
    float l_tot = l_run + __shfl_xor(l_run, 16, 64);
    l_tot += __shfl_xor(l_tot, 32, 64);
    const float inv = 1.0f / l_tot;
    if (active) {
        T8 o;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (sizeof(T) == 2) {
                o[2 * i] = f2bf(o0[i] * inv);
                o[2 * i + 1] = f2bf(o1[i] * inv);
            } else {
                o[2 * i] = o0[i] * inv;
                o[2 * i + 1] = o1[i] * inv;
            }
        }
        *(T8 *)((T *)p.out + (size_t)b * p.obs + (size_t)qtok * p.ots + h * 32 + 8 * g) = o;
    }
}

}  // namespace

hipError_t launch_nat(const NatArgs &a, bool bf16in, hipStream_t stream) {
    if (bf16in) {
        const size_t lds = nat_tile_lds_bytes(a);
        if (lds > 0 && lds <= 160 * 1024) return launch_nat_tile(a, stream);
    }
    // e4m3 contractions exist only in the tiled kernel: never fall back to
    // bf16 arithmetic for a caller that asked for them
    if (a.amax) return hipErrorNotSupported;
    return launch_nat_generic(a, bf16in, stream);
}

hipError_t launch_nat_generic(const NatArgs &a, bool bf16in, hipStream_t stream) {
    if (a.vt || a.q8 || a.o8) return hipErrorInvalidValue;     // reads token-major bf16/f32 q, k, v only
    // Workgroups of up to four lon groups, as even as they come: a wave without a
    // group would walk a halo for nothing (float32, 8 heads, window 3x5x1, us, four
    // waves always / these: 8x512x1 tokens 61.4 / 20.0, 8x512x2 61.6 / 20.3).
    const int ngx = (a.X + GX - 1) / GX, ngq = (ngx + 3) / 4, nw = (ngx + ngq - 1) / ngq;
    const long total = (long)((a.Z + GZ - 1) / GZ) * ((a.Y + GY - 1) / GY) * ngq * a.H * a.B;
    if (total == 0) return hipSuccess;
    const int nslot = (GX + a.Kx - 1 + 3) & ~3;
    const long tbl = (long)(2 * a.Kz - 1) * (2 * a.Ky - 1) * (2 * a.Kx - 1);
    const size_t span = (size_t)a.Z * a.Y * a.X * (size_t)a.ts * (bf16in ? 2 : 4);
    const bool far = span >= (1ull << 32) || nslot > 1024;
    const bool bias_lds = tbl <= BIAS_LDS;
    const size_t lds = (far ? 0 : 4 * (size_t)nw * nslot) + (bias_lds ? 4 * (size_t)(tbl + 12) : 0);
    const long most = 0x7fffffff / (64 * nw) & ~7;      // workgroups per launch: a grid has less than 2^31 threads
    auto go = [&](auto kernel) {
        for (long first = 0; first < total; first += most) {
            const long count = std::min(most, total - first);
            kernel<<<(unsigned)((count + 7) & ~7L), 64 * nw, lds, stream>>>(a, first, count, ngq, nw, nslot, bias_lds);
        }
    };
    if (bf16in) far ? go(nat_generic_kernel<bf16, true>) : go(nat_generic_kernel<bf16, false>);
    else far ? go(nat_generic_kernel<float, true>) : go(nat_generic_kernel<float, false>);
    return hipGetLastError();
}

}  // namespace wm
