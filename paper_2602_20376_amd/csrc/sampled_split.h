// Fused scorer on the matrix core from split FP32 values, K = 2, 3, 4 and
// 2 <= r <= 4: both w = V c and s = V^H z are matrix products whose operands
// hold V, c and z without loss of FP32 grade.  Internal header, included
// after sampled_kernels.h by sampled.hip and sampled_probe.hip.
#pragma once

#include "sampled_kernels.h"

namespace lrqo {
namespace {

// The FP32 scorer spends 4r (real V) or 8r (complex) FMAs per row and
// candidate on the vector ALU, two cycles each, and is bound by that issue.
// Here per 32 rows x 32 candidates (1,024 row-candidates) and wave:
//
//   w = V c    v_mfma_f32_32x32x16_f16, one chain for Re w and one for Im w.
//              A row of V is scaled by a power of two (labels depend on the
//              direction of w alone) and split into F16 parts
//              V = V1 + V2 + V3, c likewise; k-slot tau C + x holds product
//              tau of component x (C components per row: r real, 2r complex).
//              Products V1c1, V2c1, V1c2, V2c2, V3c1 leave an error of
//              0.48u to 0.58u root-mean-square relative to sum_j |V_ij c_j|
//              (u = 2^-24), all eight 0.22u to 0.36u; the FP32 scorer's chain
//              of FMAs has 0.44u to 0.46u, and with the rounded factor
//              sqrt(3) on c (K = 3; here that factor enters before the split)
//              about 0.55u.  Five are used where they fill the k-slots of a
//              chunk that six would not fit, the others get six or more.
//   labels     sign bits only.  K = 3: u = |Im w| - sqrt(3) Re w (label 0 iff
//              u < 0) and Im w; K = 4: the direction is turned by
//              e^{-i pi/4}, so the labels are the quadrants; K = 2: Re w.
//              v_perm_b32 spreads the signs of four rows over the bytes of a
//              dword as 0 / -1.
//   s = V^H z  v_mfma_i32_32x32x32_i8 of those masks against V in 30-bit
//              fixed point (one scale for the whole factor, four balanced
//              base-256 digits per value: 4C <= 32 rows of the operand).  The
//              sums are exact integers, so the only error is the rounding of
//              V to 2^-30 of its largest entry; the digits of a component are
//              put together once per candidate.
//
// Layouts (lane l, h = l / 32): operand rows/columns l % 32, F16 k-slots
// 8h .. 8h+7, I8 k-slots 16h .. 16h+15; result register i is row
// 8 (i / 4) + 4h + i % 4, column l % 32.  The byte b of label dword d of a
// lane is therefore row 8d + 4h + b, and the I8 operand holds that row in
// k-slot 16h + 4d + b: no lane exchange between the two products.
typedef float v16f __attribute__((ext_vector_type(16)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));

constexpr int kSplitBlock = 512;                           // eight waves of 32 candidates
constexpr int kSplitCands = kSplitBlock / kWave * 32;      // candidates of a block
constexpr int kSplitTile = 256;                            // rows staged at a time
constexpr int64_t kSplitMaxRows = (int64_t)1 << 23;        // rows of a slice: |digit| <= 128 keeps I32 sums exact

template <int R, bool REAL>
struct SplitShape {
    static constexpr int C = REAL ? R : 2 * R;
    static constexpr int NCH = C == 2 || C == 3 ? 1 : (C == 4 || C == 6 ? 2 : 3);   // chunks of 16 k-slots
    static constexpr int NP = 16 * NCH / C < 8 ? 16 * NCH / C : 8;                  // products kept
};
// Parts (0, 1, 2) of V and of c in product tau, by falling size.
__host__ __device__ constexpr int split_v(int tau) { return tau == 1 || tau == 3 || tau == 7 ? 1 : (tau == 4 || tau == 6 ? 2 : 0); }
__host__ __device__ constexpr int split_c(int tau) { return tau == 2 || tau == 3 || tau == 6 ? 1 : (tau == 5 || tau == 7 ? 2 : 0); }
// I8 operand rows of component x: digit p at row 4 * slot + p.  A lane's
// result registers hold slots h, 2 + h, 4 + h, 6 + h: Re and Im of a column
// (complex V) go to the same lane.
template <int R, bool REAL>
__host__ __device__ constexpr int split_slot(int x) {
    if (REAL) return x;
    const int j = x < R ? x : x - R;
    return (j & 1) + 4 * (j >> 1) + (x < R ? 0 : 2);
}

__device__ __forceinline__ void split3(double x, _Float16 (&p)[3]) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        p[k] = static_cast<_Float16>(static_cast<float>(x));
        x -= static_cast<double>(static_cast<float>(p[k]));
    }
}
__device__ __forceinline__ void split3(float x, _Float16 (&p)[3]) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        p[k] = static_cast<_Float16>(x);
        x -= static_cast<float>(p[k]);
    }
}

// Signs of a[i .. i+3] as bytes 0 / -1, as two halves to be or-ed.
__device__ __forceinline__ uint32_t signs_lo(float a, float b) {
    return __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x0c0c0b09u);
}
__device__ __forceinline__ uint32_t signs_hi(float a, float b) {
    return __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x0b090c0cu);
}

// Exponent e of the largest |V| entry (prologue's per-block maxima): V enters
// the I8 operand as round(V 2^(29-e)), below 2^30 in size.
__device__ __forceinline__ int split_exponent(const float* vmax, int count) {
    float m = 0.0f;
    for (int k = (int)(threadIdx.x & (kWave - 1)); k < count; k += kWave) m = fmaxf(m, vmax[k]);
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, kWave));
    return m > 0.0f && isfinite(m) ? ilogbf(m) : 0;
}

template <int R, bool REAL, int KS, bool PROBE>
__global__ __launch_bounds__(kSplitBlock, 4) void k_score_split(ScoreParams p) {
    using Sh = SplitShape<R, REAL>;
    constexpr int C = Sh::C, NCH = Sh::NCH, NP = Sh::NP;
    constexpr int NB = kSplitTile / 32;                  // 32-row blocks of a tile
    constexpr int NPL = KS == 2 ? 1 : 2;                 // label planes
    __shared__ __align__(16) v8h aw[2][NB][NCH][64];     // F16 operand of w: [buffer][block][chunk][lane]
    __shared__ __align__(16) signed char as[2][NB][64][16];   // I8 operand of s: [buffer][block][lane][k-slot]
    __shared__ long long tot[kSplitTile / kWave][C];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int h = lane >> 5;
    const int ev = split_exponent(p.vmax, p.vmax_count);
    // rows of the I8 operand that no component uses stay zero
    for (int e = tid; e < (int)(sizeof(as) / 16); e += kSplitBlock)
        reinterpret_cast<v4i*>(as)[e] = v4i{0, 0, 0, 0};

    // ---- this lane's candidate (lanes l and l + 32 share one): B operands
    const uint32_t idx = blockIdx.x * (uint32_t)kSplitCands + wave * 32 + (lane & 31);
    v8h bre[NCH], bim[NCH];
    int slot[1];
    {
        float c[1][2 * R];
        lane_directions<R, 1, PROBE>(p, idx, 0, blockIdx.y == 0 && h == 0, c, slot);
        double x[C], y[C];                               // factors of the components in Re w, Im w
#pragma unroll
        for (int j = 0; j < R; ++j) {
            double cr = c[0][2 * j] * 0x1p14, ci = c[0][2 * j + 1] * 0x1p14;
            if constexpr (KS == 4) {                     // c e^{-i pi/4}
                const double t = 0.70710678118654752 * (cr + ci);
                ci = 0.70710678118654752 * (ci - cr);
                cr = t;
            }
            const double sr = KS == 3 ? -1.7320508075688772 : 1.0;   // K = 3: -sqrt(3) Re w
            x[j] = sr * cr;
            y[j] = ci;
            if constexpr (!REAL) {
                x[R + j] = -sr * ci;
                y[R + j] = cr;
            }
        }
        _Float16 px[C][3], py[C][3];
#pragma unroll
        for (int k = 0; k < C; ++k) {
            split3(x[k], px[k]);
            split3(y[k], py[k]);
        }
#pragma unroll
        for (int ch = 0; ch < NCH; ++ch)
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                _Float16 r[2], i[2];
#pragma unroll
                for (int g = 0; g < 2; ++g) {
                    const int ks = 16 * ch + 8 * g + t, tau = ks / C;
                    r[g] = tau < NP ? px[ks % C][split_c(tau)] : (_Float16)0.0f;
                    i[g] = tau < NP ? py[ks % C][split_c(tau)] : (_Float16)0.0f;
                }
                bre[ch][t] = h ? r[1] : r[0];
                bim[ch][t] = h ? i[1] : i[0];
            }
    }

    v16i acc[NPL];
#pragma unroll
    for (int q = 0; q < NPL; ++q)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[q][i] = 0;

    // ---- tiles: threads 0..255 write the F16 operand of a row, 256..511 its I8 operand
    const int64_t r0 = (int64_t)blockIdx.y * p.rows_per_slice;
    const int64_t r1 = min(p.n, r0 + p.rows_per_slice);
    const int row = tid & (kSplitTile - 1);
    const bool fixed = tid >= kSplitTile;
    float v[C];                                          // REAL: V_ij; complex: Re V_ij, then Im V_ij
    auto fetch = [&](int64_t t0) {
        const bool in = t0 + row < r1;
        const float* __restrict__ src = p.V + (t0 + row) * C;
#pragma unroll
        for (int k = 0; k < C; ++k) {
            const int x = REAL ? k : ((k & 1) ? R + k / 2 : k / 2);
            v[x] = in ? src[k] : 0.0f;
        }
    };
    long long ts[C];
#pragma unroll
    for (int k = 0; k < C; ++k) ts[k] = 0;
    auto stage = [&](int buf) {
        const int blk = row >> 5, rr = row & 31;
        if (!fixed) {
            float m = fabsf(v[0]);
#pragma unroll
            for (int k = 1; k < C; ++k) m = fmaxf(m, fabsf(v[k]));
            const int e = m > 0.0f ? 14 - ilogbf(m) : 0;
            _Float16 pv[C][3];
#pragma unroll
            for (int k = 0; k < C; ++k) split3(ldexpf(v[k], e), pv[k]);
#pragma unroll
            for (int ch = 0; ch < NCH; ++ch)
#pragma unroll
                for (int g = 0; g < 2; ++g) {
                    v8h a;
#pragma unroll
                    for (int t = 0; t < 8; ++t) {
                        const int ks = 16 * ch + 8 * g + t, tau = ks / C;
                        a[t] = tau < NP ? pv[ks % C][split_v(tau)] : (_Float16)0.0f;
                    }
                    aw[buf][blk][ch][32 * g + rr] = a;
                }
        } else {
            const int d = rr >> 3, g = (rr >> 2) & 1, b = rr & 3;
#pragma unroll
            for (int k = 0; k < C; ++k) {
                const int q = __float2int_rn(ldexpf(v[k], 29 - ev));
                ts[k] += q;
                const uint32_t dig = ((uint32_t)q + 0x00808080u) ^ 0x00808080u;   // balanced digits, lowest first
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    as[buf][blk][32 * g + 4 * split_slot<R, REAL>(k) + t][4 * d + b] = (signed char)(dig >> (8 * t));
            }
        }
    };

    fetch(r0);
    __syncthreads();                                     // the zeroed operand
    stage(0);
    if (r0 + kSplitTile < r1) fetch(r0 + kSplitTile);
    __syncthreads();
    int buf = 0;
    for (int64_t t0 = r0; t0 < r1; t0 += kSplitTile, buf ^= 1) {
        // the next tile's operands go to the other buffer while this one is used
        if (t0 + kSplitTile < r1) {
            stage(buf ^ 1);
            if (t0 + 2 * kSplitTile < r1) fetch(t0 + 2 * kSplitTile);
        }
        const int nb = (int)min((int64_t)NB, (r1 - t0 + 31) / 32);
#pragma unroll 2
        for (int blk = 0; blk < nb; ++blk) {
            v16f wr = {}, wi = {};
#pragma unroll
            for (int ch = 0; ch < NCH; ++ch) {
                const v8h a = aw[buf][blk][ch][lane];
                wr = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, bre[ch], wr, 0, 0, 0);
                if constexpr (KS != 2) wi = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, bim[ch], wi, 0, 0, 0);
            }
            const v4i a8 = *reinterpret_cast<const v4i*>(as[buf][blk][lane]);
            v4i m0, m1;
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                float x[4];
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    x[b] = KS == 3 ? fabsf(wi[4 * d + b]) + wr[4 * d + b] : wr[4 * d + b];
                m0[d] = (int)(signs_lo(x[0], x[1]) | signs_hi(x[2], x[3]));
                if constexpr (KS != 2) {
                    const uint32_t si = signs_lo(wi[4 * d], wi[4 * d + 1]) | signs_hi(wi[4 * d + 2], wi[4 * d + 3]);
                    m1[d] = (int)(KS == 3 ? si & ~(uint32_t)m0[d] : si);
                }
            }
            acc[0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a8, m0, acc[0], 0, 0, 0);
            if constexpr (KS != 2) acc[1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a8, m1, acc[1], 0, 0, 0);
            if constexpr (PROBE) {
                if (slot[0] >= 0) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int64_t at = t0 + 32 * blk + 8 * (i / 4) + 4 * h + i % 4;
                        const bool f0 = (m0[i / 4] >> (8 * (i % 4))) & 1, f1 = KS != 2 && ((m1[i / 4] >> (8 * (i % 4))) & 1);
                        int lab;
                        if constexpr (KS == 2) lab = f0 ? 1 : 0;
                        else if constexpr (KS == 3) lab = f0 ? 0 : (f1 ? 2 : 1);
                        else lab = f0 ? (f1 ? 3 : 2) : (f1 ? 0 : 1);
                        if (at < r1) p.probe_out[(size_t)slot[0] * p.n + at] = (uint16_t)lab;
                    }
                }
            }
        }
        __syncthreads();
    }

    // ---- sum_i V_i over the slice (exact), then s of each candidate
#pragma unroll
    for (int k = 0; k < C; ++k) {
        long long t = ts[k];
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1) t += __shfl_xor(t, off, kWave);
        if (fixed && lane == 0) tot[wave - kSplitTile / kWave][k] = t;
    }
    __syncthreads();
    const double unit = ldexp(1.0, ev - 29);
    float f = 0.0f;
#pragma unroll
    for (int g = 0; g < (REAL ? 4 : 2); ++g) {           // the columns this lane's registers hold
        const int j = REAL ? 2 * g + h : 2 * g + h;
        if (2 * g >= R) break;
        double zr[2], zi[2];                             // sums of Re z and Im z against Re V_j and Im V_j
#pragma unroll
        for (int q = 0; q < (REAL ? 1 : 2); ++q) {
            const int i0 = REAL ? 4 * g : 8 * g + 4 * q;
            long long t = 0, n0, n1 = 0;
            if (j < R) {
                for (int w = 0; w < kSplitTile / kWave; ++w) t += tot[w][q * R + j];
            }
            n0 = -((((long long)acc[0][i0 + 3] * 256 + acc[0][i0 + 2]) * 256 + acc[0][i0 + 1]) * 256 + acc[0][i0]);
            if constexpr (KS != 2)
                n1 = -((((long long)acc[NPL - 1][i0 + 3] * 256 + acc[NPL - 1][i0 + 2]) * 256 + acc[NPL - 1][i0 + 1]) * 256 +
                       acc[NPL - 1][i0]);
            if constexpr (KS == 2) {                     // n0: rows with z = -1
                zr[q] = unit * (double)(t - 2 * n0);
                zi[q] = 0.0;
            } else if constexpr (KS == 3) {              // n0, n1: rows with label 0, 2
                zr[q] = unit * 0.5 * (double)(3 * n0 - t);
                zi[q] = unit * 0.86602540378443865 * (double)(t - n0 - 2 * n1);
            } else {                                     // n0, n1: rows with negative real, imaginary part
                zr[q] = unit * 0.70710678118654752 * (double)(t - 2 * n0);
                zi[q] = unit * 0.70710678118654752 * (double)(t - 2 * n1);
            }
        }
        const float sr = REAL ? (float)zr[0] : (float)(zr[0] + zi[1]);
        const float si = REAL ? (float)zi[0] : (float)(zi[0] - zr[1]);
        if (j >= R) continue;
        f = fmaf(sr, sr, fmaf(si, si, f));
        if (gridDim.y > 1 && idx < p.S) {
            float* out = p.partial + ((size_t)blockIdx.y * (2 * R) + 2 * j) * p.S + idx;
            out[0] = sr;
            out[p.S] = si;
        }
    }
    f += __shfl_xor(f, 32, kWave);
    if (gridDim.y == 1 && h == 0 && idx < p.S) p.f_out[idx] = f;
}

}  // namespace
}  // namespace lrqo
