// Fused scorer on the matrix core from split FP32 values, K = 2, 3, 4, 8, 16
// and 2 <= r <= 4: both w = V c and s = V^H z are matrix products whose operands
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
//              V = V1 + V2 + V3, c likewise, which hold 33 bits of each, and
//              the k-slots take their products by size (SplitShape).  The
//              matrix core adds eight k-slots at a time, cutting each product
//              off at 2^-24 of the largest of the eight, and rounds to FP32
//              after every sixteen: so the products V1 c1 lie last and apart
//              from the others, and the smallest first.  (By falling size,
//              V1 c1 first, w was off by 0.82 u sum_j |V_ij c_j| for real r = 3,
//              u = 2^-24, root mean square, against 0.44 to 0.54 for a chain of
//              FP32 FMAs; in this order one chunk has 0.61, two have 0.41.)
//   labels     sign bits only.  K = 3: u = |Im w| - sqrt(3) Re w (label 0 iff
//              u < 0) and Im w; K = 2: Re w; K = 4, 8, 16: the direction is
//              turned by e^{-i pi/K}, so the boundaries are the axes and
//              lines |b| = tan(phi) |a| of w = a + ib.  v_perm_b32 spreads the
//              signs of four rows over the bytes of a dword as 0 / -1.
//   z          label planes of one byte per row: masks of label sets
//              (K = 2, 3, 4), sign(a), sign(b) within each half of a quadrant
//              (K = 8), or for K = 16, whose roots have four magnitudes, Re z
//              and Im z in 23-bit fixed point, three balanced base-256 digits
//              each, looked up by v_perm_b32 (eight-byte tables: sector and
//              sign select the byte)
//   s = V^H z  v_mfma_i32_32x32x32_i8 of those planes against V in fixed point
//              of 45 bits (balanced base-256 digits: four in units of
//              2^(E_j - 29) for column j and two of 2^-15 of that, in operand
//              rows that would be idle; 8 rows a component) or, for more than
//              four components, 30 (4C <= 32 rows).  E_j is at most 19 or 4
//              above the exponent e of the column's largest entry in the
//              256-row tile, so an entry is off by at most 2^(e - 26), a
//              fraction of what one addition to a running FP32 sum of that size
//              rounds away, and a few large rows cost only the rows that share
//              their tile.  The sums are exact integers; their digits are put
//              together, in FP64, where an E_j changes and at the end.  (10^6
//              rows, r = 3 real, K = 3, 2^19 candidates: 69.0 ms for normal
//              rows, 70.6 for row sizes u^-3, u uniform; with 30 bits 67.6 and
//              74.2, as 88% of the tiles of such a factor change an E_j.  One
//              scale for the whole factor took 2.4 ms less, but 300,000 rows
//              of 1e-9 beside one of 3.9 left f off by 1.8e-4, now 1e-5, FP32
//              sums 1.2e-5.)
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
static_assert(kSplitTile * 2 == kSplitBlock, "a thread stages one operand of one row");

// Rows after which the I32 sums are folded: digits of V are at most 128 in size
// and plane entries 1, or 128 for K = 16, so that the sums stay at 2^30, and for
// the others a sum plus 256 times the next one as well.
__host__ __device__ constexpr int64_t split_rows(int KS) { return (int64_t)1 << (KS == 16 ? 16 : 15); }
constexpr int64_t kSplitMaxRows = (int64_t)1 << 23;

// K = 16 planes.  Entry e of a table: bits 0 and 1 name the sector of the
// quadrant, bit 2 is the sign; entries hold digit k of round(mag * kRoot16).
// The factor keeps the top digit below 128 and all four roundings below 2^-30,
// where FP32 roots have up to 2^-25.
constexpr double kRoot16 = 8312657.375;
constexpr double root16_mag(int e) {
    return (e & 3) == 3 ? 0.98078528040323043 : (e & 3) == 1 ? 0.83146961230254524 : (e & 3) == 0 ? 0.55557023301960218 : 0.19509032201612826;
}
constexpr uint32_t root16_digit(int e, int k) {
    const long long x = (long long)(root16_mag(e) * kRoot16 + 0.5) * (e & 4 ? -1 : 1);
    return (uint32_t)(((((unsigned long long)(x + 0x808080)) >> (8 * k)) & 255u) ^ 0x80u);
}
constexpr uint32_t root16_table(int half, int k) {
    return root16_digit(4 * half, k) | root16_digit(4 * half + 1, k) << 8 | root16_digit(4 * half + 2, k) << 16 |
           root16_digit(4 * half + 3, k) << 24;
}

constexpr bool root16_close() {
    for (int e = 0; e < 4; ++e) {
        const double x = root16_mag(e) * kRoot16, d = x - (double)(long long)(x + 0.5);
        if ((d < 0.0 ? -d : d) > kRoot16 / 1073741824.0) return false;
    }
    return true;
}
static_assert(root16_close(), "roundings of the K = 16 magnitudes");

// Products of the parts (0, 1, 2) of V and of c, by falling size.
constexpr int kSplitV[8] = {0, 1, 0, 1, 2, 0, 2, 1};
constexpr int kSplitC[8] = {0, 0, 1, 1, 0, 2, 1, 2};

// Shape of w's operands: chunks of 16 k-slots, as many as keep the labels at or
// below the error of FP32 ones.  Wrong labels per 10^9, normal V, this scorer /
// the FP32 scorer (20 10^9 labels each, 60 10^9 for real r = 3, K = 3 and
// complex r = 3, K = 2; one standard deviation is 7% at 10 per 10^9):
//                K = 2       3           4         8         16
//     real    2              6.2/9.4     1.0/17              42/67
//             3              11.0/10.3   12/19     31/36     63/75
//             4              6.9/12.3                        44/84
//     complex 2              6.1/10.9                        41/77
//             3  1.8/5.7     13.8/14.7   16/23     41/45     83/97
//             4              7.2/15.3                        52/103
// Real r = 3 fits one chunk, but for two products V1 c3: K = 4 and the precision
// form (QUICK; its former BF16 parts left several u) leave it at that, else Re w
// has a chunk more, for what comes last in size (K = 3 13.3 without it; 10^6
// rows, 2^19 candidates: 59.5 -> 69.0 ms, FP32 scorer 122).  Complex r = 3 leaves
// out part of V3 c1 and V1 c3, but for K = 2, which has Re w alone.
template <int R, bool REAL, int KS, bool QUICK>
struct SplitShape {
    static constexpr int C = REAL ? R : 2 * R;
    static constexpr bool EXTRA = C == 3 && KS != 4 && !QUICK;
    static constexpr int NCH = C <= 3 ? (EXTRA ? 2 : 1) : (C == 8 || (C == 6 && KS == 2) ? 3 : 2);   // chunks of V and of Re w
    static constexpr int NIM = EXTRA ? 1 : NCH;                               // the last ones, of Im w
    // k-slot s holds product tau[s] (kSplitV, kSplitC; -1: none) of component
    // comp[s], for Re w where re[s].  The eight last k-slots: V1 c1, then what
    // finds no place elsewhere (V3 has few bits, which survive beside V1 c1; for
    // C = 2 it goes there first).
    struct Slots {
        int tau[16 * NCH], comp[16 * NCH];
        bool re[16 * NCH];
        constexpr Slots() : tau{}, comp{}, re{} {
            constexpr int order[2][7] = {{1, 2, 3, 4, 5, 6, 7}, {1, 2, 3, 5, 4, 6, 7}};
            constexpr int first = EXTRA ? 16 : 0, end = 16 * NCH, last = end - 8;
            for (int s = 0; s < end; ++s) {
                tau[s] = -1;
                re[s] = true;
            }
            for (int x = 0; x < C; ++x) {
                tau[last + x] = 0;
                comp[last + x] = x;
            }
            int s = last - 1, extra = 0;
            for (int t = 0; t < 7; ++t)
                for (int x = 0; x < C; ++x) {
                    if (s == first - 1) s = last + C;    // downwards, then the rest of the last eight
                    const int tt = order[C == 2][t];
                    const bool fits = s < end;
                    if (fits) {
                        tau[s] = tt;
                        comp[s] = x;
                    }
                    if (EXTRA && (!fits || (s >= last && tt != 4)) && extra < 16) {
                        if (fits) re[s] = false;
                        tau[extra] = tt;
                        comp[extra++] = x;
                    }
                    if (fits) s += s < last ? -1 : 1;
                }
        }
    };
    static constexpr Slots slots{};
};
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

// Signs of two values as bytes 0 / -1 in the low or high half of a dword.
__device__ __forceinline__ uint32_t signs_lo(float a, float b) {
    return __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x0c0c0b09u);
}
__device__ __forceinline__ uint32_t signs_hi(float a, float b) {
    return __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x0b090c0cu);
}

__device__ __forceinline__ uint32_t signs4(float a, float b, float c, float d) {
    return signs_lo(a, b) | signs_hi(c, d);
}

// A column's exponent E (tile_exp holds those of its largest entries, tile by
// tile, from the prologue) is kept while the largest entry of the tile is in
// [2^(E - split_slack), 2^(E + 1)); else it becomes one above that entry's
// exponent (so that the next larger tile need not change it), at most that of
// the factor's largest entry.  V enters the I8 operand as round(V 2^(29-E)), at
// most 2^30 in size, and with low digits the rest of it, rounded to 2^-15.
__host__ __device__ constexpr bool split_low(int C) { return C <= 4; }   // two low digits too
__host__ __device__ constexpr int split_slack(int C) { return split_low(C) ? 19 : 4; }

// Whether a direction of a caller's list lies within the range of the F16 parts,
// which reach down to 2^-39 of a row's and of a direction's largest entry.  What
// they cannot hold is no more than 2^-27 of sum_j |V_ij||c_j| while no component
// is below 2^-12 of the largest (a row may lie on that column alone).  K = 2, 3,
// 4: the same for Re w and Im w as a whole, and no part that decides a sign alone
// may be lost or a tie (2^-24: real or imaginary c_j; K = 4: their sum and
// difference).  Of 2^20
// directions of the sphere the smallest component is near 2^-11 of the largest,
// and below 2^-16, where a row on that column alone would lose more than in
// FP32, once in a thousand calls; so only lists, which may hold axes, are looked
// at.  false for NaN, infinities and zero.
template <int R>
__device__ __forceinline__ bool direction_in_range(const float (&c)[2 * R], int K) {
    float lo = INFINITY, hi = 0.0f, small = INFINITY, re = 0.0f, im = 0.0f;
    bool finite = true;
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const float a = fabsf(c[2 * j]), b = fabsf(c[2 * j + 1]);
        finite &= isfinite(a) && isfinite(b);
        lo = fminf(lo, fmaxf(a, b));
        hi = fmaxf(hi, fmaxf(a, b));
        const float x = K == 4 ? 0.5f * a + 0.5f * b : a, y = K == 4 ? fabsf(0.5f * a - 0.5f * b) : b;
        re = fmaxf(re, x);
        im = fmaxf(im, y);
        small = fminf(small, K == 2 ? x : fminf(x, y));
    }
    const float least = hi * 0x1p-12f;
    if (!finite || !(lo > 0.0f) || !(lo >= least)) return false;
    return K > 4 || (small > 0.0f && small >= hi * 0x1p-24f && re >= least && (K == 2 || im >= least));
}

// Exponent of the largest |V| entry (prologue's per-block maxima).
__device__ __forceinline__ int split_exponent(const float* vmax, int count) {
    float m = 0.0f;
    for (int k = (int)(threadIdx.x & (kWave - 1)); k < count; k += kWave) m = fmaxf(m, vmax[k]);
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, kWave));
    return m > 0.0f && isfinite(m) ? ilogbf(m) : 0;
}

// 2^(E - 29)
__device__ __forceinline__ double split_unit(int E) { return __hiloint2double((E - 29 + 1023) << 20, 0); }

// Label planes of a K.
__host__ __device__ constexpr int split_planes(int KS) { return KS == 2 ? 1 : (KS == 8 ? 4 : (KS == 16 ? 6 : 2)); }
// Waves per SIMD asked of the compiler: K = 8 and 16 hold 64 and 96
// accumulators (K = 8 at four waves spills: r = 3 complex 3.7 against 3.1 ms
// for n = 100,000 and 131,072 candidates).
__host__ __device__ constexpr int split_waves(int KS) { return KS >= 8 ? 2 : 4; }

template <int R, bool REAL, int KS, bool PROBE, bool QUICK>
__global__ __launch_bounds__(kSplitBlock, split_waves(KS)) void k_score_split(ScoreParams p) {
    using Sh = SplitShape<R, REAL, KS, QUICK>;
    constexpr int C = Sh::C, NCH = Sh::NCH, IM0 = NCH - Sh::NIM;
    constexpr typename Sh::Slots slots = Sh::slots;
    constexpr int NB = kSplitTile / 32;                  // 32-row blocks of a tile
    constexpr int NPL = split_planes(KS);
    __shared__ __align__(16) v8h aw[2][NB][NCH][64];     // F16 operand of w: [buffer][block][chunk][lane]
    __shared__ __align__(16) signed char as[2][NB][64][16];   // I8 operand of s: [buffer][block][lane][k-slot]
    // a lane's s so far: in LDS, as 128 registers hold no more than the loop needs (8 components: 80 KB
    // in all, half of a CU's)
    constexpr int NG = (R + 1) / 2;
    __shared__ double sums[2 * NG][kSplitBlock];
    if (p.list_flags && list_is_wide(p)) return;         // left to the FP32 scorer
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int h = lane >> 5;
    const int ev = split_exponent(p.vmax, p.vmax_count);
    // rows of the I8 operand that no component uses stay zero
    for (int e = tid; e < (int)(sizeof(as) / 16); e += kSplitBlock)
        reinterpret_cast<v4i*>(as)[e] = v4i{0, 0, 0, 0};

    // ---- this lane's candidate (lanes l and l + 32 share one): B operands
    const uint32_t idx = blockIdx.x * (uint32_t)kSplitCands + wave * 32 + (lane & 31);
    v8h bre[NCH], bim[Sh::NIM];
    int slot[1];
    {
        float c[1][2 * R];
        lane_directions<R, 1, PROBE>(p, idx, 0, blockIdx.y == 0 && h == 0, c, slot);
        // scaled like a row (a caller's list need not hold unit directions)
        float m = 0.0f;
#pragma unroll
        for (int j = 0; j < 2 * R; ++j) m = fmaxf(m, fabsf(c[0][j]));
        const int e = m > 0.0f ? 14 - ilogbf(m) : 0;     // times sqrt(3), or turned: below the largest F16
        double x[C], y[C];                               // factors of the components in Re w, Im w
#pragma unroll
        for (int j = 0; j < R; ++j) {
            double cr = ldexp((double)c[0][2 * j], e), ci = ldexp((double)c[0][2 * j + 1], e);
            if constexpr (KS == 4 || KS == 8 || KS == 16) {   // c e^{-i pi/K}
                constexpr double co = KS == 4 ? 0.70710678118654752 : (KS == 8 ? 0.92387953251128676 : 0.98078528040323043);
                constexpr double sn = KS == 4 ? 0.70710678118654752 : (KS == 8 ? 0.38268343236508977 : 0.19509032201612826);
                const double t = cr * co + ci * sn;
                ci = ci * co - cr * sn;
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
                    const int ks = 16 * ch + 8 * g + t, tau = slots.tau[ks], k = slots.comp[ks];
                    r[g] = tau >= 0 && slots.re[ks] ? px[k][kSplitC[tau < 0 ? 0 : tau]] : (_Float16)0.0f;
                    i[g] = tau >= 0 ? py[k][kSplitC[tau < 0 ? 0 : tau]] : (_Float16)0.0f;
                }
                bre[ch][t] = h ? r[1] : r[0];
                if (ch >= IM0) bim[ch < IM0 ? 0 : ch - IM0][t] = h ? i[1] : i[0];
            }
    }

    v16i acc[NPL];
#pragma unroll
    for (int q = 0; q < NPL; ++q)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[q][i] = 0;

    // ---- s of the lane's columns j = 2g + h from the accumulators, which hold
    // units of 2^(E_j - 29).  K <= 4: without the terms in sum_i V_ij
    int E[R];
    // K <= 4: sums of V over the slice.  Wave w adds up the digits of block w of
    // every tile: lane l those of operand row l % 32 (digit p of a column's Re
    // or Im) over its sixteen rows of V.
    const int uwave = __builtin_amdgcn_readfirstlane(wave);
    constexpr bool LOW = split_low(C);
    const int dslot = (lane & 31) >> 2, dcol = LOW ? dslot & (REAL ? 3 : 1) : (dslot & 1) + 2 * (dslot >> 2);
    int digits = 0;
    double dsum = 0.0;
#pragma unroll
    for (int g = 0; g < 2 * NG; ++g) sums[g][tid] = 0.0;
    auto fold = [&]() {
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const double unit = split_unit(h && 2 * g + 1 < R ? E[2 * g + 1 < R ? 2 * g + 1 : 0] : E[2 * g]);
            double zr[2] = {0.0, 0.0}, zi[2] = {0.0, 0.0};   // sums of Re z, Im z times Re V_j and times Im V_j
#pragma unroll
            for (int q = 0; q < (REAL ? 1 : 2); ++q) {
                const int i0 = REAL ? 4 * g : 8 * g + 4 * q;
                auto pair = [&](int k, int i) {
                    return KS == 16 ? fma(256.0, (double)acc[k][i + 1], (double)acc[k][i])
                                    : (double)(acc[k][i + 1] * 256 + acc[k][i]);
                };
                auto plane = [&](int k) {
                    const double v = fma(65536.0, pair(k, i0 + 2), pair(k, i0));
                    return unit * (LOW ? fma(0x1p-15, pair(k, i0 + (LOW ? 8 : 0)), v) : v);
                };
                if constexpr (KS <= 4) {
                    const double n0 = -plane(0), n1 = -plane(NPL - 1);   // masks are 0 / -1
                    if constexpr (KS == 2) {             // n0: rows with z = -1
                        zr[q] = -2.0 * n0;
                    } else if constexpr (KS == 3) {      // n0, n1: rows with label 0, 2
                        zr[q] = 1.5 * n0;
                        zi[q] = -0.86602540378443865 * (n0 + 2.0 * n1);
                    } else {                             // n0, n1: rows with negative real, imaginary part
                        zr[q] = -1.4142135623730950 * n0;
                        zi[q] = -1.4142135623730950 * n1;
                    }
                } else if constexpr (KS == 8) {
                    zr[q] = 0.92387953251128676 * plane(0) + 0.38268343236508977 * plane(1);
                    zi[q] = 0.38268343236508977 * plane(2) + 0.92387953251128676 * plane(3);
                } else {
                    zr[q] = ((plane(2) * 256.0 + plane(1)) * 256.0 + plane(0)) * (1.0 / kRoot16);
                    zi[q] = ((plane(5) * 256.0 + plane(4)) * 256.0 + plane(3)) * (1.0 / kRoot16);
                }
            }
            sums[2 * g][tid] += REAL ? zr[0] : zr[0] + zi[1];
            sums[2 * g + 1][tid] += REAL ? zi[0] : zi[0] - zr[1];
        }
#pragma unroll
        for (int q = 0; q < NPL; ++q)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[q][i] = 0;
        if constexpr (KS <= 4) {
            double unit = 0.0;                           // of this lane's column
#pragma unroll
            for (int j = 0; j < R; ++j) unit += dcol == j ? split_unit(E[j]) : 0.0;
            if (LOW && dslot > 3) unit *= 0x1p-15;
            dsum += unit * (double)((long long)digits << (8 * (lane & 3)));
            digits = 0;
        }
    };

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
    // Exponents for a tile; true if one of them changes.
    auto exponents = [&](int2 te, const int (&from)[R], int (&to)[R]) {
        const int w[2] = {__builtin_amdgcn_readfirstlane(te.x), __builtin_amdgcn_readfirstlane(te.y)};
        bool change = false;
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int e = (w[j / 2] << (16 - 16 * (j & 1))) >> 16;
            to[j] = e == kZeroColumn || (e <= from[j] && e >= from[j] - split_slack(C)) ? from[j] : min(e + 1, ev);
            change |= to[j] != from[j];
        }
        return change;
    };
    auto stage = [&](int buf, const int (&Et)[R]) {
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
                        const int ks = 16 * ch + 8 * g + t, tau = slots.tau[ks];
                        a[t] = tau >= 0 ? pv[slots.comp[ks]][kSplitV[tau < 0 ? 0 : tau]] : (_Float16)0.0f;
                    }
                    aw[buf][blk][ch][32 * g + rr] = a;
                }
        } else {
            const int d = rr >> 3, g = (rr >> 2) & 1, b = rr & 3;
#pragma unroll
            for (int k = 0; k < C; ++k) {
                const float x = ldexpf(v[k], 29 - Et[k % R]);
                const int q = __float2int_rn(x);
                const uint32_t dig = ((uint32_t)q + 0x00808080u) ^ 0x00808080u;   // balanced digits, lowest first
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    as[buf][blk][32 * g + 4 * split_slot<R, REAL>(k) + t][4 * d + b] = (signed char)(dig >> (8 * t));
                if constexpr (LOW) {                     // the rest, in units of 2^-15
                    const int ql = __float2int_rn((x - (float)q) * 32768.0f);
                    const uint32_t low = ((uint32_t)ql + 0x80u) ^ 0x80u;
#pragma unroll
                    for (int t = 0; t < 2; ++t)
                        as[buf][blk][32 * g + 4 * split_slot<R, REAL>(k) + 16 + t][4 * d + b] = (signed char)(low >> (8 * t));
                }
            }
        }
    };

    const int2* __restrict__ te = reinterpret_cast<const int2*>(p.tile_exp) + r0 / kSplitTile;   // a slice begins with a tile
    int2 tn = te[0];
    fetch(r0);
    __syncthreads();                                     // the zeroed operand
#pragma unroll
    for (int j = 0; j < R; ++j) E[j] = ev;
    exponents(tn, E, E);
    stage(0, E);
    if (r0 + kSplitTile < r1) {
        fetch(r0 + kSplitTile);
        tn = *++te;
    }
    __syncthreads();
    int buf = 0;
    for (int64_t t0 = r0; t0 < r1; t0 += kSplitTile, buf ^= 1) {
        // the next tile's operands go to the other buffer while this one is used
        int En[R];
#pragma unroll
        for (int j = 0; j < R; ++j) En[j] = E[j];
        bool change = false;
        if (t0 + kSplitTile < r1) {
            change = exponents(tn, E, En);
            stage(buf ^ 1, En);
            if (t0 + 2 * kSplitTile < r1) {
                fetch(t0 + 2 * kSplitTile);
                tn = *++te;
            }
        }
        const int nb = (int)min((int64_t)NB, (r1 - t0 + 31) / 32);
#pragma unroll 2
        for (int blk = 0; blk < nb; ++blk) {
            v16f wr = {}, wi = {};
#pragma unroll
            for (int ch = 0; ch < NCH; ++ch) {
                const v8h a = aw[buf][blk][ch][lane];
                wr = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, bre[ch], wr, 0, 0, 0);
                if constexpr (KS != 2)
                    if (ch >= IM0) wi = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, bim[ch < IM0 ? 0 : ch - IM0], wi, 0, 0, 0);
            }
            const v4i a8 = *reinterpret_cast<const v4i*>(as[buf][blk][lane]);
            v4i m[NPL];
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                float a[4], c[4];
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    a[b] = wr[4 * d + b];
                    c[b] = wi[4 * d + b];
                }
                if constexpr (KS == 3) {
#pragma unroll
                    for (int b = 0; b < 4; ++b) a[b] += fabsf(c[b]);
                }
                const uint32_t sa = signs4(a[0], a[1], a[2], a[3]);
                m[0][d] = (int)sa;
                if constexpr (KS != 2) {
                    const uint32_t sb = signs4(c[0], c[1], c[2], c[3]);
                    if constexpr (KS == 3) m[1][d] = (int)(sb & ~sa);
                    else m[1][d] = (int)sb;
                    if constexpr (KS == 8) {             // halves of the quadrant: |a| >= |b| or not
                        float t[4];
#pragma unroll
                        for (int b = 0; b < 4; ++b) t[b] = fabsf(a[b]) - fabsf(c[b]);
                        const uint32_t st = signs4(t[0], t[1], t[2], t[3]);
                        m[0][d] = (int)((sa | 0x01010101u) & ~st);
                        m[1][d] = (int)((sa | 0x01010101u) & st);
                        m[2][d] = (int)((sb | 0x01010101u) & ~st);
                        m[3][d] = (int)((sb | 0x01010101u) & st);
                    }
                    if constexpr (KS == 16) {            // |b| against tan(pi/8), 1, tan(3 pi/8) times |a|
                        float t[3][4];
#pragma unroll
                        for (int b = 0; b < 4; ++b) {
                            t[0][b] = fmaf(-0.41421356237309505f, fabsf(a[b]), fabsf(c[b]));
                            t[1][b] = fabsf(c[b]) - fabsf(a[b]);
                            t[2][b] = fmaf(-2.41421356237309505f, fabsf(a[b]), fabsf(c[b]));
                        }
                        const uint32_t s0 = signs4(t[0][0], t[0][1], t[0][2], t[0][3]);
                        const uint32_t s1 = signs4(t[1][0], t[1][1], t[1][2], t[1][3]);
                        const uint32_t s2 = signs4(t[2][0], t[2][1], t[2][2], t[2][3]);
                        // sector code: bit 0 below the diagonal, bit 1 next to an axis; Im z has
                        // the magnitudes of Re z mirrored on the diagonal
                        const uint32_t axis = (s0 | ~s2) & 0x02020202u;
                        const uint32_t er = (axis | (s1 & 0x01010101u)) | (sa & 0x04040404u);
                        const uint32_t ei = (axis | (~s1 & 0x01010101u)) | (sb & 0x04040404u);
#pragma unroll
                        for (int k = 0; k < 3; ++k) {
                            m[k][d] = (int)__builtin_amdgcn_perm(root16_table(1, k), root16_table(0, k), er);
                            m[3 + k][d] = (int)__builtin_amdgcn_perm(root16_table(1, k), root16_table(0, k), ei);
                        }
                    }
                }
            }
#pragma unroll
            for (int q = 0; q < NPL; ++q) acc[q] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a8, m[q], acc[q], 0, 0, 0);
            if constexpr (PROBE) {
                if (slot[0] >= 0) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int64_t at = t0 + 32 * blk + 8 * (i / 4) + 4 * h + i % 4;
                        int lab;
                        if constexpr (KS <= 4) {
                            const bool f0 = (m[0][i / 4] >> (8 * (i % 4))) & 1, f1 = (m[NPL - 1][i / 4] >> (8 * (i % 4))) & 1;
                            if constexpr (KS == 2) lab = f0 ? 1 : 0;
                            else if constexpr (KS == 3) lab = f0 ? 0 : (f1 ? 2 : 1);
                            else lab = f0 ? (f1 ? 3 : 2) : (f1 ? 0 : 1);
                        } else {                         // the root the planes hold, turned back
                            auto at_byte = [&](int q) { return (float)(signed char)(m[q][i / 4] >> (8 * (i % 4))); };
                            float zr, zi;
                            if constexpr (KS == 8) {
                                zr = kCos8 * at_byte(0) + kSin8 * at_byte(1);
                                zi = kSin8 * at_byte(2) + kCos8 * at_byte(3);
                            } else {
                                zr = (at_byte(2) * 256.0f + at_byte(1)) * 256.0f + at_byte(0);
                                zi = (at_byte(5) * 256.0f + at_byte(4)) * 256.0f + at_byte(3);
                            }
                            constexpr float co = KS == 8 ? kCos8 : kCos16, sn = KS == 8 ? kSin8 : kSin16;
                            lab = root_index(zr * co - zi * sn, zr * sn + zi * co, KS);
                        }
                        if (at < r1) p.probe_out[(size_t)slot[0] * p.n + at] = (uint16_t)lab;
                    }
                }
            }
        }
        if constexpr (KS <= 4) {
            if (uwave < nb) {
                const v4i a8 = *reinterpret_cast<const v4i*>(as[buf][uwave][lane]);
#pragma unroll
                for (int d = 0; d < 4; ++d) digits = __builtin_amdgcn_sdot4(a8[d], 0x01010101, digits, false);
            }
        }
        const bool full = (t0 - r0) % split_rows(KS) == split_rows(KS) - kSplitTile;
        if (change || full) {
            fold();
#pragma unroll
            for (int j = 0; j < R; ++j) E[j] = En[j];
        }
        __syncthreads();
    }

    fold();
    double sum[NG][2];
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int u = 0; u < 2; ++u) sum[g][u] = sums[2 * g + u][tid];
    // ---- K <= 4: the terms in sum_i V_i over the slice; then s of each candidate
    if constexpr (KS <= 4) {
        double* tot = reinterpret_cast<double*>(aw);     // no longer in use: the loop ends with a barrier
        tot[tid] = dsum;
        __syncthreads();
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            double t[2] = {0.0, 0.0};                    // sums of Re V_j, Im V_j, j = 2g + h
#pragma unroll
            for (int q = 0; q < (REAL ? 1 : 2); ++q) {
                const int at = 4 * (REAL ? 2 * g + h : 4 * g + 2 * q + h);   // its first digit
#pragma unroll 1
                for (int w = 0; w < kSplitBlock / kWave; ++w)
#pragma unroll
                    for (int d = 0; d < 4; ++d) {
                        t[q] += tot[w * kWave + at + d] + tot[w * kWave + 32 + at + d];
                        if constexpr (LOW) t[q] += tot[w * kWave + 16 + at + d] + tot[w * kWave + 48 + at + d];
                    }
            }
            // z = a + ib in every row, corrected by the masks
            constexpr double a = KS == 2 ? 1.0 : (KS == 3 ? -0.5 : 0.70710678118654752);
            constexpr double b = KS == 2 ? 0.0 : (KS == 3 ? 0.86602540378443865 : 0.70710678118654752);
            sum[g][0] += a * t[0] + b * t[1];
            sum[g][1] += b * t[0] - a * t[1];
        }
    }
    float f = 0.0f;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        const int j = 2 * g + h;
        if (j >= R) continue;
        const float sr = (float)sum[g][0], si = (float)sum[g][1];
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
