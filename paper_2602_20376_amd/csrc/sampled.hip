// Sampled maximisation (Sec. 4.2): fused FP32 scorer over uniform sphere
// directions, top-T selection, FP64 rescore of the T best, label write-out.
//
// Kernels, in launch order:
//   k_prologue      roots of unity and the zeroed result record (block 0);
//                   per block, whether its share of V holds a NaN or an
//                   infinity (k_pick gathers the blocks' flags)
//   k_score*        fused candidate generation + scoring (sampled_kernels.h):
//                   each lane owns CPL directions in registers; row tiles of V
//                   stream through LDS; per row-candidate w = V_i c, the
//                   nearest K-th root of arg(w), s += conj(V_i) z_i.  With
//                   several row slices (gridDim.y > 1) partial sums instead.
//                   The precision form's scorers are in sampled_bf16.h, the
//                   matrix-core scorer of larger problems in sampled_split.h.
//   k_finalize      sums the slice partials in a fixed order -> f = ||s||^2,
//                   and sorts each wave's 64 keys for the selection
//   topk_select     best T packed (f, index) keys (select.hip)
//   k_rescore       FP64 re-evaluation of each kept direction, row-sliced
//   k_pick          FP64 arg-max of the rescored candidates (ties -> lowest index)
//   k_labels        FP64 decision rule of the winner -> uint8 labels
//   k_tail          small problems: the selection to the labels in one block,
//                   and where the scorer needs neither, the prologue's checks
#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>

#include "lrqo_device.h"
#include "lrqo_runtime.h"
#include "sampled_internal.h"
#include "sampled_kernels.h"
#include "sampled_bf16.h"
#include "sampled_split.h"
#include "select.h"

#ifndef LRQO_SCORE_BLOCKS
#define LRQO_SCORE_BLOCKS 2048
#endif

namespace lrqo {

namespace {

// ------------------------------------------------------------ set-up and checks
// Block 0: roots of unity omega^k = (cos, sin)(2 pi k / K) in FP64 and their
// FP32 roundings, and the zeroed result record.  Every block: whether its
// share of V holds a NaN or an infinity, into bad[blockIdx.x] (so that no
// block writes the record while block 0 clears it; k_pick gathers them), and
// the largest finite |V| entry of the share, into vmax[blockIdx.x] (the real
// K = 3 scorer sizes its quantiser scale from it).  TILES: also the exponents
// of the columns' largest entries over each tile of the matrix-core scorer, and
// whether a caller's list of directions is outside its range.
template <int R, bool REAL, bool TILES>
__global__ __launch_bounds__(kBlock) void k_prologue(int K, double2* __restrict__ roots64,
                                                     float2* __restrict__ roots32, DevResult* __restrict__ res,
                                                     const float* __restrict__ V, int64_t n,
                                                     int* __restrict__ bad, float* __restrict__ vmax,
                                                     TileExp* __restrict__ tile_exp,
                                                     const float* __restrict__ dirs, uint32_t S) {
    constexpr int RF = Row<R, REAL>::F;
    __shared__ float wmax[kBlock / kWave];
    if (blockIdx.x == 0) {
        for (int k = threadIdx.x; k < K; k += blockDim.x) {
            double sn, cs;
            sincospi(2.0 * (double)k / (double)K, &sn, &cs);
            roots64[k] = make_double2(cs, sn);
            roots32[k] = make_float2((float)cs, (float)sn);
        }
        if (threadIdx.x == 0) *res = DevResult{};
    }
    bool b = false;
    float m = 0.0f;
    bool wide = false;
    if constexpr (TILES) {
        for (int64_t q = blockIdx.x * kBlock + threadIdx.x; dirs && q < (int64_t)S; q += (int64_t)gridDim.x * kBlock) {
            float c[2 * R];
#pragma unroll
            for (int j = 0; j < 2 * R; ++j) c[j] = dirs[q * (2 * R) + j];
            wide |= !direction_in_range<R>(c, K);
        }
        // a wave takes whole tiles: four rows a lane, and the columns' maxima over the wave
        const int lane = threadIdx.x & (kWave - 1);
        const int64_t tiles = (n + kSplitTile - 1) / kSplitTile;
        for (int64_t t = blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave; t < tiles;
             t += (int64_t)gridDim.x * (kBlock / kWave)) {
            float x[kSplitTile / kWave][RF], c[R];
#pragma unroll
            for (int u = 0; u < kSplitTile / kWave; ++u) {
                const int64_t i = t * kSplitTile + u * kWave + lane;
#pragma unroll
                for (int e = 0; e < RF; ++e) x[u][e] = i < n ? V[i * RF + e] : 0.0f;
            }
#pragma unroll
            for (int j = 0; j < R; ++j) {
                c[j] = 0.0f;
#pragma unroll
                for (int u = 0; u < kSplitTile / kWave; ++u)
#pragma unroll
                    for (int e = j * (RF / R); e < (j + 1) * (RF / R); ++e) {
                        const bool fin = isfinite(x[u][e]);
                        b |= !fin;
                        c[j] = fin ? fmaxf(c[j], fabsf(x[u][e])) : c[j];
                    }
#pragma unroll
                for (int off = kWave / 2; off > 0; off >>= 1) c[j] = fmaxf(c[j], __shfl_xor(c[j], off, kWave));
                m = fmaxf(m, c[j]);
            }
            if (lane == 0) {
                TileExp te{};
#pragma unroll
                for (int j = 0; j < R; ++j) te.e[j] = (int16_t)(c[j] > 0.0f ? ilogbf(c[j]) : kZeroColumn);
                tile_exp[t] = te;
            }
        }
    } else {
        for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n * RF;
             e += (int64_t)gridDim.x * blockDim.x) {
            const float x = V[e];
            const bool fin = isfinite(x);
            b |= !fin;
            m = fin ? fmaxf(m, fabsf(x)) : m;
        }
    }
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, kWave));
    if ((threadIdx.x & (kWave - 1)) == 0) wmax[threadIdx.x / kWave] = m;
    const int any = __syncthreads_or(b), any_wide = __syncthreads_or(wide);
    if (threadIdx.x == 0) {
        bad[blockIdx.x] = (any ? kFlagNonfinite : 0) | (any_wide ? kFlagWide : 0);
        float mm = 0.0f;
        for (int w = 0; w < kBlock / kWave; ++w) mm = fmaxf(mm, wmax[w]);
        vmax[blockIdx.x] = mm;
    }
}

// Slice sums: f of each candidate from the scorer's per-slice partial sums
// (slices in order, then the components in order).  Each wave also sorts its
// 64 keys across its lanes, so the first top-T pass merges sorted lists.
template <int R>
__global__ __launch_bounds__(kBlock) void k_finalize(const float* __restrict__ partial, int P,
                                                     uint32_t S, float* __restrict__ f_out,
                                                     unsigned long long* __restrict__ lists) {
    constexpr int U = R <= 4 ? 8 : 4;      // slices loaded together
    const uint32_t idx = blockIdx.x * kBlock + threadIdx.x;
    const int lane = threadIdx.x & (kWave - 1);
    unsigned long long key = 0;
    if (idx < S) {
        float acc[2 * R];
#pragma unroll
        for (int j = 0; j < 2 * R; ++j) acc[j] = 0.0f;
        int p0 = 0;
        for (; p0 + U <= P; p0 += U) {          // whole groups: every load issued before the adds
            float v[U][2 * R];
#pragma unroll
            for (int q = 0; q < U; ++q)
#pragma unroll
                for (int j = 0; j < 2 * R; ++j) v[q][j] = partial[((size_t)(p0 + q) * (2 * R) + j) * S + idx];
#pragma unroll
            for (int q = 0; q < U; ++q)
#pragma unroll
                for (int j = 0; j < 2 * R; ++j) acc[j] += v[q][j];
        }
        for (; p0 < P; ++p0)
#pragma unroll
            for (int j = 0; j < 2 * R; ++j) acc[j] += partial[((size_t)p0 * (2 * R) + j) * S + idx];
        float f = 0.0f;
#pragma unroll
        for (int j = 0; j < 2 * R; ++j) f = fmaf(acc[j], acc[j], f);
        f_out[idx] = f;
        key = pack_key(f, idx);
    }
    lists[idx] = wave_sort_desc(key, lane);
}

// ------------------------------------------------------------ FP64 rescore
// One row's FP64 terms of conj(V_i) z_i, added to acc (a real V leaves out
// the products with Im V: half the FP64 work).
template <int R, bool REAL, int KS>
__device__ __forceinline__ void rescore_row(const float (&row)[Row<R, REAL>::F], const double (&c)[2 * R], int K,
                                            const double2* roots, double (&acc)[2 * R]) {
    double wr = 0.0, wi = 0.0;
#pragma unroll
    for (int j = 0; j < R; ++j) {
        if constexpr (REAL) {
            const double vr = (double)row[j];
            wr += vr * c[2 * j];
            wi += vr * c[2 * j + 1];
        } else {
            const double vr = (double)row[2 * j], vi = (double)row[2 * j + 1];
            wr += vr * c[2 * j] - vi * c[2 * j + 1];
            wi += vr * c[2 * j + 1] + vi * c[2 * j];
        }
    }
    double zr, zi;
    nearest_root64<KS>(wr, wi, K, roots, zr, zi);
#pragma unroll
    for (int j = 0; j < R; ++j) {
        if constexpr (REAL) {
            const double vr = (double)row[j];
            acc[2 * j] += vr * zr;
            acc[2 * j + 1] += vr * zi;
        } else {
            const double vr = (double)row[2 * j], vi = (double)row[2 * j + 1];
            acc[2 * j] += vr * zr + vi * zi;
            acc[2 * j + 1] += vr * zi - vi * zr;
        }
    }
}

template <int R, bool REAL, int KS>
__global__ __launch_bounds__(kBlock) void k_rescore(RescoreParams p) {
    __shared__ double2 roots_s[LRQO_MAX_K];
    __shared__ double red[kBlock / kWave][2 * R];
    for (int k = threadIdx.x; k < p.K; k += kBlock) roots_s[k] = p.roots64[k];
    __syncthreads();
    const int t = blockIdx.x;
    const uint32_t idx = key_index(p.keys[t]);
    float cf[2 * R];
    direction_any<R>(p.dirs, p.seed, p.first + idx, p.instance, cf);
    double c[2 * R], acc[2 * R];
#pragma unroll
    for (int j = 0; j < 2 * R; ++j) {
        c[j] = (double)cf[j];
        acc[j] = 0.0;
    }
    const int64_t r0 = (int64_t)blockIdx.y * p.rows_per_slice;
    const int64_t r1 = min(p.n, r0 + p.rows_per_slice);
    constexpr int RF = Row<R, REAL>::F;
    // four rows' loads in flight; the rows are still added in order
    int64_t i = r0 + threadIdx.x;
    for (; i + 3 * kBlock < r1; i += 4 * kBlock) {
        float rows[4][RF];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int e = 0; e < RF; ++e) rows[u][e] = p.V[(i + (int64_t)u * kBlock) * RF + e];
#pragma unroll
        for (int u = 0; u < 4; ++u) rescore_row<R, REAL, KS>(rows[u], c, p.K, roots_s, acc);
    }
    for (; i < r1; i += kBlock) {
        float row[RF];
#pragma unroll
        for (int e = 0; e < RF; ++e) row[e] = p.V[i * RF + e];
        rescore_row<R, REAL, KS>(row, c, p.K, roots_s, acc);
    }
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
#pragma unroll
    for (int j = 0; j < 2 * R; ++j) {
        const double s = wave_sum_f64(acc[j]);
        if (lane == 0) red[wave][j] = s;
    }
    __syncthreads();
    if (threadIdx.x < 2 * R) {
        double s = 0.0;
        for (int w = 0; w < kBlock / kWave; ++w) s += red[w][threadIdx.x];
        p.partial[((size_t)t * gridDim.y + blockIdx.y) * (2 * R) + threadIdx.x] = s;
    }
}

// FP64 arg-max over the wave of the kept candidates' values f (lane t: key of
// candidate t), ties to the lowest index; every lane gets the winner.
__device__ __forceinline__ void wave_pick(double& f, unsigned long long& key, uint32_t& idx) {
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        const double fo = __shfl_xor(f, off, kWave);
        const uint32_t io = __shfl_xor(idx, off, kWave);
        const unsigned long long ko = __shfl_xor(key, off, kWave);
        if (fo > f || (fo == f && io < idx)) {
            f = fo;
            idx = io;
            key = ko;
        }
    }
}

// Thread (t, j) sums component j of kept candidate t over the slices
// (fixed order, eight loads in flight); lane t of wave 0 forms f_t, and a
// butterfly over the wave takes the FP64 arg-max, ties to the lowest index.
template <int R>
__global__ __launch_bounds__(64 * 2 * R) void k_pick(const double* __restrict__ partial, int T, int P,
                                                     const unsigned long long* __restrict__ keys,
                                                     uint64_t seed, uint32_t instance, uint64_t first,
                                                     const float* dirs, const int* __restrict__ bad, int nbad,
                                                     DevResult* res) {
    __shared__ double comp[64][2 * R];
    const int t = threadIdx.x / (2 * R), j = threadIdx.x % (2 * R);
    if (t < T) {
        const double* src = partial + (size_t)t * P * (2 * R) + j;
        double a = 0.0;
        int q = 0;
        for (; q + 8 <= P; q += 8) {
            double v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = src[(size_t)(q + u) * (2 * R)];
#pragma unroll
            for (int u = 0; u < 8; ++u) a += v[u];
        }
        for (; q < P; ++q) a += src[(size_t)q * (2 * R)];
        comp[t][j] = a;
    }
    int b = 0;                                   // the prologue's finiteness flags
    for (int q = threadIdx.x; q < nbad; q += blockDim.x) b |= bad[q] & kFlagNonfinite;
    const int any_bad = __syncthreads_or(b);
    if (threadIdx.x >= kWave) return;
    const int lane = threadIdx.x;
    double f = -1.0;
    unsigned long long key = 0ull;
    uint32_t idx = 0xFFFFFFFFu;
    if (lane < T) {
        double s = 0.0;
        for (int jj = 0; jj < 2 * R; ++jj) s += comp[lane][jj] * comp[lane][jj];
        key = keys[lane];
        idx = key_index(key);
        f = s >= 0.0 ? s : -1.0;      // a non-finite score is never picked
    }
    wave_pick(f, key, idx);
    if (lane != 0) return;
    if (f < 0.0) {  // only with non-finite scores; the host reports the error
        key = keys[0];
        idx = key_index(key);
    }
    float cf[2 * R];
    direction_any<R>(dirs, seed, first + idx, instance, cf);
    res->nonfinite = any_bad ? 1 : 0;
    res->best_index = (int64_t)(first + idx);
    res->obj = f;
    res->fp32_obj = (double)key_value(key);
    for (int jj = 0; jj < 2 * LRQO_MAX_R; ++jj) res->c[jj] = jj < 2 * R ? (double)cf[jj] : 0.0;
}

// FP64 decision rule of one row at direction c.
template <int R, bool REAL>
__device__ __forceinline__ uint8_t row_label(const float* row, const double* c, int K) {
    double wr = 0.0, wi = 0.0;
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const double vr = REAL ? (double)row[j] : (double)row[2 * j];
        const double vi = REAL ? 0.0 : (double)row[2 * j + 1];
        wr += vr * c[2 * j] - vi * c[2 * j + 1];
        wi += vr * c[2 * j + 1] + vi * c[2 * j];
    }
    return (uint8_t)label_f64(wr, wi, K);
}

template <int R, bool REAL>
__global__ __launch_bounds__(kBlock) void k_labels(const float* __restrict__ V, int64_t n, int K,
                                                   const DevResult* __restrict__ res,
                                                   uint8_t* __restrict__ z) {
    constexpr int RF = Row<R, REAL>::F;
    const int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x;
    if (i >= n) return;
    z[i] = row_label<R, REAL>(V + i * RF, res->c, K);
}

// ------------------------------------------------------------ small problems
// Everything after the scorer in one block: the best T keys, their FP64
// values, the pick and the labels.  With at most kTailRows rows a thread of
// k_rescore holds one row, and the four kernels (17 us for the selection, 5, 4
// and 2 for the others at n = 64, S = 1,024) are latency and launches; here
// sixteen waves sort a tile of scores each and merge them in a tree; then a
// lane holds a kept candidate and the waves split the rows, in the order of
// k_rescore's sums, so every value is the same number.  A call also loses the prologue and the copy of the
// record: 81 -> 52 us at n = 64, r = 2, K = 4, S = 1,024, 116 -> 103 us at
// n = 256, r = 4, K = 16, S = 8,192.  One compute unit does all of it, so the
// range ends there; an arbitrary K (an FP64 arctangent for each row and
// candidate) took 146 -> 165 us at n = 256 and keeps to one group of 64 rows.
constexpr int kTailRows = 256;         // k_rescore's block: one row a thread
constexpr int kTailRowsAnyK = 64;
constexpr int64_t kTailScores = 8192;  // eight tiles a wave
constexpr int kTailWaves = 16;

struct TailParams {
    RescoreParams rs;
    const float* f;
    uint32_t S;
    int T;
    int ks;                            // k_special(K)
    const int* bad;                    // the prologue's finiteness flags; null: no prologue ran
    int nbad;
    const DevResult* prev;             // the record the scorer counted flagged rows in
    DevResult* res;
    uint8_t* z;
};

// Rows g + w, + 16, + 32 and + 48 of a group of 64 for candidate `lane`: the
// first two levels of k_rescore's sum over the group (it pairs lanes 32 apart,
// then 16, 8, 4, 2, 1).  Rows beyond n count as zeros there too.
template <int R, bool REAL, int KS>
__device__ __forceinline__ void tail_rows(const TailParams& p, const float* Vs, int i0, const double (&c)[2 * R],
                                          double (&out)[2 * R]) {
    constexpr int RF = Row<R, REAL>::F;
#pragma unroll 1
    for (int h = 0; h < 2; ++h) {                    // pairs (0, 32) and (16, 48); one at a time: registers
        double a[2][2 * R];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int i = i0 + 16 * h + 32 * u;
#pragma unroll
            for (int j = 0; j < 2 * R; ++j) a[u][j] = 0.0;
            if (i < (int)p.rs.n) {                   // the same in every lane
                float row[RF];
#pragma unroll
                for (int e = 0; e < RF; ++e) row[e] = Vs[i * RF + e];
                rescore_row<R, REAL, KS>(row, c, p.rs.K, p.rs.roots64, a[u]);
            }
        }
#pragma unroll
        for (int j = 0; j < 2 * R; ++j) {
            const double pair = a[0][j] + a[1][j];
            out[j] = h == 0 ? pair : out[j] + pair;
        }
    }
}

template <int R, bool REAL>
__global__ __launch_bounds__(kTailWaves * kWave) void k_tail(TailParams p) {
    constexpr int RF = Row<R, REAL>::F;
    __shared__ float Vs[kTailRows * RF];
    __shared__ unsigned long long top[kTailWaves][kWave];
    __shared__ double part[kTailWaves][2 * R][kWave];
    __shared__ double comp[2 * R][kWave];
    __shared__ double cbest[2 * R];
    const int tid = threadIdx.x, lane = tid % kWave, w = tid / kWave;
    const int n = (int)p.rs.n;
    int b = 0;
    for (int e = tid; e < n * RF; e += kTailWaves * kWave) {
        const float x = p.rs.V[e];
        Vs[e] = x;
        b |= !isfinite(x);
    }
    if (p.bad)
        for (int q = tid; q < p.nbad; q += kTailWaves * kWave) b |= p.bad[q] & kFlagNonfinite;
    // the best 64 keys
    unsigned long long run = 0;
    for (uint32_t g0 = w * kWave; g0 < p.S; g0 += kTailWaves * kWave) {
        const uint32_t g = g0 + lane;
        const unsigned long long key = g < p.S ? pack_key(p.f[g], g) : 0ull;
        const unsigned long long floor64 = __shfl(run, 63, kWave);
        if (__ballot(key > floor64) == 0) continue;  // uniform across the wave
        const unsigned long long tile = wave_sort_desc(key, lane);
        run = g0 == (uint32_t)(w * kWave) ? tile : wave_top_union(run, tile, lane);
    }
    top[w][lane] = run;
    const int any_bad = __syncthreads_or(b);
    for (int h = kTailWaves / 2; h > 0; h >>= 1) {
        if (w < h && (uint32_t)((w + h) * kWave) < p.S) {   // uniform across the wave; beyond S: empty lists
            run = wave_top_union(run, top[w + h][lane], lane);
            top[w][lane] = run;
        }
        __syncthreads();
    }
    // lane t: candidate t
    unsigned long long key = lane < p.T ? top[0][lane] : 0ull;
    uint32_t idx = lane < p.T ? key_index(key) : 0u;
    float cf[2 * R];
    direction_any<R>(p.rs.dirs, p.rs.seed, p.rs.first + idx, p.rs.instance, cf);
    double c[2 * R];
#pragma unroll
    for (int j = 0; j < 2 * R; ++j) c[j] = (double)cf[j];
    double sum = 0.0;                            // thread (component w, candidate lane)
    for (int g = 0; g < n; g += kWave) {
        double s[2 * R];
        switch (p.ks) {
            case 2: tail_rows<R, REAL, 2>(p, Vs, g + w, c, s); break;
            case 3: tail_rows<R, REAL, 3>(p, Vs, g + w, c, s); break;
            case 4: tail_rows<R, REAL, 4>(p, Vs, g + w, c, s); break;
            case 8: tail_rows<R, REAL, 8>(p, Vs, g + w, c, s); break;
            case 16: tail_rows<R, REAL, 16>(p, Vs, g + w, c, s); break;
            default: tail_rows<R, REAL, 0>(p, Vs, g + w, c, s); break;
        }
#pragma unroll
        for (int j = 0; j < 2 * R; ++j) part[w][j][lane] = s[j];
        __syncthreads();
        if (w < 2 * R) {
            double v[kTailWaves];
#pragma unroll
            for (int q = 0; q < kTailWaves; ++q) v[q] = part[q][w][lane];
#pragma unroll
            for (int h = kTailWaves / 2; h > 0; h >>= 1)
#pragma unroll
                for (int q = 0; q < h; ++q) v[q] += v[q + h];
            sum += v[0];
        }
        __syncthreads();
    }
    if (w < 2 * R) comp[w][lane] = sum;
    __syncthreads();
    if (w == 0) {
        double f = -1.0;
        if (lane < p.T) {
            double s = 0.0;
            for (int jj = 0; jj < 2 * R; ++jj) s += comp[jj][lane] * comp[jj][lane];
            f = s >= 0.0 ? s : -1.0;      // a non-finite score is never picked
        } else {
            idx = 0xFFFFFFFFu;
        }
        const uint32_t own = idx;
        const unsigned long long key0 = __shfl(key, 0, kWave);
        wave_pick(f, key, idx);
        if (f < 0.0) {  // only with non-finite scores; the host reports the error
            key = key0;
            idx = key_index(key);
        }
        if (own == idx && lane < p.T) {   // the winner's lane: one, as the kept indices differ
            DevResult o{};
            o.nonfinite = any_bad ? 1 : 0;
            o.best_index = (int64_t)(p.rs.first + idx);
            o.obj = f;
            o.fp32_obj = (double)key_value(key);
#pragma unroll
            for (int jj = 0; jj < 2 * R; ++jj) o.c[jj] = c[jj];
            o.flagged_rows = p.bad ? p.prev->flagged_rows : 0ull;
            *p.res = o;
#pragma unroll
            for (int jj = 0; jj < 2 * R; ++jj) cbest[jj] = c[jj];
        }
    }
    __syncthreads();
    if (tid < n) p.z[tid] = row_label<R, REAL>(Vs + tid * RF, cbest, p.rs.K);
}

// ------------------------------------------------------------ host driver
// Candidates per lane, and per block (the MFMA scorers' waves hold distinct
// ones; the four waves of the r <= 4 vector-ALU scorer share one set of
// 64*CPL candidates, the lanes of the r > 4 one hold distinct ones).
int cands_per_lane(int R) { return R <= 4 ? LRQO_SCORE_CPL : 1; }
int cands_per_block(int R) { return R <= 4 ? kWave * cands_per_lane(R) : kBlock * cands_per_lane(R); }
int cands_per_block(const SampledJob& job, ScoreForm form) {
    if (form == kFormSplit) return kSplitCands;
    const bool mfma = form == kFormPrecision && job.r <= 4 && (job.K == 2 || job.K == 3 || job.K == 4) && bf16_form() == 0;
    return mfma ? kBf16xCands : cands_per_block(job.r);
}

// The scorer of a call.  k_score_split takes K = 2, 3, 4, 8, 16 and
// 2 <= r <= 4 in both precisions: it is 1.7 to 3.9 times as fast as the FP32
// scorer at every n tried (5,000 rows, r = 3 real, K = 3: 0.049 against
// 0.155 ms for 4,096 candidates; 10^6 rows: 17.3 against 30.5 ms for 131,072;
// r = 3 complex, K = 16, 200,000 rows: 5.0 against 14.9 ms for 65,536) and its
// scores lie 4 to 70 times closer to FP64.  It is kept to problems whose
// assignments far outnumber the candidates of an ordinary call (2^20): where
// many candidates round to one assignment up to a rotation their objectives are
// equal, only the rounding of the score orders them, and the scorers that
// served such sizes before keep doing so.  The count is the order of the
// arrangement's vertices, n^(2r-1), at least 2^33 from n = 2,048 on; for real V
// and K = 4 the quadrants of the turned w depend on Re c and Im c apart
// (n^(2r-2): r = 2 from 2^32 on) and for real V and K = 2 on Re c alone (few
// assignments, not taken).  The call's own S has no part in it: the pieces of a
// range of directions are scored as the whole.
ScoreForm score_form(const SampledJob& job) {
    const ScoreForm plain = job.precision == 1 ? kFormPrecision : kFormFp32;
    if (k_special(job.K) == 0 || job.r < 2 || job.r > 4 || (job.real && job.K == 2)) return plain;
    if (job.n < 2048 || job.n > kSplitMaxRows || (plain == kFormPrecision && bf16_form() == 1)) return plain;
    if (job.real && job.K == 4 && job.r == 2 && job.n < 65536) return plain;
    return kFormSplit;
}

template <int R, bool REAL, int KS>
void launch_score(const ScoreParams& p, dim3 grid, hipStream_t st) {
    constexpr int CPL = R <= 4 ? LRQO_SCORE_CPL : 1;
    if constexpr (R <= 4) {
        hipLaunchKernelGGL((k_score_rows<R, CPL, REAL, KS, false>), grid, dim3(kBlock), 0, st, p);
    } else {
        hipLaunchKernelGGL((k_score<R, CPL, REAL, KS, false>), grid, dim3(kBlock), 0, st, p);
    }
}

template <int R, bool REAL, int KS>
void launch_score_bf16(const ScoreParams& p, dim3 grid, hipStream_t st) {
    if constexpr (R <= 4) {
        if constexpr (KS == 2 || KS == 3 || KS == 4) {
            if (bf16_form() == 0) {
                hipLaunchKernelGGL((k_score_bf16x<R, REAL, KS, false>), grid, dim3(kBlock), 0, st, p);
                return;
            }
        }
        hipLaunchKernelGGL((k_score_bf16<R, LRQO_SCORE_CPL, REAL, KS, LRQO_BF16_SPLIT, false>), grid, dim3(kBlock), 0,
                           st, p);
    }
}

template <int R, bool REAL, int KS>
void launch_score_split(const ScoreParams& p, dim3 grid, hipStream_t st) {
    if constexpr (R >= 2 && R <= 4 && !(REAL && KS == 2)) {
        if constexpr (R == 3 && REAL) {
            if (p.quick) {
                hipLaunchKernelGGL((k_score_split<R, REAL, KS, false, true>), grid, dim3(kSplitBlock), 0, st, p);
                return;
            }
        }
        hipLaunchKernelGGL((k_score_split<R, REAL, KS, false, false>), grid, dim3(kSplitBlock), 0, st, p);
    }
}

template <int R, bool REAL>
void launch_score_k(const ScoreParams& p, dim3 grid, hipStream_t st, ScoreForm form) {
    if (p.probe_count > 0) {   // the same scorers with the probed candidates' labels written out
        launch_score_probe(p, grid, st, R, REAL, form);
        return;
    }
    if (form == kFormSplit) {
        switch (p.K) {
            case 2: launch_score_split<R, REAL, 2>(p, grid, st); break;
            case 3: launch_score_split<R, REAL, 3>(p, grid, st); break;
            case 4: launch_score_split<R, REAL, 4>(p, grid, st); break;
            case 8: launch_score_split<R, REAL, 8>(p, grid, st); break;
            default: launch_score_split<R, REAL, 16>(p, grid, st); break;
        }
        return;
    }
    if (form == kFormPrecision) {
        switch (p.K) {
            case 2: launch_score_bf16<R, REAL, 2>(p, grid, st); break;
            case 3: launch_score_bf16<R, REAL, 3>(p, grid, st); break;
            case 4: launch_score_bf16<R, REAL, 4>(p, grid, st); break;
            default: launch_score_bf16<R, REAL, 0>(p, grid, st); break;
        }
        return;
    }
    switch (p.K) {
        case 2: launch_score<R, REAL, 2>(p, grid, st); break;
        case 3: launch_score<R, REAL, 3>(p, grid, st); break;
        case 4: launch_score<R, REAL, 4>(p, grid, st); break;
        case 8: launch_score<R, REAL, 8>(p, grid, st); break;
        case 16: launch_score<R, REAL, 16>(p, grid, st); break;
        default: launch_score<R, REAL, 0>(p, grid, st); break;
    }
}

template <int R, bool REAL>
lrqo_status run_sampled(const SampledJob& job, Scratch& sc, hipStream_t st) {
    const uint32_t S = (uint32_t)job.S;
    if (sc.prologue) {
        if constexpr (R >= 2 && R <= 4) {
            if (sc.form == kFormSplit)
                hipLaunchKernelGGL((k_prologue<R, REAL, true>), dim3(kCheckBlocks), dim3(kBlock), 0, st, job.K,
                                   sc.roots64, sc.roots32, sc.result, job.V, job.n, sc.bad_blocks, sc.vmax, sc.tile_exp,
                                   job.dirs, S);
        }
        if (sc.form != kFormSplit)       // V as one column of floats
            hipLaunchKernelGGL((k_prologue<1, true, false>), dim3(kCheckBlocks), dim3(kBlock), 0, st, job.K,
                               sc.roots64, sc.roots32, sc.result, job.V, job.n * Row<R, REAL>::F, sc.bad_blocks,
                               sc.vmax, nullptr, nullptr, 0u);
        LRQO_HIP(hipGetLastError());
    }

    // ---- fused scorer
    ScoreParams p{};
    p.V = job.V;
    p.n = job.n;
    p.K = job.K;
    p.seed = job.seed;
    p.instance = job.instance;
    p.first = job.first;
    p.S = S;
    p.f_out = sc.f32;
    p.partial = sc.partial;
    p.roots32 = sc.roots32;
    p.rows_per_slice = sc.rows_per_slice;
    LRQO_HIP(hipEventRecord(job.ev_score0, st));
    p.flagged = &sc.result->flagged_rows;
    p.dirs = job.dirs;
    p.dirs_out = job.dirs_out;
    p.probe_out = job.probe_out;
    p.probe_count = job.probe_count;
    for (int t = 0; t < job.probe_count; ++t) p.probe_idx[t] = job.probe_idx[t];
    p.vmax = sc.vmax;
    p.vmax_count = kCheckBlocks;
    p.tile_exp = sc.tile_exp;
    p.quick = job.precision == 1;
    const auto launch = [&](ScoreForm form) {
        const int64_t cpb = cands_per_block(job, form);
        launch_score_k<R, REAL>(p, dim3((unsigned)((S + cpb - 1) / cpb), (unsigned)sc.slices), st, form);
    };
    if (sc.form == kFormSplit && job.dirs) {   // one of the two returns at once (4 us)
        p.list_flags = sc.bad_blocks;
        p.list_flag_count = kCheckBlocks;
        launch(kFormSplit);
        launch(kFormFp32);
    } else {
        launch(sc.form);
    }
    LRQO_HIP(hipGetLastError());
    LRQO_HIP(hipEventRecord(job.ev_score1, st));
    const int T = sc.topk;
    RescoreParams rp{};
    rp.V = job.V;
    rp.n = job.n;
    rp.K = job.K;
    rp.seed = job.seed;
    rp.instance = job.instance;
    rp.first = job.first;
    rp.roots64 = sc.roots64;
    rp.partial = sc.rescore;
    rp.rows_per_slice = sc.rescore_rows;
    rp.dirs = job.dirs;
    if constexpr (R <= 4) {
        if (sc.tail) {
            hipLaunchKernelGGL((k_tail<R, REAL>), dim3(1), dim3(kTailWaves * kWave), 0, st,
                               TailParams{rp, sc.f32, S, T, k_special(job.K), sc.prologue ? sc.bad_blocks : nullptr,
                                          kCheckBlocks, sc.result, job.host_result ? job.host_result : sc.result,
                                          job.z});
            LRQO_HIP(hipGetLastError());
            return LRQO_OK;
        }
    }
    // ---- top-T
    const unsigned long long* keys = nullptr;
    if (sc.slices > 1) {
        const uint32_t fblocks = (S + kBlock - 1) / kBlock;
        hipLaunchKernelGGL((k_finalize<R>), dim3(fblocks), dim3(kBlock), 0, st, sc.partial, sc.slices, S, sc.f32,
                           sc.lists);
        LRQO_HIP(hipGetLastError());
        LRQO_TRY(topk_select_lists(sc.lists, fblocks * kBlock, T, sc.keys_a, sc.keys_b, st, &keys));
    } else {
        LRQO_TRY(topk_select(sc.f32, S, T, sc.keys_a, sc.keys_b, st, &keys));
    }

    // ---- FP64 rescore of the T kept keys
    rp.keys = keys;
    const dim3 rgrid(T, sc.rescore_slices);
    switch (k_special(job.K)) {
        case 2: hipLaunchKernelGGL((k_rescore<R, REAL, 2>), rgrid, dim3(kBlock), 0, st, rp); break;
        case 3: hipLaunchKernelGGL((k_rescore<R, REAL, 3>), rgrid, dim3(kBlock), 0, st, rp); break;
        case 4: hipLaunchKernelGGL((k_rescore<R, REAL, 4>), rgrid, dim3(kBlock), 0, st, rp); break;
        case 8: hipLaunchKernelGGL((k_rescore<R, REAL, 8>), rgrid, dim3(kBlock), 0, st, rp); break;
        case 16: hipLaunchKernelGGL((k_rescore<R, REAL, 16>), rgrid, dim3(kBlock), 0, st, rp); break;
        default: hipLaunchKernelGGL((k_rescore<R, REAL, 0>), rgrid, dim3(kBlock), 0, st, rp); break;
    }
    LRQO_HIP(hipGetLastError());
    hipLaunchKernelGGL((k_pick<R>), dim3(1), dim3(64 * 2 * R), 0, st, sc.rescore, T, sc.rescore_slices, keys,
                       job.seed, job.instance, job.first, job.dirs, sc.bad_blocks, kCheckBlocks, sc.result);
    LRQO_HIP(hipGetLastError());
    hipLaunchKernelGGL((k_labels<R, REAL>), dim3((unsigned)((job.n + kBlock - 1) / kBlock)),
                       dim3(kBlock), 0, st, job.V, job.n, job.K, sc.result, job.z);
    LRQO_HIP(hipGetLastError());
    return LRQO_OK;
}

template <bool REAL>
lrqo_status dispatch_r(const SampledJob& job, Scratch& sc, hipStream_t st) {
    switch (job.r) {
        case 1: return run_sampled<1, REAL>(job, sc, st);
        case 2: return run_sampled<2, REAL>(job, sc, st);
        case 3: return run_sampled<3, REAL>(job, sc, st);
        case 4: return run_sampled<4, REAL>(job, sc, st);
        case 5: return run_sampled<5, REAL>(job, sc, st);
        case 6: return run_sampled<6, REAL>(job, sc, st);
        case 7: return run_sampled<7, REAL>(job, sc, st);
        case 8: return run_sampled<8, REAL>(job, sc, st);
        default: return fail(LRQO_EINVAL, "r out of range");
    }
}

}  // namespace

// Doubles of the rescore's buffer, which holds the tiles' exponents before it
// (they fit in it where the call keeps 64 candidates).
static size_t rescore_doubles(const SampledJob& job, const ScratchPlan& plan) {
    static_assert(sizeof(TileExp) == sizeof(double), "one per tile");
    const size_t tiles = plan.form == kFormSplit ? (size_t)((job.n + kSplitTile - 1) / kSplitTile) : 0;
    return std::max(tiles, (size_t)plan.topk * plan.rescore_slices * 2 * job.r);
}

// Plans the launch shapes and the scratch layout of one sampled solve.
void plan_sampled(const SampledJob& job, ScratchPlan& plan) {
    const int R = job.r;
    plan.form = score_form(job);
    const int cpb = cands_per_block(job, job.precision == 1 ? kFormPrecision : kFormFp32);
    const int64_t cand_blocks = (job.S + cpb - 1) / cpb;
    // enough blocks to fill 256 CUs several times over, slices of >= 1024 rows
    int64_t slices = std::max<int64_t>(1, (LRQO_SCORE_BLOCKS + cand_blocks - 1) / cand_blocks);
    slices = std::min<int64_t>(slices, std::max<int64_t>(1, job.n / 1024));
    if (plan.form == kFormSplit) {
        // two blocks fit a CU, one for K = 8 and 16: of the slice counts up to
        // that of the other scorers (so no call needs more scratch than it
        // did), the smallest whose last round of blocks is nearly full, or
        // the one that fills it best (the finer split among equals)
        const int64_t blocks = (job.S + kSplitCands - 1) / kSplitCands, slots = 256 * split_waves(job.K) / 2;
        int64_t best = slices;
        double best_fill = 0.0;
        for (int64_t s = 1; s <= slices; ++s) {
            const double fill = (double)(blocks * s) / (double)((blocks * s + slots - 1) / slots * slots);
            if (fill > best_fill - 0.01) {
                best_fill = std::max(best_fill, fill);
                best = s;
            }
            if (fill >= 0.95) break;
        }
        slices = best;
    }
    int64_t rows = (job.n + slices - 1) / slices;
    const int64_t align = plan.form == kFormSplit ? kSplitTile : 64;
    rows = ((rows + align - 1) / align) * align;
    slices = (job.n + rows - 1) / rows;
    plan.slices = (int)slices;
    plan.rows_per_slice = rows;
    plan.topk = (int)std::min<int64_t>(job.topk, job.S);
    int64_t rrows = std::max<int64_t>(4096, (job.n + 127) / 128);
    plan.rescore_rows = rrows;
    plan.rescore_slices = (int)((job.n + rrows - 1) / rrows);
    plan.tail = R <= 4 && job.n <= (k_special(job.K) ? kTailRows : kTailRowsAnyK) &&
                job.S <= kTailScores && plan.slices == 1;
    CarveSize cs;
    cs.add<DevResult>(1);
    cs.add<float2>(LRQO_MAX_K);
    cs.add<double2>(LRQO_MAX_K);
    cs.add<float>(job.f_out ? 0 : job.S);
    cs.add<float>(slices > 1 ? (size_t)slices * 2 * R * job.S : 0);
    cs.add<unsigned long long>(topk_buffer_keys((uint32_t)job.S, plan.topk));
    cs.add<unsigned long long>(topk_buffer_keys((uint32_t)job.S, plan.topk));
    cs.add<unsigned long long>(slices > 1 ? (size_t)(job.S + kBlock - 1) / kBlock * kBlock : 0);
    cs.add<double>(rescore_doubles(job, plan));
    cs.add<int>(kCheckBlocks);
    cs.add<float>(kCheckBlocks);
    plan.bytes = cs.bytes;
}

lrqo_status launch_sampled(const SampledJob& job, const ScratchPlan& plan, void* arena, hipStream_t st) {
    Carve cv(arena);
    Scratch sc{};
    sc.result = cv.take<DevResult>(1);
    sc.roots32 = cv.take<float2>(LRQO_MAX_K);
    sc.roots64 = cv.take<double2>(LRQO_MAX_K);
    sc.f32 = job.f_out ? job.f_out : cv.take<float>(job.S);
    sc.form = plan.form;
    sc.slices = plan.slices;
    sc.rows_per_slice = plan.rows_per_slice;
    sc.partial = plan.slices > 1 ? cv.take<float>((size_t)plan.slices * 2 * job.r * job.S) : nullptr;
    sc.topk = plan.topk;
    sc.keys_a = cv.take<unsigned long long>(topk_buffer_keys((uint32_t)job.S, plan.topk));
    sc.keys_b = cv.take<unsigned long long>(topk_buffer_keys((uint32_t)job.S, plan.topk));
    sc.lists = plan.slices > 1 ? cv.take<unsigned long long>((size_t)(job.S + kBlock - 1) / kBlock * kBlock)
                               : nullptr;
    sc.rescore_slices = plan.rescore_slices;
    sc.rescore_rows = plan.rescore_rows;
    sc.rescore = cv.take<double>(rescore_doubles(job, plan));
    sc.tile_exp = reinterpret_cast<TileExp*>(sc.rescore);   // used up before the rescore

    sc.bad_blocks = cv.take<int>(kCheckBlocks);
    sc.vmax = cv.take<float>(kCheckBlocks);

    // a small solve whose scorer reads neither the roots, nor the largest
    // entry, nor counts into the record leaves the checks to k_tail
    sc.tail = plan.tail;
    sc.prologue = !(plan.tail && plan.form == kFormFp32 && k_special(job.K) != 0 && !(job.real && job.K == 3));
    return job.real ? dispatch_r<true>(job, sc, st) : dispatch_r<false>(job, sc, st);
}

}  // namespace lrqo
