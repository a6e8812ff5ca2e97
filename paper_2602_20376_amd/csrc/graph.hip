// Objective on the graph and greedy local refinement (appendix "Rank-1 at
// Scale": incremental scoring, eq. incremental; hybrid warm start) for the
// Laplacian Q = L = D - A of a weighted graph in CSR.
//
// Kernels:
//   k_check_ptr     row_ptr[0] = 0, non-decreasing, row_ptr[n] = nnz
//   k_check_rows    0 <= col < n, no self loop, finite weights, labels < K
//                   (only after k_check_ptr passed: it reads col through row_ptr)
//   k_objective     per vertex: sum over its entries of w |z_i - z_j|^2 and of
//                   w [k_i != k_j] (each edge is seen from both ends), block
//                   partial sums in a fixed order
//   k_sum2          fixed-order sum of the block partials
//   k_gain          per vertex whose own label or a neighbour's changed since
//                   its last gain: neighbour label weights c_k in LDS, the best
//                   other label and its gain 2 sum_k c_k (cos(a-k) - cos(b-k));
//                   the others keep theirs
//   k_move          per candidate: moves when its (gain, -index) beats every
//                   neighbouring candidate, and marks itself and its neighbours
//                   for the next k_gain; the movers are an independent set and
//                   no label is read here, so labels change in place; moves
//                   counted per round (per block, into 64 counters)
// Later rounds move few vertices, so most gains stand (10^5 vertices, mean
// degree 10, 24 launched rounds: gains 203 -> 149 us; moves, which now also
// leave the marks, 124 -> 142; the whole call 0.49 -> 0.44 ms).  A round that
// changes nothing still takes 5 us a kernel, against 1.8 us for one that
// returns at once: what is left is the chain of dependent reads.
// Rounds go out in batches between host checks; a round whose predecessor
// moved nothing returns at once, so a batch that converges early costs a
// launch per remaining round.  The layout checks, the first objective and the
// first batch are queued together: each kernel returns at once when a check
// before it failed, and the host reads the verdict with the batch's counts.
// The checks, the objective and the gains of weighted graphs or K > 4 take a
// thread per vertex, which reads its CSR entries in order; unit gains and the
// moves give a row to sixteen lanes and add whole numbers or compare.  So every
// per-vertex sum has a fixed order.
#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstring>
#include <string>

#include "graph_internal.h"
#include "lrqo_device.h"
#include "lrqo_runtime.h"

namespace lrqo {

namespace {

constexpr int kBlock = 256;
#ifndef LRQO_REFINE_BLOCK
#define LRQO_REFINE_BLOCK 512
#endif
constexpr int kRefineBlock = LRQO_REFINE_BLOCK;   // threads per block of the gain and move kernels
constexpr int kMaxKRefine = 16;

enum : int { kBadPtr = 1, kBadCol = 2, kBadWeight = 4, kBadLabel = 8 };

struct GraphDev {
    const int64_t* row_ptr;
    const int32_t* col;
    const double* w;
    int64_t n;
    int64_t nnz;
};

__global__ __launch_bounds__(kBlock) void k_check_ptr(GraphDev g, int* flag) {
    const int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x;
    bool bad = false;
    if (i < g.n) bad = g.row_ptr[i] > g.row_ptr[i + 1];
    if (i == 0) bad = bad || g.row_ptr[0] != 0 || g.row_ptr[g.n] != g.nnz;
    if (bad) atomicOr(flag, kBadPtr);
}

__global__ __launch_bounds__(kBlock) void k_check_rows(GraphDev g, int K, const uint8_t* z, int* flag) {
    const int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x;
    if (i >= g.n || (*flag & kBadPtr)) return;   // k_check_ptr failed: row_ptr must not be followed
    int bad = (z && z[i] >= K) ? kBadLabel : 0;
    for (int64_t e = g.row_ptr[i]; e < g.row_ptr[i + 1]; ++e) {
        const int32_t j = g.col[e];
        if (j < 0 || j >= g.n || j == i) bad |= kBadCol;
        if (g.w && !isfinite(g.w[e])) bad |= kBadWeight;
    }
    if (bad) atomicOr(flag, bad);
}

// Block sums of two doubles per thread, fixed tree order.
__device__ __forceinline__ void block_sum2(double a, double b, double* out) {
    __shared__ double sa[kBlock], sb[kBlock];
    sa[threadIdx.x] = a;
    sb[threadIdx.x] = b;
    __syncthreads();
    for (unsigned h = kBlock / 2; h > 0; h >>= 1) {
        if (threadIdx.x < h) {
            sa[threadIdx.x] += sa[threadIdx.x + h];
            sb[threadIdx.x] += sb[threadIdx.x + h];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        out[0] = sa[0];
        out[1] = sb[0];
    }
}

// sqd[d] = |1 - omega^d|^2 for the label difference d = (k_i - k_j) mod K.
// The terms of the entries [e, e1) of vertex i (label a) in chunks of U:
// the U column and weight loads, then the U label loads, are issued
// together; the additions keep entry order.  Leaves e at the first entry of
// an incomplete chunk.
template <int U>
__device__ __forceinline__ void objective_chunk(const GraphDev& g, int K, const uint8_t* __restrict__ z,
                                                const double* __restrict__ sqd, int a, int64_t& e, int64_t e1,
                                                double& q, double& cut) {
    for (; e + U <= e1; e += U) {
        int32_t c[U];
        double w[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            c[u] = g.col[e + u];
            w[u] = g.w ? g.w[e + u] : 1.0;
        }
        int b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) b[u] = z[c[u]];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            int d = a - b[u];
            d += d < 0 ? K : 0;
            q += w[u] * sqd[d];
            cut += a != b[u] ? w[u] : 0.0;
        }
    }
}

__global__ __launch_bounds__(kBlock) void k_objective(GraphDev g, int K, const uint8_t* __restrict__ z,
                                                      const double* __restrict__ sqd,
                                                      double* __restrict__ partial, const int* __restrict__ flag) {
    const int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x;
    double q = 0.0, cut = 0.0;
    if (i < g.n && *flag == 0) {
        const int a = z[i];
        int64_t e = g.row_ptr[i];
        const int64_t e1 = g.row_ptr[i + 1];
        objective_chunk<8>(g, K, z, sqd, a, e, e1, q, cut);
        objective_chunk<4>(g, K, z, sqd, a, e, e1, q, cut);
        for (; e < e1; ++e) {
            const int b = z[g.col[e]];
            const double w = g.w ? g.w[e] : 1.0;
            int d = a - b;
            d += d < 0 ? K : 0;
            q += w * sqd[d];
            cut += a != b ? w : 0.0;
        }
    }
    block_sum2(q, cut, partial + 2 * blockIdx.x);
}

__global__ __launch_bounds__(kBlock) void k_sum2(const double* __restrict__ partial, int64_t blocks,
                                                 double* __restrict__ out) {
    double a = 0.0, b = 0.0;
    for (int64_t t = threadIdx.x; t < blocks; t += kBlock) {
        a += partial[2 * t];
        b += partial[2 * t + 1];
    }
    block_sum2(a, b, out);
}

constexpr int kMoveLanes = 64;

// Whether the previous round (its kMoveLanes counters; none for the first
// round of a batch) moved nothing: then this round and every later one of
// the batch would leave the labels unchanged, and is skipped.  Lane l reads
// counter l and the wave votes, so every lane of the wave must be active.
static_assert(kMoveLanes == kWave, "one move counter per lane");
__device__ __forceinline__ bool no_moves(const unsigned long long* __restrict__ prev) {
    if (!prev) return false;
    return __ballot(prev[threadIdx.x & (kWave - 1)] != 0ull) == 0ull;
}

// Label weights of the entries [e, e1) in chunks of U: the U column and
// weight loads, then the U label loads, are issued together; the additions
// keep entry order.  Leaves e at the first entry of an incomplete chunk.
template <int U>
__device__ __forceinline__ void gain_chunk(const GraphDev& g, const uint8_t* __restrict__ z, int64_t& e,
                                           int64_t e1, double (*cnt)[kRefineBlock], double& wdeg) {
    for (; e + U <= e1; e += U) {
        int32_t c[U];
        double w[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            c[u] = g.col[e + u];
            w[u] = g.w ? g.w[e + u] : 1.0;
        }
        uint8_t l[U];
#pragma unroll
        for (int u = 0; u < U; ++u) l[u] = z[c[u]];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            cnt[l[u]][threadIdx.x] += w[u];
            wdeg += fabs(w[u]);
        }
    }
}

// A vertex's byte of `target` holds its best label (below 16) and this mark:
// its label or a neighbour's changed since its gain was taken.
constexpr int kStale = 0x80;

// cosd[d] = cos(2 pi d / K).  Gain of moving i from a to b:
// 2 sum_k c_k (cosd[(a-k) mod K] - cosd[(b-k) mod K]).  first: every vertex.
template <int KM>
__global__ __launch_bounds__(kRefineBlock) void k_gain(GraphDev g, int K, const uint8_t* __restrict__ z,
                                                 const double* __restrict__ cosd,
                                                 double* __restrict__ gain, uint8_t* __restrict__ target, bool first,
                                                 const unsigned long long* __restrict__ prev,
                                                 const int* __restrict__ flag) {
    __shared__ double cnt[KM][kRefineBlock];   // KM >= K rows
    const int64_t i = blockIdx.x * (int64_t)kRefineBlock + threadIdx.x;
    if (no_moves(prev) || *flag || i >= g.n) return;   // the vote first, with every lane active
    if (!first && !(target[i] & kStale)) return;
    for (int k = 0; k < K; ++k) cnt[k][threadIdx.x] = 0.0;
    double wdeg = 0.0;
    int64_t e = g.row_ptr[i];
    const int64_t e1 = g.row_ptr[i + 1];
    // eight, then four entries' loads in flight at a time; the sums stay in
    // entry order
    gain_chunk<8>(g, z, e, e1, cnt, wdeg);
    gain_chunk<4>(g, z, e, e1, cnt, wdeg);
    for (; e < e1; ++e) {
        const double w = g.w ? g.w[e] : 1.0;
        cnt[z[g.col[e]]][threadIdx.x] += w;
        wdeg += fabs(w);
    }
    const int a = z[i];
    double best = -INFINITY;
    int bl = a;
    for (int b = 0; b < K; ++b) {
        if (b == a) continue;
        double d = 0.0;
        for (int k = 0; k < K; ++k) {
            const int da = a - k + (a < k ? K : 0), db = b - k + (b < k ? K : 0);
            d += cnt[k][threadIdx.x] * (cosd[da] - cosd[db]);
        }
        d *= 2.0;
        if (d > best) {
            best = d;
            bl = b;
        }
    }
    const bool cand = best > 1e-12 * wdeg;
    gain[i] = cand ? best : 0.0;
    target[i] = (uint8_t)(cand ? bl : a);
}

// Rows by groups of sixteen lanes: a wave takes kRowsPerWave = 16 vertices,
// lane l looks after vertex l % 16, and in trip q of four the group l / 16
// reads the entries of vertex 4 q + l / 16, one a lane.  The columns of all
// four trips are in flight together, then whatever they point at.  A thread a
// vertex instead reads its row entry by entry, 64 rows apart in memory across
// the wave (24 rounds as above: gains 160 us, moves 177; with sixteen entries
// of a row in flight 197 and 148).
constexpr int kRowsPerWave = 16;

struct WaveRows {
    int64_t i;            // this lane's vertex
    bool in;
    int64_t e0, e1;       // its entries (read_rows)
};

__device__ __forceinline__ WaveRows wave_rows(const GraphDev& g) {
    const int64_t wave = blockIdx.x * (int64_t)(kRefineBlock / kWave) + threadIdx.x / kWave;
    WaveRows r;
    r.i = wave * kRowsPerWave + (threadIdx.x & (kRowsPerWave - 1));
    r.in = r.i < g.n;
    r.e0 = r.e1 = 0;
    return r;
}
__device__ __forceinline__ void read_rows(const GraphDev& g, WaveRows& r) {
    if (r.in) {
        r.e0 = g.row_ptr[r.i];
        r.e1 = g.row_ptr[r.i + 1];
    }
}

// Unit weights, K <= 4: label counts by ballots (whole numbers, so the FP64
// sums of the general kernel are the same).
__global__ __launch_bounds__(kRefineBlock) void k_gain_unit(GraphDev g, int K, const uint8_t* __restrict__ z,
                                                      const double* __restrict__ cosd,
                                                      double* __restrict__ gain, uint8_t* __restrict__ target,
                                                      bool first, const unsigned long long* __restrict__ prev,
                                                      const int* __restrict__ flag) {
    __shared__ double ctab[4];
    if ((int)threadIdx.x < K) ctab[threadIdx.x] = cosd[threadIdx.x];
    __syncthreads();
    const int lane = threadIdx.x & (kWave - 1), grp = lane / kRowsPerWave, sub = lane & (kRowsPerWave - 1);
    const int bad = *flag;
    WaveRows r = wave_rows(g);
    const bool stale = r.in && (first || (target[r.i] & kStale));
    const int a = r.in ? z[r.i] : 0;
    if (no_moves(prev) || bad || __ballot(stale) == 0ull) return;   // uniform over the wave
    read_rows(g, r);
    int64_t e[4], e1[4];
    int32_t c[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        e[q] = __shfl(r.e0, 4 * q + grp, kWave) + sub;
        const int64_t end = __shfl(r.e1, 4 * q + grp, kWave);   // every lane takes part in a shuffle
        e1[q] = __shfl((int)stale, 4 * q + grp, kWave) ? end : 0;
        c[q] = e[q] < e1[q] ? g.col[e[q]] : -1;
    }
    int cnt[4] = {0, 0, 0, 0};
    bool more = true;
    while (more) {        // once, unless a row has more than sixteen entries
        int l[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) l[q] = c[q] >= 0 ? z[c[q]] : -1;
        more = false;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const unsigned long long b = __ballot(l[q] == k);
                if (sub / 4 == q) cnt[k] += __popcll((b >> (kRowsPerWave * (sub & 3))) & 0xffffull);
            }
            e[q] += kRowsPerWave;
            c[q] = e[q] < e1[q] ? g.col[e[q]] : -1;
            more |= __ballot(c[q] >= 0) != 0ull;
        }
    }
    if (!stale || grp != 0) return;
    double best = -INFINITY;
    int bl = a;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        if (b >= K || b == a) continue;
        double d = 0.0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (k >= K) break;
            const int da = a - k + (a < k ? K : 0), db = b - k + (b < k ? K : 0);
            d += (double)cnt[k] * (ctab[da] - ctab[db]);
        }
        d *= 2.0;
        if (d > best) {
            best = d;
            bl = b;
        }
    }
    const bool cand = best > 1e-12 * (double)(r.e1 - r.e0);
    gain[r.i] = cand ? best : 0.0;
    target[r.i] = (uint8_t)(cand ? bl : a);
}

// The marks: several movers may mark one vertex in the same launch; its label
// bits are constant here, so all of them store the same byte.
__global__ __launch_bounds__(kRefineBlock) void k_move(GraphDev g, uint8_t* __restrict__ z,
                                                 const double* __restrict__ gain, uint8_t* target,
                                                 unsigned long long* __restrict__ moves,
                                                 const unsigned long long* __restrict__ prev,
                                                 const int* __restrict__ flag) {
    const int lane = threadIdx.x & (kWave - 1), grp = lane / kRowsPerWave, sub = lane & (kRowsPerWave - 1);
    const int bad = *flag;
    WaveRows r = wave_rows(g);
    const double mine = r.in ? gain[r.i] : 0.0;
    if (no_moves(prev) || bad) return;   // uniform over the grid
    unsigned lost = 0;                   // bit v: a neighbour beats vertex v of the wave
    const unsigned cand = (unsigned)__ballot(mine > 0.0) & 0xffffu;
    if (cand) {
        read_rows(g, r);
        int64_t e[4], e1[4];
        int32_t c[4];
        double gi[4];
        int ii[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int v = 4 * q + grp;
            gi[q] = __shfl(mine, v, kWave);
            ii[q] = (int)__shfl(r.i, v, kWave);
            e[q] = __shfl(r.e0, v, kWave) + sub;
            const int64_t end = __shfl(r.e1, v, kWave);
            e1[q] = gi[q] > 0.0 ? end : 0;
            c[q] = e[q] < e1[q] ? g.col[e[q]] : -1;
        }
        bool more = true;
        while (more) {
            double gj[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) gj[q] = c[q] >= 0 ? gain[c[q]] : 0.0;
            more = false;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const bool beaten = gj[q] > 0.0 && (gj[q] > gi[q] || (gj[q] == gi[q] && c[q] < ii[q]));
                const unsigned long long b = __ballot(beaten);
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if ((b >> (kRowsPerWave * v)) & 0xffffull) lost |= 1u << (4 * q + v);
                e[q] += kRowsPerWave;
                c[q] = e[q] < e1[q] ? g.col[e[q]] : -1;
                more |= __ballot(c[q] >= 0) != 0ull;
            }
        }
    }
    const unsigned wins = cand & ~lost;
    if (wins) {
        // no neighbour of a mover moves, so nobody marks a mover
        if (grp == 0 && ((wins >> sub) & 1u)) {
            const uint8_t t = target[r.i] & (kStale - 1);
            z[r.i] = t;
            target[r.i] = t | kStale;
        }
        int64_t e[4], e1[4];
        bool more = false;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int v = 4 * q + grp;
            e[q] = __shfl(r.e0, v, kWave) + sub;
            const int64_t end = __shfl(r.e1, v, kWave);
            e1[q] = (wins >> v) & 1u ? end : 0;
            more |= __ballot(e[q] < e1[q]) != 0ull;
        }
        while (more) {
            int32_t c[4];
            uint8_t t[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) c[q] = e[q] < e1[q] ? g.col[e[q]] : -1;
#pragma unroll
            for (int q = 0; q < 4; ++q) t[q] = c[q] >= 0 ? target[c[q]] : 0;
            more = false;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (c[q] >= 0) target[c[q]] = t[q] | kStale;
                e[q] += kRowsPerWave;
                more |= __ballot(e[q] < e1[q]) != 0ull;
            }
        }
    }
    // the block's count into one of kMoveLanes counters (block index mod
    // kMoveLanes), so that same-address atomics stay few
    __shared__ unsigned int wm[kRefineBlock / kWave];
    if (lane == 0) wm[threadIdx.x / kWave] = (unsigned)__popc(wins);
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long b = 0;
        for (int w = 0; w < kRefineBlock / kWave; ++w) b += wm[w];
        if (b) atomicAdd(&moves[blockIdx.x % kMoveLanes], b);
    }
}

constexpr int kMaxCheck = 64;

// What the host reads back, in one copy: the checks' verdict, an objective and
// the move counters of the rounds of a batch.
struct GraphReport {
    int flag;
    int pad;
    double out[2];
    alignas(256) unsigned long long moves[kMaxCheck * kMoveLanes];
};
constexpr size_t kReportHead = offsetof(GraphReport, moves);

struct GraphScratch {
    GraphReport* rep;     // moves only for the local search
    double* partial;
    double* table;        // sqd[K] then cosd[K]
    double* gain;
    uint8_t* target;
};

struct HostScratch {
    GraphReport* rep;
    double* table;                // [2 * LRQO_MAX_K]
};

lrqo_status reserve_graph(DeviceCtx* ctx, int64_t n, bool refine, GraphScratch& s, HostScratch& h) {
    const int64_t blocks = (n + kBlock - 1) / kBlock;
    CarveSize cs;
    cs.add<char>(refine ? sizeof(GraphReport) : kReportHead);
    cs.add<double>(2 * blocks);
    cs.add<double>(2 * LRQO_MAX_K);
    if (refine) {
        cs.add<double>(n);
        cs.add<uint8_t>(n);
    }
    CarveSize hs;
    hs.add<GraphReport>(1);
    hs.add<double>(2 * LRQO_MAX_K);
    LRQO_TRY(reserve_arena(ctx, cs.bytes));
    LRQO_TRY(reserve_host(ctx, hs.bytes));
    Carve cv(ctx->arena);
    s.rep = reinterpret_cast<GraphReport*>(cv.take<char>(refine ? sizeof(GraphReport) : kReportHead));
    s.partial = cv.take<double>(2 * blocks);
    s.table = cv.take<double>(2 * LRQO_MAX_K);
    s.gain = refine ? cv.take<double>(n) : nullptr;
    s.target = refine ? cv.take<uint8_t>(n) : nullptr;
    Carve hv(ctx->host);
    h.rep = hv.take<GraphReport>(1);
    h.table = hv.take<double>(2 * LRQO_MAX_K);
    return LRQO_OK;
}

lrqo_status upload_tables(int K, const GraphScratch& s, double* h_tab, hipStream_t st) {
    for (int d = 0; d < K; ++d) {
        const double a = 6.283185307179586476925286766559 * (double)d / (double)K;
        const double c = std::cos(a), sn = std::sin(a);
        // |1 - omega^d|^2 = (1 - cos)^2 + sin^2
        h_tab[d] = (1.0 - c) * (1.0 - c) + sn * sn;
        h_tab[LRQO_MAX_K + d] = c;
    }
    if (K == 2 || K == 3 || K == 4) {
        // these values are the integers 0..4 and cos in {1, 0, -1/2, -1}
        for (int d = 0; d < K; ++d) {
            h_tab[d] = std::round(h_tab[d]);
            h_tab[LRQO_MAX_K + d] = std::round(2.0 * h_tab[LRQO_MAX_K + d]) / 2.0;
        }
    }
    LRQO_HIP(hipMemcpyAsync(s.table, h_tab, sizeof(double) * 2 * LRQO_MAX_K, hipMemcpyHostToDevice, st));
    return LRQO_OK;
}

// Queues the objective of z into the report (skipped when a check failed).
lrqo_status launch_objective(const GraphDev& gd, int K, const uint8_t* z, const GraphScratch& s, hipStream_t st) {
    const int64_t blocks = (gd.n + kBlock - 1) / kBlock;
    hipLaunchKernelGGL(k_objective, dim3((unsigned)blocks), dim3(kBlock), 0, st, gd, K, z, s.table, s.partial,
                       &s.rep->flag);
    hipLaunchKernelGGL(k_sum2, dim3(1), dim3(kBlock), 0, st, s.partial, blocks, s.rep->out);
    LRQO_HIP(hipGetLastError());
    return LRQO_OK;
}

// Queues the layout checks: *d_flag is cleared, then holds what they found.
lrqo_status launch_checks(const GraphDev& gd, int K, const uint8_t* z, int* d_flag, int* h_flag, hipStream_t st) {
    const unsigned blocks = (unsigned)((gd.n + kBlock - 1) / kBlock);
    *h_flag = 0;
    LRQO_HIP(hipMemcpyAsync(d_flag, h_flag, sizeof(int), hipMemcpyHostToDevice, st));
    hipLaunchKernelGGL(k_check_ptr, dim3(blocks), dim3(kBlock), 0, st, gd, d_flag);
    hipLaunchKernelGGL(k_check_rows, dim3(blocks), dim3(kBlock), 0, st, gd, K, z, d_flag);
    LRQO_HIP(hipGetLastError());
    return LRQO_OK;
}

lrqo_status read_checks(int flag) {
    if (flag & kBadPtr)
        return fail(LRQO_EINVAL, "row_ptr is not a CSR row pointer (row_ptr[0] = 0, non-decreasing, row_ptr[n] = nnz)");
    if (flag & kBadCol) return fail(LRQO_EINVAL, "a column index is out of range or a self loop");
    if (flag & kBadWeight) return fail(LRQO_EINVAL, "a weight is not finite");
    if (flag & kBadLabel) return fail(LRQO_EINVAL, "a label is not below K");
    return LRQO_OK;
}

// The report (its first `bytes`) to the host.
lrqo_status read_report(const GraphScratch& s, const HostScratch& h, size_t bytes, hipStream_t st) {
    LRQO_HIP(hipMemcpyAsync(h.rep, s.rep, bytes, hipMemcpyDeviceToHost, st));
    LRQO_HIP(hipStreamSynchronize(st));
    return LRQO_OK;
}

}  // namespace

lrqo_status check_graph_args(const lrqo_graph* g) {
    if (!g) return fail(LRQO_EINVAL, "null graph");
    if (!g->row_ptr) return fail(LRQO_EINVAL, "null row_ptr");
    if (g->nnz > 0 && !g->col) return fail(LRQO_EINVAL, "null col with nnz > 0");
    if (g->n < 1 || g->n > 0x7fffffffLL) return fail(LRQO_EINVAL, "n must be in [1, 2^31 - 1]");
    if (g->nnz < 0) return fail(LRQO_EINVAL, "nnz must be >= 0");
    if (!is_device_pointer(g->row_ptr)) return fail(LRQO_EINVAL, "row_ptr is not device memory");
    if (g->nnz > 0 && !is_device_pointer(g->col)) return fail(LRQO_EINVAL, "col is not device memory");
    if (g->w && !is_device_pointer(g->w)) return fail(LRQO_EINVAL, "w is not device memory");
    return LRQO_OK;
}

lrqo_status validate_graph(const lrqo_graph* g, int K, const uint8_t* z, int* d_flag, int* h_flag,
                           hipStream_t st) {
    const GraphDev gd{g->row_ptr, g->col, g->w, g->n, g->nnz};
    LRQO_TRY(launch_checks(gd, K, z, d_flag, h_flag, st));
    LRQO_HIP(hipMemcpyAsync(h_flag, d_flag, sizeof(int), hipMemcpyDeviceToHost, st));
    LRQO_HIP(hipStreamSynchronize(st));
    return read_checks(*h_flag);
}

}  // namespace lrqo

extern "C" {

lrqo_status lrqo_graph_objective(const lrqo_graph* g, int32_t K, const uint8_t* z, double* quad,
                                 double* cut) {
    using namespace lrqo;
    clear_error();
    LRQO_TRY(check_graph_args(g));
    if (!z || !quad || !cut) return fail(LRQO_EINVAL, "null pointer argument");
    if (K < 2 || K > LRQO_MAX_K) return fail(LRQO_EINVAL, "K must be in [2, 255]");
    if (!is_device_pointer(z)) return fail(LRQO_EINVAL, "z is not device memory");
    DeviceCtx* ctx = device_ctx();
    if (!ctx) return LRQO_EDEVICE;
    std::lock_guard<std::mutex> lk(ctx->mu);
    const hipStream_t st = current_stream();
    GraphScratch s{};
    HostScratch h{};
    LRQO_TRY(reserve_graph(ctx, g->n, false, s, h));
    const GraphDev gd{g->row_ptr, g->col, g->w, g->n, g->nnz};
    LRQO_TRY(launch_checks(gd, K, z, &s.rep->flag, &h.rep->flag, st));
    LRQO_TRY(upload_tables(K, s, h.table, st));
    LRQO_TRY(launch_objective(gd, K, z, s, st));
    LRQO_TRY(read_report(s, h, kReportHead, st));
    LRQO_TRY(read_checks(h.rep->flag));
    *quad = 0.5 * h.rep->out[0];          // every edge was seen from both of its ends
    *cut = 0.5 * h.rep->out[1];
    return LRQO_OK;
}

lrqo_status lrqo_refine_greedy(const lrqo_graph* g, int32_t K, uint8_t* z, const lrqo_refine_options* opt,
                               lrqo_refine_result* res) {
    using namespace lrqo;
    clear_error();
    LRQO_TRY(check_graph_args(g));
    if (!z) return fail(LRQO_EINVAL, "null pointer argument");
    if (K < 2 || K > kMaxKRefine) return fail(LRQO_EINVAL, "K must be in [2, 16] for the local search");
    lrqo_refine_options o{};
    if (opt) o = *opt;
    if (o.max_rounds < 0) return fail(LRQO_EINVAL, "max_rounds must be >= 0");
    if (o.check_every < 0 || o.check_every > kMaxCheck) return fail(LRQO_EINVAL, "check_every must be in [0, 64]");
    const int64_t max_rounds = o.max_rounds ? o.max_rounds : 1000000;
    const int chunk = o.check_every ? o.check_every : 8;
    if (!is_device_pointer(z)) return fail(LRQO_EINVAL, "z is not device memory");
    DeviceCtx* ctx = device_ctx();
    if (!ctx) return LRQO_EDEVICE;
    std::lock_guard<std::mutex> lk(ctx->mu);
    const hipStream_t st = current_stream();
    GraphScratch s{};
    HostScratch h{};
    LRQO_TRY(reserve_graph(ctx, g->n, true, s, h));
    const GraphDev gd{g->row_ptr, g->col, g->w, g->n, g->nnz};
    LRQO_TRY(launch_checks(gd, K, z, &s.rep->flag, &h.rep->flag, st));
    LRQO_TRY(upload_tables(K, s, h.table, st));
    LRQO_TRY(launch_objective(gd, K, z, s, st));

    lrqo_refine_result r{};
    constexpr int64_t kRowsPerBlock = kRefineBlock / kWave * kRowsPerWave;
    const unsigned blocks = (unsigned)((gd.n + kRefineBlock - 1) / kRefineBlock);
    const unsigned row_blocks = (unsigned)((gd.n + kRowsPerBlock - 1) / kRowsPerBlock);
    const double* cosd = s.table + LRQO_MAX_K;
    const int* flag = &s.rep->flag;
    int64_t rounds = 0, moves = 0, launched = 0;
    bool converged = false;
    float total_ms = 0.0f;
    while (!converged && rounds < max_rounds) {
        const int todo = (int)std::min<int64_t>(chunk, max_rounds - rounds);
        LRQO_HIP(hipMemsetAsync(s.rep->moves, 0, sizeof(unsigned long long) * todo * kMoveLanes, st));
        LRQO_HIP(hipEventRecord(ctx->ev_start, st));
        for (int t = 0; t < todo; ++t) {
            // the batch runs only after rounds that all moved something
            const unsigned long long* prev = t ? s.rep->moves + (size_t)(t - 1) * kMoveLanes : nullptr;
            const bool first = launched == 0 && t == 0;
            if (K <= 4 && !g->w)
                hipLaunchKernelGGL(k_gain_unit, dim3(row_blocks), dim3(kRefineBlock), 0, st, gd, K, z, cosd, s.gain,
                                   s.target, first, prev, flag);
            else if (K <= 4)
                hipLaunchKernelGGL(k_gain<4>, dim3(blocks), dim3(kRefineBlock), 0, st, gd, K, z, cosd, s.gain,
                                   s.target, first, prev, flag);
            else
                hipLaunchKernelGGL(k_gain<kMaxKRefine>, dim3(blocks), dim3(kRefineBlock), 0, st, gd, K, z, cosd,
                                   s.gain, s.target, first, prev, flag);
            hipLaunchKernelGGL(k_move, dim3(row_blocks), dim3(kRefineBlock), 0, st, gd, z, s.gain, s.target,
                               s.rep->moves + (size_t)t * kMoveLanes, prev, flag);
        }
        LRQO_HIP(hipGetLastError());
        LRQO_HIP(hipEventRecord(ctx->ev_stop, st));
        const bool head = launched == 0;
        launched += todo;
        LRQO_TRY(read_report(s, h, kReportHead + sizeof(unsigned long long) * todo * kMoveLanes, st));
        if (head) {
            LRQO_TRY(read_checks(h.rep->flag));
            r.quad_before = 0.5 * h.rep->out[0];
            r.cut_before = 0.5 * h.rep->out[1];
        }
        float ms = 0.0f;
        LRQO_HIP(hipEventElapsedTime(&ms, ctx->ev_start, ctx->ev_stop));
        total_ms += ms;
        // a round without moves leaves the labels as they were, and so do all after it
        for (int t = 0; t < todo; ++t) {
            unsigned long long m = 0;
            for (int l = 0; l < kMoveLanes; ++l) m += h.rep->moves[(size_t)t * kMoveLanes + l];
            if (m == 0) {
                converged = true;
                break;
            }
            ++rounds;
            moves += (int64_t)m;
        }
    }
    LRQO_TRY(launch_objective(gd, K, z, s, st));
    LRQO_TRY(read_report(s, h, kReportHead, st));
    r.quad_after = 0.5 * h.rep->out[0];
    r.cut_after = 0.5 * h.rep->out[1];
    r.moves = moves;
    r.rounds = (int32_t)rounds;
    r.converged = converged ? 1 : 0;
    r.device_ms = total_ms;
    r.launched = (int32_t)launched;
    if (res) *res = r;
    return LRQO_OK;
}

}  // extern "C"
