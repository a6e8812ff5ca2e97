// Exact rank-1 maximisation by the phase sweep (Sec. 2.5, Alg. 1,
// Thm. rank1): max |z^H q|^2 over z in A_K^n.
//
// Every coordinate changes its label once as the auxiliary angle phi sweeps
// (-pi/K, pi/K]: at phi_i = (2 pi/K)(1/2 + floor(x_i) - x_i), x_i =
// K arg(q_i)/(2 pi).  Starting from k_i = floor(x_i) mod K (the assignment
// at phi = -pi/K), the n+1 cells of the sweep are the prefixes of the
// boundary points in sorted order, and s = sum_i conj(q_i) omega^k_i moves
// by d_i = conj(q_i)(omega^(k_i+1) - omega^k_i) at each of them, so the
// objective of cell l is |s_0 + d_(1) + ... + d_(l)|^2.
//
// Kernels:
//   k_r1_prep     per coordinate: phi (same FP64 expression as Alg. 1), its
//                 exact sortable key and 32-bit image, k_0; per tile: counts
//                 of the images' leading bits (the buckets), partial of s_0,
//                 finiteness
// Bucket form (n up to 2^24, points spread over the range): six launches and
// one wait in all.
//   k_rb_scan     each tile's offset within each bucket, the bucket sizes
//   k_rb_scatter  (image, coordinate, k_0) into the buckets, any order inside
//   k_rb_sort     a block per bucket: its points sorted in LDS by (key,
//                 coordinate), a total order, so the result is that of a
//                 stable sort; d gathered into sorted order, bucket sums
//   k_rb_cells    per bucket: s at its first point, the running s, best cell
//   k_r1_labels   best cell over the buckets; labels in coordinate order: k_0
//                 advanced by one where (key, coordinate) is at or below that
//                 of the cell's last point; block partials of z^H q (added on
//                 the host)
// A bucket of more than kRbCap points, or a run of more than 16 equal images
// with differing keys, raises a flag, and the call goes on with the general
// form from the prep's results.
// General form:
//   radix sort    stable (sort.hip), by the 32-bit fixed-point image of phi
//                 (four passes; it never reverses the order of two points),
//                 so equal images keep coordinate order
//   k_r1_fixup    runs of equal images whose exact keys differ (rare: points
//                 closer than 2^-32 of the range) are put in (key,
//                 coordinate) order by insertion; a run longer than 16 with
//                 differing keys makes the host sort the exact 64-bit keys
//                 instead (eight passes; digits that are the same in every
//                 key, found by k_r1_orand, skip theirs) and run what follows
//                 again, so the order is always that of (key, coordinate)
//   k_r1_gather   per span of sorted positions: gathers d into sorted order
//                 and sums the span; k_rb_cells and k_r1_labels then take
//                 the spans as the buckets
// All sums run in a fixed order (shuffle trees and block scans of fixed
// shape), so a run is reproducible.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "lrqo_device.h"
#include "lrqo_runtime.h"
#include "sort.h"

namespace lrqo {

namespace {

constexpr int kBlock = 256;
constexpr double kPi = 3.141592653589793238462643383279502884;

__device__ __forceinline__ unsigned long long order_key(double v) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}

// A 32-bit image of phi in (-pi/K, pi/K] that never reverses the order of
// two values: (phi K/(2 pi) + 1/2) 2^32, truncated and clamped; every step
// is non-decreasing in phi.
__device__ __forceinline__ uint32_t fixed_key(double phi, int K) {
    double u = fma(phi, (double)K / (2.0 * kPi), 0.5) * 4294967296.0;
    u = u > 0.0 ? u : 0.0;   // also maps a NaN to 0 (reported separately)
    return u >= 4294967295.0 ? 0xFFFFFFFFu : (uint32_t)u;
}

__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }

// conj(q) * w
__device__ __forceinline__ double2 cconj_mul(double2 q, double2 w) {
    return make_double2(q.x * w.x + q.y * w.y, q.x * w.y - q.y * w.x);
}

__device__ __forceinline__ double2 shfl_xor_c(double2 v, int m) {
    return make_double2(__shfl_xor(v.x, m, kWave), __shfl_xor(v.y, m, kWave));
}

__device__ __forceinline__ double2 shfl_up_c(double2 v, int off) {
    return make_double2(__shfl_up(v.x, off, kWave), __shfl_up(v.y, off, kWave));
}

// Fixed-order block sum of a complex value per thread: a shuffle tree in
// each wave, then the waves' sums in wave order.  Every thread gets it.
template <int BT = kBlock>
__device__ __forceinline__ double2 block_sum_c(double2 v) {
    __shared__ double2 ws[BT / kWave];
#pragma unroll
    for (int m = kWave / 2; m > 0; m >>= 1) v = cadd(v, shfl_xor_c(v, m));
    if ((threadIdx.x & (kWave - 1)) == 0) ws[threadIdx.x / kWave] = v;
    __syncthreads();
    double2 r = ws[0];
    for (int w = 1; w < BT / kWave; ++w) r = cadd(r, ws[w]);
    __syncthreads();
    return r;
}

// init + the sum of the values of the threads before this one (fixed
// order: a shuffle scan in each wave, the lower waves' totals before it).
template <int BT = kBlock>
__device__ __forceinline__ double2 block_excl_scan_c(double2 v, double2 init) {
    __shared__ double2 ws[BT / kWave];
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    double2 incl = v;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const double2 y = shfl_up_c(incl, off);
        if (lane >= off) incl = cadd(y, incl);
    }
    if (lane == kWave - 1) ws[w] = incl;
    const double2 below = shfl_up_c(incl, 1);
    __syncthreads();
    double2 r = init;
    for (int u = 0; u < w; ++u) r = cadd(r, ws[u]);
    if (lane > 0) r = cadd(r, below);
    __syncthreads();
    return r;
}

// The boundary point phi of q_i and k_0: the expressions of Alg. 1, rounded
// step by step as written.
__device__ __forceinline__ double sweep_point(double2 q, int K, int& k) {
    const double theta = atan2(q.y, q.x);
    const double x = __ddiv_rn(__dmul_rn((double)K, theta), 2.0 * kPi);
    const double fl = floor(x);
    k = (int)fmod(fl, (double)K);
    k += k < 0 ? K : 0;
    return __dmul_rn(__ddiv_rn(2.0 * kPi, (double)K), __dsub_rn(__dadd_rn(0.5, fl), x));
}

// The step of s at the boundary point of q_i: d_i.
__device__ __forceinline__ double2 sweep_step(double2 q, int k, int K, const double2* roots) {
    const int k1 = k + 1 == K ? 0 : k + 1;
    const double2 a = roots[k], b = roots[k1];
    return cconj_mul(q, make_double2(b.x - a.x, b.y - a.y));
}

// ------------------------------------------------------------ bucket form
// What bounds the sweep is not the arithmetic (17 bytes and one atan2 a
// coordinate) but how often the pairs cross memory: the general form moves
// them through four radix passes (twelve launches) and gathers the result
// once more.  The images are spread evenly for vectors in general position,
// so one split by their leading bits leaves buckets that a block sorts in
// LDS, and the same block gathers d.  Complex normal q, K = 3, a call: 228 ->
// 119 us at n = 10^6 (device work 187 -> 85 us: prep 12, scan 5, scatter 12,
// sort with the gather 29, cells 11, labels 9), 166 -> 74 us at n = 100,
// 542 -> 284 us at n = 4 10^6.  A real q (two points only) leaves this form
// after the scan and takes the general one from the prep's results: 223 ->
// 221 us at n = 10^6.
constexpr int kRbThreads = 512;
constexpr int kRbTiles = 512;               // blocks of the passes over the coordinates: two per CU
// Points of one bucket: 64 KB of LDS, two blocks per CU, four times the mean,
// so that uneven points still fit.  Half of it (four blocks per CU, buckets of
// half the size) took 92 us of device work for 85.
constexpr int kRbCap = 8192;
constexpr int kRbBins = 2048;               // second-level bins of a bucket
constexpr int kRbBin = 32;                  // points of one bin sorted by insertion
constexpr int kRunMax = 16;                 // longest run of equal images sorted in place
// Coordinate index and k_0 share 32 bits.  The form still leads at this size:
// 1,731 -> 1,200 us at n = 1.5 10^7.
constexpr int64_t kRbMaxN = 1ll << 24;

struct Best {
    double f;
    int64_t cell;
    unsigned long long key;   // key of the cell's last boundary point (cell >= 1)
    uint32_t coord;           // and its coordinate
    int32_t pad;
};

struct RbOut {                // what the host reads; the partials of z^H q follow
    Best best;
    int32_t flag[4];
};
static_assert(sizeof(RbOut) % sizeof(double2) == 0, "the partials follow");

struct RbDev {
    const double2* q;
    const double2* roots;
    unsigned long long* keys;
    uint32_t* img;
    uint8_t* k0;
    uint32_t* hist;           // [tiles][nb]: counts, then offsets within the bucket
    uint32_t* total;          // [nb]
    uint32_t* start;          // [nb]
    unsigned long long* ent;  // image << 32 | coordinate << 8 | k_0, by bucket
    uint32_t* order;          // coordinates in sorted order
    double2* d_sorted;
    double2* part;            // [tiles] partials of s_0
    double2* bsum;            // [nb]
    Best* bbest;              // [nb]
    RbOut* out;
    double2* lpart;           // [tiles]
    uint8_t* z;
    int* flag;                // [0] non-finite q, [1] a bucket too large, [2], [3] a long run with differing keys
                              // (bucket form, general form)
    int64_t n;
    int64_t per;              // coordinates per tile
    int64_t span;             // general form: sorted positions per span (0: buckets)
    int K, lb, nb, tiles;     // nb = 2^lb buckets (0: general form only), or the spans
};

__device__ __forceinline__ uint32_t rb_bucket(uint32_t img, int lb) { return lb ? img >> (32 - lb) : 0u; }

__global__ __launch_bounds__(kRbThreads) void k_r1_prep(RbDev p) {
    extern __shared__ uint32_t cnt[];       // [nb]
    for (int b = threadIdx.x; b < p.nb; b += kRbThreads) cnt[b] = 0u;
    __syncthreads();
    const int64_t lo = blockIdx.x * p.per, hi = min(p.n, lo + p.per);
    double2 c0 = make_double2(0.0, 0.0);
    for (int64_t i = lo + threadIdx.x; i < hi; i += kRbThreads) {
        const double2 q = p.q[i];
        if (!isfinite(q.x) || !isfinite(q.y)) atomicOr(p.flag, 1);
        int k;
        const double phi = sweep_point(q, p.K, k);
        const uint32_t img = fixed_key(phi, p.K);
        p.keys[i] = order_key(phi);
        p.img[i] = img;
        p.k0[i] = (uint8_t)k;
        c0 = cadd(c0, cconj_mul(q, p.roots[k]));
        if (p.nb) atomicAdd(&cnt[rb_bucket(img, p.lb)], 1u);
    }
    const double2 s = block_sum_c<kRbThreads>(c0);   // synchronises the block
    if (threadIdx.x == 0) p.part[blockIdx.x] = s;
    for (int b = threadIdx.x; b < p.nb; b += kRbThreads) p.hist[(size_t)blockIdx.x * p.nb + b] = cnt[b];
}

// Sixteen buckets per block, sixteen segments of tiles each: the segments'
// sums, their prefix, then the tiles' prefixes written over the counts.
constexpr int kRbSeg = 16;

__global__ __launch_bounds__(kRbSeg * kRbSeg) void k_rb_scan(RbDev p) {
    __shared__ uint32_t seg[kRbSeg][kRbSeg + 1];
    const int bl = threadIdx.x % kRbSeg, sg = threadIdx.x / kRbSeg;
    const int b = blockIdx.x * kRbSeg + bl;
    const int len = (p.tiles + kRbSeg - 1) / kRbSeg;
    const int t0 = sg * len, t1 = min(p.tiles, t0 + len);
    constexpr int U = kRbTiles / kRbSeg;    // tiles of a segment at most
    uint32_t v[U];
    uint32_t sum = 0u;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        v[u] = (b < p.nb && t0 + u < t1) ? p.hist[(size_t)(t0 + u) * p.nb + b] : 0u;
        sum += v[u];
    }
    seg[sg][bl] = sum;
    __syncthreads();
    uint32_t run = 0u;
    for (int s = 0; s < sg; ++s) run += seg[s][bl];
    if (b < p.nb) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (t0 + u < t1) p.hist[(size_t)(t0 + u) * p.nb + b] = run;
            run += v[u];
        }
        if (sg == kRbSeg - 1) {
            p.total[b] = run;
            if (run > (uint32_t)kRbCap) p.flag[1] = 1;   // every writer stores the same value
        }
    }
}

// Exclusive prefix over the block of one count per thread.
__device__ __forceinline__ uint32_t rb_excl_scan(uint32_t x) {
    __shared__ uint32_t ws[kRbThreads / kWave];
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    uint32_t incl = x;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t y = __shfl_up(incl, off, kWave);
        if (lane >= off) incl += y;
    }
    if (lane == kWave - 1) ws[w] = incl;
    __syncthreads();
    uint32_t ex = incl - x;
    for (int v = 0; v < w; ++v) ex += ws[v];
    __syncthreads();
    return ex;
}

__global__ __launch_bounds__(kRbThreads) void k_rb_scatter(RbDev p) {
    extern __shared__ uint32_t cur[];       // [nb]: the tile's next slot in each bucket
    if (p.flag[1]) return;                  // set by an earlier kernel: the same in every thread
    const int m = (p.nb + kRbThreads - 1) / kRbThreads;
    const int b0 = min(p.nb, (int)threadIdx.x * m), b1 = min(p.nb, b0 + m);
    uint32_t sum = 0u;
    for (int b = b0; b < b1; ++b) sum += p.total[b];
    uint32_t run = rb_excl_scan(sum);
    const uint32_t* row = p.hist + (size_t)blockIdx.x * p.nb;
    for (int b = b0; b < b1; ++b) {
        if (blockIdx.x == 0) p.start[b] = run;
        cur[b] = run + row[b];
        run += p.total[b];
    }
    __syncthreads();
    const int64_t lo = blockIdx.x * p.per, hi = min(p.n, lo + p.per);
    for (int64_t i = lo + threadIdx.x; i < hi; i += kRbThreads) {
        const uint32_t img = p.img[i];
        const uint32_t pos = atomicAdd(&cur[rb_bucket(img, p.lb)], 1u);
        p.ent[pos] = ((unsigned long long)img << 32) | (unsigned long long)((uint32_t)i << 8 | p.k0[i]);
    }
}

__device__ __forceinline__ uint32_t ent_coord(unsigned long long e) { return (uint32_t)e >> 8; }

// One bin by insertion (image, then coordinate: the low word's order).
__device__ __forceinline__ void rb_sort_bin(unsigned long long* e, uint32_t cnt) {
    for (uint32_t a = 1; a < cnt; ++a) {
        const unsigned long long v = e[a];
        uint32_t b = a;
        while (b > 0 && e[b - 1] > v) {
            e[b] = e[b - 1];
            --b;
        }
        e[b] = v;
    }
}

// The whole bucket by a bitonic network (points in a few places only).
__device__ void rb_sort_network(unsigned long long* es, uint32_t cnt) {
    uint32_t m = 1;
    while (m < cnt) m <<= 1;
    for (uint32_t e = cnt + threadIdx.x; e < m; e += kRbThreads) es[e] = ~0ull;
    for (uint32_t k = 2; k <= m; k <<= 1)
        for (uint32_t j = k >> 1; j > 0; j >>= 1) {
            __syncthreads();
            for (uint32_t t = threadIdx.x; t < m / 2; t += kRbThreads) {
                const uint32_t i = 2 * t - (t & (j - 1)), l = i + j;
                const unsigned long long x = es[i], y = es[l];
                if ((x > y) == ((i & k) == 0)) {
                    es[i] = y;
                    es[l] = x;
                }
            }
        }
    __syncthreads();
}

__device__ __forceinline__ uint32_t ent_image(unsigned long long e) { return (uint32_t)(e >> 32); }

// Runs of equal images (points closer than 2^-32 of the range) at position
// e of the sorted bucket, as k_r1_fixup does it: a run of at most kRunMax is
// put in (key, coordinate) order by its first position's thread; false for an
// inside position whose key differs from its predecessor's in a longer run
// (those are never moved).
__device__ bool rb_fix_run(unsigned long long* es, uint32_t e, uint32_t cnt,
                           const unsigned long long* __restrict__ keys) {
    const uint32_t img = ent_image(es[e]);
    if (e == 0 || ent_image(es[e - 1]) != img) {
        uint32_t h = e + 1;
        while (h < cnt && ent_image(es[h]) == img && h - e <= (uint32_t)kRunMax) ++h;
        if (h - e > (uint32_t)kRunMax) return true;      // checked by its members
        for (uint32_t u = e + 1; u < h; ++u) {
            const unsigned long long v = es[u];
            const unsigned long long kv = keys[ent_coord(v)];
            uint32_t b = u;
            while (b > e) {
                const unsigned long long w = es[b - 1];
                const unsigned long long kw = keys[ent_coord(w)];
                if (kw < kv || (kw == kv && w < v)) break;
                es[b] = w;
                --b;
            }
            es[b] = v;
        }
        return true;
    }
    uint32_t lo = e, hi = e + 1;
    while (lo > 0 && ent_image(es[lo - 1]) == img && hi - lo <= (uint32_t)kRunMax) --lo;
    while (hi < cnt && ent_image(es[hi]) == img && hi - lo <= (uint32_t)kRunMax) ++hi;
    if (hi - lo <= (uint32_t)kRunMax) return true;       // its first position's thread moves it
    return keys[ent_coord(es[e])] == keys[ent_coord(es[e - 1])];
}

// A block per bucket: counting sort by the next eleven bits in LDS, each bin
// (about one point) by insertion, or the whole bucket by a network when a bin
// is large; then the gather of d in sorted order.
// The gather (16 bytes a point at random) is what bounds it: two blocks of
// eight waves per CU keep four gathers a thread in flight.
__global__ __launch_bounds__(kRbThreads) void k_rb_sort(RbDev p) {
    __shared__ unsigned long long es[kRbCap];
    __shared__ uint32_t bin[kRbBins];
    if (p.flag[1]) return;
    const int tid = threadIdx.x;
    const uint32_t s = p.start[blockIdx.x], cnt = p.total[blockIdx.x];
    for (int b = tid; b < kRbBins; b += kRbThreads) bin[b] = 0u;
    __syncthreads();
    constexpr int kShift = 32 - 11;
    static_assert(kRbBins == 1 << 11, "eleven bits");
    for (uint32_t e = tid; e < cnt; e += kRbThreads)
        atomicAdd(&bin[((uint32_t)(p.ent[s + e] >> 32) << p.lb) >> kShift], 1u);
    __syncthreads();
    constexpr int kPer = kRbBins / kRbThreads;
    uint32_t c[kPer], sum = 0u;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        c[u] = bin[tid * kPer + u];
        sum += c[u];
    }
    const uint32_t first = rb_excl_scan(sum);   // synchronises the block
    uint32_t run = first;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        bin[tid * kPer + u] = run;
        run += c[u];
    }
    __syncthreads();
    for (uint32_t e = tid; e < cnt; e += kRbThreads) {
        const unsigned long long v = p.ent[s + e];
        es[atomicAdd(&bin[((uint32_t)(v >> 32) << p.lb) >> kShift], 1u)] = v;
    }
    __syncthreads();
    run = first;
    bool large = false;
#pragma unroll
    for (int u = 0; u < kPer; ++u) large |= c[u] > (uint32_t)kRbBin;
    if (__syncthreads_or(large)) {
        rb_sort_network(es, cnt);
    } else {
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            if (c[u] > 1u) rb_sort_bin(es + run, c[u]);
            run += c[u];
        }
        __syncthreads();
    }
    bool runs = true;
    for (uint32_t e = tid; e < cnt; e += kRbThreads) {
        const uint32_t img = ent_image(es[e]);
        if ((e > 0 && ent_image(es[e - 1]) == img) || (e + 1 < cnt && ent_image(es[e + 1]) == img))
            runs &= rb_fix_run(es, e, cnt, p.keys);
    }
    if (!runs) p.flag[2] = 1;               // every writer stores the same value
    __syncthreads();
    double2 a = make_double2(0.0, 0.0);
    constexpr int U = 4;
    for (uint32_t e0 = tid; e0 < cnt; e0 += U * kRbThreads) {
        unsigned long long v[U];
        double2 q[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t e = e0 + u * kRbThreads;
            v[u] = e < cnt ? es[e] : 0ull;
            q[u] = p.q[ent_coord(v[u])];         // coordinate 0 beyond the end: n >= 1
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t e = e0 + u * kRbThreads;
            if (e >= cnt) break;
            const double2 d = sweep_step(q[u], (int)(v[u] & 0xFFu), p.K, p.roots);
            p.d_sorted[s + e] = d;
            p.order[s + e] = ent_coord(v[u]);
            a = cadd(a, d);
        }
    }
    const double2 t = block_sum_c<kRbThreads>(a);
    if (tid == 0) p.bsum[blockIdx.x] = t;
}

// ------------------------------------------------------------ general form
// OR and AND of the exact keys: one pair of partials per block.
__global__ __launch_bounds__(kBlock) void k_r1_orand(const unsigned long long* __restrict__ keys, int64_t n,
                                                     unsigned long long* __restrict__ part) {
    __shared__ unsigned long long wo[kBlock / kWave], wa[kBlock / kWave];
    unsigned long long o = 0ull, a = ~0ull;
    for (int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock) {
        o |= keys[i];
        a &= keys[i];
    }
    for (int off = kWave / 2; off > 0; off >>= 1) {
        o |= __shfl_xor(o, off, kWave);
        a &= __shfl_xor(a, off, kWave);
    }
    if ((threadIdx.x & (kWave - 1)) == 0) {
        wo[threadIdx.x / kWave] = o;
        wa[threadIdx.x / kWave] = a;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kBlock / kWave; ++w) {
            o |= wo[w];
            a &= wa[w];
        }
        part[2 * blockIdx.x] = o;
        part[2 * blockIdx.x + 1] = a;
    }
}

// Span b holds sorted positions b*span .. b*span + span-1 (bucket b of the
// kernels that follow): their d gathered into d_sorted, and its sum.
__global__ __launch_bounds__(kRbThreads) void k_r1_gather(RbDev p) {
    const int64_t lo = blockIdx.x * p.span, hi = min(p.n, lo + p.span);
    double2 a = make_double2(0.0, 0.0);
    constexpr int U = 4;
    for (int64_t e0 = lo + threadIdx.x; e0 < hi; e0 += U * kRbThreads) {
        uint32_t i[U];
        double2 d[U];
#pragma unroll
        for (int u = 0; u < U; ++u) i[u] = e0 + u * kRbThreads < hi ? p.order[e0 + u * kRbThreads] : 0u;
#pragma unroll
        for (int u = 0; u < U; ++u) d[u] = sweep_step(p.q[i[u]], p.k0[i[u]], p.K, p.roots);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t e = e0 + u * kRbThreads;
            if (e >= hi) break;
            p.d_sorted[e] = d[u];
            a = cadd(a, d[u]);
        }
    }
    const double2 t = block_sum_c<kRbThreads>(a);
    if (threadIdx.x == 0) p.bsum[blockIdx.x] = t;
}

// After the stable sort by image, position p starts a run of equal images
// or sits inside one.  A run start with a run of at most kRunMax puts it in
// (key, coordinate) order by insertion (a run of equal keys is already in
// coordinate order and costs one comparison per member).  An inside
// position whose key differs from its predecessor's, in a run longer than
// kRunMax, sets *overflow; such runs are never touched here.
__global__ __launch_bounds__(kBlock) void k_r1_fixup(const uint32_t* __restrict__ img, uint32_t* __restrict__ order,
                                                     const unsigned long long* __restrict__ keys, int64_t n,
                                                     int* __restrict__ overflow) {
    const int64_t p = blockIdx.x * (int64_t)kBlock + threadIdx.x;
    if (p >= n) return;
    const uint32_t q = img[p];
    const bool start = p == 0 || img[p - 1] != q;
    if (start) {
        if (p + 1 >= n || img[p + 1] != q) return;
        int64_t e = p + 1;
        while (e < n && img[e] == q && e - p <= kRunMax) ++e;
        if (e - p > kRunMax) return;     // long run: checked by its members
        for (int64_t a = p + 1; a < e; ++a) {
            const uint32_t v = order[a];
            const unsigned long long kv = keys[v];
            int64_t b = a;
            while (b > p) {
                const uint32_t u = order[b - 1];
                const unsigned long long ku = keys[u];
                if (ku < kv || (ku == kv && u < v)) break;
                order[b] = u;
                --b;
            }
            order[b] = v;
        }
        return;
    }
    // inside a run; order[] of a run of at most kRunMax may be changing
    // under this read, but then the length test below ends it
    if (keys[order[p]] == keys[order[p - 1]]) return;
    int64_t lo = p, hi = p + 1;
    while (lo > 0 && img[lo - 1] == q && hi - lo <= kRunMax) --lo;
    while (hi < n && img[hi] == q && hi - lo <= kRunMax) ++hi;
    if (hi - lo > kRunMax) *overflow = 1;   // every writer stores the same value
}

__device__ __forceinline__ bool better(double f, int64_t c, double g, int64_t e) {
    return f > g || (f == g && c < e);
}

__device__ __forceinline__ int64_t shfl_xor_i64(int64_t v, int m) {
    const int lo = __shfl_xor((int)(uint32_t)v, m, kWave);
    const int hi = __shfl_xor((int)(v >> 32), m, kWave);
    return (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

// Best (value, cell) over the block, ties to the lower cell; thread 0 gets it.
template <int BT = kBlock>
__device__ __forceinline__ void block_best(double& f, int64_t& c) {
    __shared__ double wf[BT / kWave];
    __shared__ int64_t wc[BT / kWave];
#pragma unroll
    for (int m = kWave / 2; m > 0; m >>= 1) {
        const double g = __shfl_xor(f, m, kWave);
        const int64_t e = shfl_xor_i64(c, m);
        if (better(g, e, f, c)) {
            f = g;
            c = e;
        }
    }
    if ((threadIdx.x & (kWave - 1)) == 0) {
        wf[threadIdx.x / kWave] = f;
        wc[threadIdx.x / kWave] = c;
    }
    __syncthreads();
    if (threadIdx.x == 0)
        for (int w = 1; w < BT / kWave; ++w)
            if (better(wf[w], wc[w], f, c)) {
                f = wf[w];
                c = wc[w];
            }
}

// Bucket (or span) b: s before its first point (s_0 and the earlier buckets' sums, in
// a fixed order), then its cells.  Thread t owns consecutive points.
__global__ __launch_bounds__(kRbThreads) void k_rb_cells(RbDev p) {
    if (!p.span && (p.flag[1] | p.flag[2])) return;
    const int tid = threadIdx.x;
    double2 a = make_double2(0.0, 0.0);
    for (int t = tid; t < p.tiles; t += kRbThreads) a = cadd(a, p.part[t]);
    for (int t = tid; t < (int)blockIdx.x; t += kRbThreads) a = cadd(a, p.bsum[t]);
    const double2 s0 = block_sum_c<kRbThreads>(a);
    const uint32_t st = p.span ? (uint32_t)(blockIdx.x * p.span) : p.start[blockIdx.x];
    const uint32_t cnt = p.span ? (uint32_t)min(p.span, p.n - (int64_t)st) : p.total[blockIdx.x];
    const uint32_t per = (cnt + kRbThreads - 1) / kRbThreads;
    const uint32_t lo = min(cnt, (uint32_t)tid * per), hi = min(cnt, lo + per);
    a = make_double2(0.0, 0.0);
    for (uint32_t e = lo; e < hi; ++e) a = cadd(a, p.d_sorted[st + e]);
    double2 s = block_excl_scan_c<kRbThreads>(a, s0);
    double best = -1.0;
    int64_t cell = INT64_MAX;
    if (blockIdx.x == 0 && tid == 0) {      // the cell before the first point
        best = s0.x * s0.x + s0.y * s0.y;
        cell = 0;
    }
    for (uint32_t e = lo; e < hi; ++e) {
        s = cadd(s, p.d_sorted[st + e]);
        const double f = s.x * s.x + s.y * s.y;
        if (f > best) {          // strict: ties keep the earlier cell
            best = f;
            cell = (int64_t)(st + e) + 1;   // cell l follows the l-th boundary point
        }
    }
    block_best<kRbThreads>(best, cell);
    if (tid == 0) {
        Best b{best, cell, 0ull, 0u, 0};
        if (cell >= 1 && cell <= p.n) {     // an empty bucket has none
            b.coord = p.order[cell - 1];
            b.key = p.keys[b.coord];
        }
        p.bbest[blockIdx.x] = b;
    }
}

// Best cell over the buckets or spans (every block, the same), then the labels of the
// block's tile: coordinate i moves to k_0 + 1 when its boundary point sits at
// a sorted position below the best cell, which is when (key_i, i) <= (key,
// coordinate) of the cell's last point.  Also the partials of z^H q.
__global__ __launch_bounds__(kRbThreads) void k_r1_labels(RbDev p) {
    __shared__ Best win;
    const int tid = threadIdx.x;
    if (blockIdx.x == 0 && tid < 4) p.out->flag[tid] = p.flag[tid];
    if (!p.span && (p.flag[1] | p.flag[2])) return;
    // the first bucket's best stands where no value is a number (q near the
    // largest FP64: the cell before the first point)
    double f = tid ? -1.0 : p.bbest[0].f;
    int64_t c = tid ? INT64_MAX : p.bbest[0].cell;
    int own = tid ? -1 : 0;
    for (int t = tid; t < p.nb; t += kRbThreads)
        if (better(p.bbest[t].f, p.bbest[t].cell, f, c)) {
            f = p.bbest[t].f;
            c = p.bbest[t].cell;
            own = t;
        }
    const int64_t mine = c;
    block_best<kRbThreads>(f, c);
    if (tid == 0) win.cell = c;
    __syncthreads();
    const bool holds = own >= 0 && mine == win.cell;   // cells differ between buckets: one thread
    __syncthreads();
    if (holds) win = p.bbest[own];
    __syncthreads();
    const Best b = win;
    if (blockIdx.x == 0 && tid == 0) p.out->best = b;
    const int64_t lo = blockIdx.x * p.per, hi = min(p.n, lo + p.per);
    double2 v = make_double2(0.0, 0.0);
    for (int64_t i = lo + tid; i < hi; i += kRbThreads) {
        const unsigned long long key = p.keys[i];
        const bool adv = b.cell >= 1 && (key < b.key || (key == b.key && (uint32_t)i <= b.coord));
        int k = p.k0[i] + (adv ? 1 : 0);
        k = k == p.K ? 0 : k;
        p.z[i] = (uint8_t)k;
        v = cadd(v, cconj_mul(p.q[i], p.roots[k]));
    }
    const double2 s = block_sum_c<kRbThreads>(v);
    if (tid == 0) p.lpart[blockIdx.x] = s;
}

int ceil_log2(int64_t x) {
    int b = 0;
    while ((1ll << b) < x) ++b;
    return b;
}

thread_local int t_form = -1;      // form of the thread's last call

// Buckets of 1,024 to 2,048 points; from 256 to 512 points each while that
// leaves fewer than 256 buckets (a block each) for the chip's 256 CUs.
int rb_bucket_bits(int64_t n) {
    return std::max(ceil_log2((n + 2047) / 2048), std::min(8, ceil_log2((n + 511) / 512)));
}

}  // namespace
}  // namespace lrqo

extern "C" {

int32_t lrqo_rank1_form(void) { return lrqo::t_form; }

lrqo_status lrqo_solve_rank1(const double* q, int64_t n, int32_t K, uint8_t* z, lrqo_rank1_result* res) {
    using namespace lrqo;
    clear_error();
    if (!q || !z) return fail(LRQO_EINVAL, "null pointer argument");
    if (n < 1 || n > 0x7fffffffLL) return fail(LRQO_EINVAL, "n must be in [1, 2^31 - 1]");
    if (K < 2 || K > LRQO_MAX_K) return fail(LRQO_EINVAL, "K must be in [2, 255]");
    if (!is_device_pointer(q)) return fail(LRQO_EINVAL, "q is not device memory");
    if (!is_device_pointer(z)) return fail(LRQO_EINVAL, "z is not device memory");
    DeviceCtx* ctx = device_ctx();
    if (!ctx) return LRQO_EDEVICE;
    std::lock_guard<std::mutex> lk(ctx->mu);
    const hipStream_t st = current_stream();

    const int64_t blocks = (n + kBlock - 1) / kBlock;
    // spans of the general form: 2,048 positions, at most 2,048 of them (each
    // block of the cells adds the sums of the spans before its own)
    const int64_t span = std::max<int64_t>(2048, (n + 2047) / 2048);
    const int spans = (int)((n + span - 1) / span);
    const bool buckets = n <= kRbMaxN;
    RbDev p{};
    p.n = n;
    p.K = K;
    p.lb = buckets ? rb_bucket_bits(n) : 0;
    p.nb = buckets ? 1 << p.lb : 0;
    p.tiles = (int)std::min<int64_t>(kRbTiles, (n + kRbThreads - 1) / kRbThreads);
    p.per = (n + p.tiles - 1) / p.tiles;
    const size_t out_bytes = sizeof(RbOut) + sizeof(double2) * (size_t)p.tiles;
    CarveSize cs;
    cs.add<unsigned long long>(n);
    cs.add<uint32_t>(n);
    cs.add<unsigned long long>(n);
    cs.add<uint32_t>(n);
    cs.add<unsigned long long>(n);
    cs.add<uint32_t>(n);
    cs.add<uint32_t>(radix_hist_entries(n));
    cs.add<uint8_t>(n);
    cs.add<double2>(n);
    cs.add<double2>(p.tiles);
    cs.add<double2>(spans);
    cs.add<Best>(spans);
    cs.add<double2>(1 + LRQO_MAX_K);   // the flags, then the roots: one copy
    cs.add<char>(out_bytes);
    cs.add<char>((size_t)p.nb * (sizeof(double2) + sizeof(Best) + sizeof(uint32_t) * (size_t)(2 + p.tiles)));
    CarveSize hs;
    hs.add<double2>(1 + LRQO_MAX_K);
    hs.add<char>(out_bytes);
    LRQO_TRY(reserve_arena(ctx, cs.bytes));
    LRQO_TRY(reserve_host(ctx, hs.bytes));
    Carve cv(ctx->arena);
    p.keys = cv.take<unsigned long long>(n);
    p.img = cv.take<uint32_t>(n);
    unsigned long long* keys_a = cv.take<unsigned long long>(n);
    uint32_t* vals_a = cv.take<uint32_t>(n);
    unsigned long long* keys_b = cv.take<unsigned long long>(n);
    uint32_t* vals_b = cv.take<uint32_t>(n);
    uint32_t* hist = cv.take<uint32_t>(radix_hist_entries(n));
    p.k0 = cv.take<uint8_t>(n);
    p.d_sorted = cv.take<double2>(n);
    p.part = cv.take<double2>(p.tiles);
    double2* span_sum = cv.take<double2>(spans);
    Best* span_best = cv.take<Best>(spans);
    double2* head = cv.take<double2>(1 + LRQO_MAX_K);
    p.out = reinterpret_cast<RbOut*>(cv.take<char>(out_bytes));
    p.bsum = reinterpret_cast<double2*>(cv.take<char>(0));
    p.bbest = reinterpret_cast<Best*>(p.bsum + p.nb);
    p.total = reinterpret_cast<uint32_t*>(p.bbest + p.nb);
    p.start = p.total + p.nb;
    p.hist = p.start + p.nb;
    p.q = reinterpret_cast<const double2*>(q);
    p.roots = head + 1;
    p.flag = reinterpret_cast<int*>(head);
    p.ent = keys_a;
    p.order = vals_a;
    p.lpart = reinterpret_cast<double2*>(p.out + 1);
    p.z = z;
    Carve hv(ctx->host);
    double2* h_head = hv.take<double2>(1 + LRQO_MAX_K);
    RbOut* h_out = reinterpret_cast<RbOut*>(hv.take<char>(out_bytes));

    // roots omega^k = exp(2 pi i k / K), argument (2 pi k)/K; the flags zero
    h_head[0] = make_double2(0.0, 0.0);
    for (int k = 0; k < K; ++k) {
        const double a = (2.0 * kPi * (double)k) / (double)K;
        h_head[1 + k] = make_double2(std::cos(a), std::sin(a));
    }
    LRQO_HIP(hipEventRecord(ctx->ev_start, st));
    LRQO_HIP(hipMemcpyAsync(head, h_head, sizeof(double2) * (size_t)(1 + K), hipMemcpyHostToDevice, st));
    const size_t lds = sizeof(uint32_t) * (size_t)p.nb;
    hipLaunchKernelGGL(k_r1_prep, dim3(p.tiles), dim3(kRbThreads), lds, st, p);
    LRQO_HIP(hipGetLastError());

    // the labels from p's bests, and what the host reads
    const auto finish = [&](const RbDev& b) -> lrqo_status {
        hipLaunchKernelGGL(k_r1_labels, dim3(b.tiles), dim3(kRbThreads), 0, st, b);
        LRQO_HIP(hipGetLastError());
        LRQO_HIP(hipEventRecord(ctx->ev_stop, st));
        LRQO_HIP(hipMemcpyAsync(h_out, b.out, out_bytes, hipMemcpyDeviceToHost, st));
        LRQO_HIP(hipStreamSynchronize(st));
        if (h_out->flag[0]) return fail(LRQO_ENOTFINITE, "q holds a NaN or an infinity");
        return LRQO_OK;
    };
    bool done = false;
    if (buckets) {
        hipLaunchKernelGGL(k_rb_scan, dim3((p.nb + kRbSeg - 1) / kRbSeg), dim3(kRbSeg * kRbSeg), 0, st, p);
        hipLaunchKernelGGL(k_rb_scatter, dim3(p.tiles), dim3(kRbThreads), lds, st, p);
        hipLaunchKernelGGL(k_rb_sort, dim3(p.nb), dim3(kRbThreads), 0, st, p);
        hipLaunchKernelGGL(k_rb_cells, dim3(p.nb), dim3(kRbThreads), 0, st, p);
        LRQO_TRY(finish(p));
        done = !(h_out->flag[1] | h_out->flag[2]);
    }
    int passes = 4;
    if (!done) {
        RbDev g = p;
        g.span = span;
        g.nb = spans;
        g.bsum = span_sum;
        g.bbest = span_best;
        const auto from_order = [&](const uint32_t* order) -> lrqo_status {
            g.order = const_cast<uint32_t*>(order);   // a work buffer of this call
            hipLaunchKernelGGL(k_r1_gather, dim3(spans), dim3(kRbThreads), 0, st, g);
            hipLaunchKernelGGL(k_rb_cells, dim3(spans), dim3(kRbThreads), 0, st, g);
            return finish(g);
        };
        // images first (the 64-bit work buffers hold the 32-bit pairs)
        SortedPairs32 by_img{};
        LRQO_TRY(radix_sort_pairs32(p.img, reinterpret_cast<uint32_t*>(keys_a), vals_a,
                                    reinterpret_cast<uint32_t*>(keys_b), vals_b, hist, n, 0xFu, st, &by_img));
        uint32_t* order_img = const_cast<uint32_t*>(by_img.vals);   // a work buffer of this call
        hipLaunchKernelGGL(k_r1_fixup, dim3((unsigned)blocks), dim3(kBlock), 0, st, by_img.keys, order_img, p.keys, n,
                           p.flag + 3);
        LRQO_TRY(from_order(order_img));
        if (h_out->flag[3]) {
            // the exact keys, skipping digits that are the same in all of them
            const int ob = p.tiles;
            unsigned long long* orand = reinterpret_cast<unsigned long long*>(p.lpart);   // as many pairs as partials
            const unsigned long long* h_orand = reinterpret_cast<const unsigned long long*>(h_out + 1);
            hipLaunchKernelGGL(k_r1_orand, dim3(ob), dim3(kBlock), 0, st, p.keys, n, orand);
            LRQO_HIP(hipGetLastError());
            LRQO_HIP(hipMemcpyAsync(h_out, p.out, out_bytes, hipMemcpyDeviceToHost, st));
            LRQO_HIP(hipStreamSynchronize(st));
            unsigned long long o = 0ull, a = ~0ull;
            for (int t = 0; t < ob; ++t) {
                o |= h_orand[2 * t];
                a &= h_orand[2 * t + 1];
            }
            unsigned mask = 0;
            for (int dgt = 0; dgt < 8; ++dgt)
                if (((o ^ a) >> (8 * dgt)) & 0xFFull) mask |= 1u << dgt;
            if (!mask) mask = 1u;   // the sort runs one pass at least
            SortedPairs exact{};
            LRQO_TRY(radix_sort_pairs(p.keys, keys_a, vals_a, keys_b, vals_b, hist, n, mask, st, &exact));
            LRQO_TRY(from_order(exact.vals));
            passes += __builtin_popcount(mask);
        }
    }
    const double2* lp = reinterpret_cast<const double2*>(h_out + 1);
    double sx = 0.0, sy = 0.0;
    for (int t = 0; t < p.tiles; ++t) {
        sx += lp[t].x;
        sy += lp[t].y;
    }
    float ms = 0.0f;
    LRQO_HIP(hipEventElapsedTime(&ms, ctx->ev_start, ctx->ev_stop));
    t_form = done ? 1 : 0;
    if (res) {
        std::memset(res, 0, sizeof *res);
        res->obj = sx * sx + sy * sy;
        res->sweep_obj = h_out->best.f;
        res->best_cell = h_out->best.cell;
        res->device_ms = ms;
        res->sort_passes = passes;
    }
    return LRQO_OK;
}

}  // extern "C"
