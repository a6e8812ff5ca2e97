// Learned direction proposal for the sampled maximiser (rank r = 3).
//
// A permutation-invariant network reads the rows of V in a canonical gauge
// and returns a mixture of von Mises-Fisher densities on the unit sphere of
// C^3 = R^6; directions drawn from it (with a share of uniform directions
// kept as fallback) are scored by the sampled solver like any other
// candidates, and its objective is always the FP64 rescore.
//
//   gauge     M = sum_i |v_i|^2 v_i^H v_i (FP64); G = eigenvectors of M in
//             descending order, column phases fixed so that sum_i (V G)_ij^K
//             is real positive and arg sum_i (V G)_ij lies in [-pi/K, pi/K);
//             features x_i = s v_i G, s = sqrt(n / ||V||_F^2)
//   network   h1 = relu(W1 x + b1) (64), h2 = relu(W2 h1 + b2) (64),
//             m = mean_i h2, y = W3 m + b3 (32 x (6 + 2)): component k has
//             mean direction mu_k = y_k[0:6]/|.|, logit a_k, kappa_k = exp(y_k[7])
//   density   vMF on S^5: C_6(kappa) exp(kappa mu . x),
//             C_6 = kappa^2 / ((2 pi)^3 I_2(kappa))
//   loss      -log( (1/K) sum_t p(omega^t c*) ) for the canonical target c*
//   training  hand-written backward (row MLP gradients accumulated over LDS
//             row tiles), fixed-order reduction, Adam
//   sampling  Wood's rejection sampler (Beta(5/2, 5/2) from Gamma(2) and
//             Gamma(1/2) variates), Philox-driven, bounded retries
#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "lrqo_device.h"
#include "lrqo_runtime.h"

namespace lrqo {

namespace {

constexpr int DIN = 6, H = 64, NC = 32, OUT = NC * (DIN + 2);
constexpr int NP = H * DIN + H + H * H + H + OUT * H + OUT;   // 21,248 parameters
constexpr int OFF_W1 = 0, OFF_B1 = H * DIN, OFF_W2 = OFF_B1 + H, OFF_B2 = OFF_W2 + H * H,
              OFF_W3 = OFF_B2 + H, OFF_B3 = OFF_W3 + OUT * H;
constexpr int kBlock = 256;
constexpr int kRowTile = 32;   // rows per backward tile (columns of its products)
constexpr int kMaxRetry = 32;  // rejection-sampler attempts before falling back to the mean

struct Frame {                 // canonical gauge of one instance
    double g[18];              // G (3x3 complex, row-major, (re, im))
    double s;
    double pad;
};

// ---------------------------------------------------------------- Bessel
// log I_nu(k): power series below 30, four-term asymptotic expansion above.
__device__ float log_bessel_i(int nu, float k) {
    if (k < 30.0f) {
        const float h2 = 0.25f * k * k;
        float term = nu == 2 ? 0.125f * k * k : k * k * k / 48.0f;   // (k/2)^nu / nu!
        float tot = term;
        for (int m = 1; m < 120; ++m) {
            term *= h2 / (float)(m * (m + nu));
            tot += term;
            if (term < 1e-9f * tot) break;
        }
        return logf(tot);
    }
    const float mu = 4.0f * nu * nu;
    float a = 1.0f, ser = 1.0f, kp = 1.0f, sg = -1.0f;
    for (int j = 1; j <= 4; ++j) {
        a *= (mu - (float)((2 * j - 1) * (2 * j - 1))) / (8.0f * j);
        kp *= k;
        ser += sg * a / kp;
        sg = -sg;
    }
    return k - 0.5f * logf(6.283185307179586f * k) + logf(ser);
}

__device__ float log_vmf_norm(float k) {
    return 2.0f * logf(k) - 3.0f * 1.8378770664093453f - log_bessel_i(2, k);   // 3 log(2 pi)
}

__device__ float mean_resultant(float k) {   // I_3 / I_2 = -d log C_6 / d kappa
    return expf(log_bessel_i(3, k) - log_bessel_i(2, k));
}

// ---------------------------------------------------------------- gauge
// Eigenvectors of a 3x3 Hermitian M in descending eigenvalue order, by
// cyclic complex Jacobi: rotation (p, q) turns column q by e^{-i alpha},
// alpha = arg M_pq, and then zeroes the real off-diagonal entry.  One thread;
// every index is a constant, so M and U stay in registers.  Three rotations a
// sweep with three-entry updates, where the 6x6 real form of M took fifteen
// with six (k_frame_eig, 64 instances: 71 -> 12 us).
__device__ void hermitian_eig3(const double (&Mr)[3][3], const double (&Mi)[3][3],
                               double (&Ur)[3][3], double (&Ui)[3][3]) {
    double d[3], ar[3][3], ai[3][3];           // diagonal; entries above it
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        d[i] = Mr[i][i];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            ar[i][j] = Mr[i][j];
            ai[i][j] = Mi[i][j];
            Ur[i][j] = i == j ? 1.0 : 0.0;
            Ui[i][j] = 0.0;
        }
    }
    for (int sweep = 0; sweep < 30; ++sweep) {
        double off = 0.0;
        const double dia = d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = i + 1; j < 3; ++j) off += ar[i][j] * ar[i][j] + ai[i][j] * ai[i][j];
        // converged when the off-diagonal part is at FP64 rounding of the
        // diagonal (an absolute bound would never be met for large M)
        if (off <= 1e-32 * dia || off < 1e-300) break;
#pragma unroll
        for (int p = 0; p < 3; ++p)
#pragma unroll
            for (int q = p + 1; q < 3; ++q) {
                const double m = sqrt(ar[p][q] * ar[p][q] + ai[p][q] * ai[p][q]);
                if (m < 1e-300) continue;
                const double er = ar[p][q] / m, ei = -ai[p][q] / m;           // e^{-i alpha}
                const double th = (d[q] - d[p]) / (2.0 * m);
                const double t = (th >= 0 ? 1.0 : -1.0) / (fabs(th) + sqrt(th * th + 1.0));
                const double c = 1.0 / sqrt(t * t + 1.0), s = t * c;
                d[p] -= t * m;
                d[q] += t * m;
                ar[p][q] = ai[p][q] = 0.0;
                const int k = 3 - p - q;                                       // the third index
                // M_kp and M_kq from the entries above the diagonal
                double pr = k < p ? ar[k][p] : ar[p][k], pi = k < p ? ai[k][p] : -ai[p][k];
                double qr = k < q ? ar[k][q] : ar[q][k], qi = k < q ? ai[k][q] : -ai[q][k];
                double tr = qr * er - qi * ei;
                qi = qr * ei + qi * er;
                qr = tr;
                const double npr = c * pr - s * qr, npi = c * pi - s * qi;
                const double nqr = s * pr + c * qr, nqi = s * pi + c * qi;
                if (k < p) { ar[k][p] = npr; ai[k][p] = npi; } else { ar[p][k] = npr; ai[p][k] = -npi; }
                if (k < q) { ar[k][q] = nqr; ai[k][q] = nqi; } else { ar[q][k] = nqr; ai[q][k] = -nqi; }
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const double upr = Ur[i][p], upi = Ui[i][p];
                    const double uqr = Ur[i][q] * er - Ui[i][q] * ei, uqi = Ur[i][q] * ei + Ui[i][q] * er;
                    Ur[i][p] = c * upr - s * uqr;
                    Ui[i][p] = c * upi - s * uqi;
                    Ur[i][q] = s * upr + c * uqr;
                    Ui[i][q] = s * upi + c * uqi;
                }
            }
    }
#pragma unroll
    for (int pass = 0; pass < 3; ++pass) {     // compare-exchange (0,1), (1,2), (0,1)
        const int p = pass == 1 ? 1 : 0, q = p + 1;
        const bool sw = d[q] > d[p];
        const double dp = d[p];
        d[p] = sw ? d[q] : d[p];
        d[q] = sw ? dp : d[q];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const double xr = Ur[i][p], xi = Ui[i][p];
            Ur[i][p] = sw ? Ur[i][q] : xr;
            Ui[i][p] = sw ? Ui[i][q] : xi;
            Ur[i][q] = sw ? xr : Ur[i][q];
            Ui[i][q] = sw ? xi : Ui[i][q];
        }
    }
}

// Block sums of N values: each wave's sum (butterfly), then the waves in
// order; out[e] is written by thread e.
template <int N>
__device__ __forceinline__ void block_sums(const double (&x)[N], double (*red)[kBlock / kWave], double* out) {
    const int w = threadIdx.x / kWave;
#pragma unroll
    for (int e = 0; e < N; ++e) {
        const double v = wave_sum_f64(x[e]);
        if ((threadIdx.x & (kWave - 1)) == 0) red[e][w] = v;
    }
    __syncthreads();
    if (threadIdx.x < N) {
        double t = 0.0;
        for (int i = 0; i < kBlock / kWave; ++i) t += red[threadIdx.x][i];
        out[threadIdx.x] = t;
    }
}

// Canonical frame of each instance in four stages, the two row passes split
// over `splits` blocks per instance (row range q of ceil(n / splits) rows),
// their partial sums added in split order (FP64):
//   k_frame_m    per split: sum_i |v_i|^2 conj(v_ia) v_ib and sum_i |v_i|^2
//   k_frame_eig  per instance: M, its eigenvectors (descending) -> g, scale s
//   k_frame_p    per split: sum_i (s V U)_ib^K (binary exponentiation of the
//                complex number) and sum_i (s V U)_ib
//   k_frame_fin  per instance: column phases from the two sums -> g
constexpr int kFrameM = 19, kFrameP = 12;

__device__ __forceinline__ void split_rows(int64_t n, int q, int splits, int64_t& r0, int64_t& r1) {
    const int64_t per = (n + splits - 1) / splits;
    r0 = min(n, (int64_t)q * per);
    r1 = min(n, r0 + per);
}

__global__ __launch_bounds__(kBlock) void k_frame_m(const float* __restrict__ V, const int64_t* voff,
                                                   const int64_t* nrows, int splits, double* __restrict__ work) {
    __shared__ double red[kFrameM][kBlock / kWave];
    const int t = blockIdx.x, q = blockIdx.y;
    const float* Vt = V + voff[t];
    int64_t r0, r1;
    split_rows(nrows[t], q, splits, r0, r1);
    double acc[kFrameM] = {0};   // 9 complex entries of M, then sum |v|^2
    for (int64_t i = r0 + threadIdx.x; i < r1; i += kBlock) {
        double vr[3], vi[3], w = 0.0;
        for (int j = 0; j < 3; ++j) {
            vr[j] = Vt[i * 6 + 2 * j];
            vi[j] = Vt[i * 6 + 2 * j + 1];
            w += vr[j] * vr[j] + vi[j] * vi[j];
        }
        for (int a = 0; a < 3; ++a)
            for (int b = 0; b < 3; ++b) {   // conj(v_a) v_b
                acc[2 * (3 * a + b)] += w * (vr[a] * vr[b] + vi[a] * vi[b]);
                acc[2 * (3 * a + b) + 1] += w * (vr[a] * vi[b] - vi[a] * vr[b]);
            }
        acc[18] += w;
    }
    block_sums<kFrameM>(acc, red, work + ((size_t)t * splits + q) * kFrameM);
}

// One wave sums each entry e < W of instance t over the splits into tot[e]:
// lane l adds splits l, l + 64, ... in order (all W entries' loads in flight
// together), then the 64 lane sums are added by a butterfly (a fixed order).
template <int W>
__device__ __forceinline__ void sum_splits(const double* __restrict__ work, int t, int splits, double* tot) {
    const int l = threadIdx.x;              // blockDim.x == kWave
    const double* src = work + (size_t)t * splits * W;
    double a[W];
#pragma unroll
    for (int e = 0; e < W; ++e) a[e] = 0.0;
    for (int q = l; q < splits; q += kWave) {
#pragma unroll
        for (int e = 0; e < W; ++e) a[e] += src[(size_t)q * W + e];
    }
#pragma unroll
    for (int e = 0; e < W; ++e) {
        const double x = wave_sum_f64(a[e]);
        if (l == 0) tot[e] = x;
    }
    __syncthreads();
}

__global__ __launch_bounds__(kWave) void k_frame_eig(const double* __restrict__ work, const int64_t* nrows, int splits,
                            Frame* __restrict__ frames) {
    __shared__ double tot[kFrameM];
    const int t = blockIdx.x;
    sum_splits<kFrameM>(work, t, splits, tot);
    if (threadIdx.x != 0) return;
    double Mr[3][3], Mi[3][3], Ur[3][3], Ui[3][3];
    for (int a = 0; a < 3; ++a)
        for (int b = 0; b < 3; ++b) {
            Mr[a][b] = tot[2 * (3 * a + b)];
            Mi[a][b] = tot[2 * (3 * a + b) + 1];
        }
    hermitian_eig3(Mr, Mi, Ur, Ui);
    Frame f;
    for (int a = 0; a < 3; ++a)
        for (int b = 0; b < 3; ++b) {
            f.g[2 * (3 * a + b)] = Ur[a][b];
            f.g[2 * (3 * a + b) + 1] = Ui[a][b];
        }
    f.s = sqrt((double)nrows[t] / tot[18]);
    f.pad = 0.0;
    frames[t] = f;
}

// w^K for an integer K >= 1 by binary exponentiation
__device__ __forceinline__ void cpow_int(double wr, double wi, int K, double& pr, double& pi) {
    double rr = 1.0, ri = 0.0, br = wr, bi = wi;
    for (int e = K; e > 0; e >>= 1) {
        if (e & 1) {
            const double x = rr * br - ri * bi;
            ri = rr * bi + ri * br;
            rr = x;
        }
        if (e > 1) {
            const double x = br * br - bi * bi;
            bi = 2.0 * br * bi;
            br = x;
        }
    }
    pr = rr;
    pi = ri;
}

__global__ __launch_bounds__(kBlock) void k_frame_p(const float* __restrict__ V, const int64_t* voff,
                                                   const int64_t* nrows, int splits, int K,
                                                   const Frame* __restrict__ frames, double* __restrict__ work) {
    __shared__ double red[kFrameP][kBlock / kWave];
    __shared__ double Us[18];
    const int t = blockIdx.x, q = blockIdx.y;
    if (threadIdx.x < 18) Us[threadIdx.x] = frames[t].g[threadIdx.x];
    __syncthreads();
    const double s = frames[t].s;
    const float* Vt = V + voff[t];
    int64_t r0, r1;
    split_rows(nrows[t], q, splits, r0, r1);
    double sums[kFrameP] = {0};   // K-th moments, then first moments
    for (int64_t i = r0 + threadIdx.x; i < r1; i += kBlock) {
        double vr[3], vi[3];
        for (int j = 0; j < 3; ++j) {
            vr[j] = s * Vt[i * 6 + 2 * j];
            vi[j] = s * Vt[i * 6 + 2 * j + 1];
        }
        for (int b = 0; b < 3; ++b) {
            double wr = 0.0, wi = 0.0;
            for (int a = 0; a < 3; ++a) {
                const double ur = Us[2 * (3 * a + b)], ui = Us[2 * (3 * a + b) + 1];
                wr += vr[a] * ur - vi[a] * ui;
                wi += vr[a] * ui + vi[a] * ur;
            }
            sums[6 + 2 * b] += wr;
            sums[6 + 2 * b + 1] += wi;
            double pr, pim;
            cpow_int(wr, wi, K, pr, pim);
            sums[2 * b] += pr;
            sums[2 * b + 1] += pim;
        }
    }
    block_sums<kFrameP>(sums, red, work + ((size_t)t * splits + q) * kFrameP);
}

__global__ __launch_bounds__(kWave) void k_frame_fin(const double* __restrict__ work, int splits, int K, Frame* __restrict__ frames) {
    __shared__ double tot[kFrameP];
    const int t = blockIdx.x;
    sum_splits<kFrameP>(work, t, splits, tot);
    if (threadIdx.x != 0) return;
    double PK[6], P1[6];
    for (int e = 0; e < 6; ++e) {
        PK[e] = tot[e];
        P1[e] = tot[6 + e];
    }
    Frame f = frames[t];
    double Us[18];
    for (int e = 0; e < 18; ++e) Us[e] = f.g[e];
    const double two_pi = 6.283185307179586476925286766559;
    for (int b = 0; b < 3; ++b) {
        const double phi = atan2(PK[2 * b + 1], PK[2 * b]) / K;
        // first moment after the K-th-moment phase: rotate into [-pi/K, pi/K)
        const double c1 = cos(-phi), s1 = sin(-phi);
        const double fr = P1[2 * b] * c1 - P1[2 * b + 1] * s1;
        const double fi = P1[2 * b] * s1 + P1[2 * b + 1] * c1;
        const double psi = atan2(fi, fr);
        const double m = floor(psi * K / two_pi + 0.5);
        const double ang = -phi - two_pi * m / K;
        const double cr = cos(ang), ci = sin(ang);
        for (int a = 0; a < 3; ++a) {
            const double ur = Us[2 * (3 * a + b)], ui = Us[2 * (3 * a + b) + 1];
            f.g[2 * (3 * a + b)] = ur * cr - ui * ci;
            f.g[2 * (3 * a + b) + 1] = ur * ci + ui * cr;
        }
    }
    frames[t] = f;
}

// Row splits for frames of `count` instances of at most max_n rows: about
// 1024 blocks in all, at least 1024 rows per split.
int frame_splits(int count, int64_t max_n) {
    int64_t sp = (1024 + count - 1) / count;
    sp = std::min<int64_t>(sp, std::max<int64_t>(1, max_n / 1024));
    return (int)std::max<int64_t>(1, std::min<int64_t>(sp, 256));
}

// Work doubles the frame stages need.
size_t frame_work(int count, int splits) { return (size_t)count * splits * (kFrameM + kFrameP); }

void launch_frames(const float* V, const int64_t* voff, const int64_t* n, int count, int splits, int K,
                   Frame* frames, double* work, hipStream_t st) {
    double* wm = work;
    double* wp = work + (size_t)count * splits * kFrameM;
    hipLaunchKernelGGL(k_frame_m, dim3(count, splits), dim3(kBlock), 0, st, V, voff, n, splits, wm);
    hipLaunchKernelGGL(k_frame_eig, dim3(count), dim3(64), 0, st, wm, n, splits, frames);
    hipLaunchKernelGGL(k_frame_p, dim3(count, splits), dim3(kBlock), 0, st, V, voff, n, splits, K, frames, wp);
    hipLaunchKernelGGL(k_frame_fin, dim3(count), dim3(64), 0, st, wp, splits, K, frames);
}

__device__ __forceinline__ void feature_row(const float* Vt, int64_t i, const Frame& f, float (&x)[DIN]) {
    float vr[3], vi[3];
    for (int j = 0; j < 3; ++j) {
        vr[j] = Vt[i * 6 + 2 * j];
        vi[j] = Vt[i * 6 + 2 * j + 1];
    }
    for (int b = 0; b < 3; ++b) {
        float wr = 0.0f, wi = 0.0f;
        for (int a = 0; a < 3; ++a) {
            const float gr = (float)f.g[2 * (3 * a + b)], gi = (float)f.g[2 * (3 * a + b) + 1];
            wr += vr[a] * gr - vi[a] * gi;
            wi += vr[a] * gi + vi[a] * gr;
        }
        x[2 * b] = (float)f.s * wr;
        x[2 * b + 1] = (float)f.s * wi;
    }
}

// ---------------------------------------------------------------- forward
// Blocks of 256 rows; item j covers rows [start, start+256) of instance inst.
struct RowItems {
    const int32_t* inst;
    const int64_t* start;
    int32_t count;
};

// The row network on the matrix core, in FP32 (v_mfma_f32_32x32x2_f32, which
// adds its two products to the accumulator as two FMAs in k order, so a sum
// over k is the same FP32 chain as on the vector ALU, bit for bit).  The
// vector form read every weight from LDS once per row and FMA and was bound by
// those reads (262,144 rows: 68 us, 354,000 rows of a mini-batch 107 us; now
// 33 and 46, against 15 and 21 us of matrix-core time).  A wave takes 32 rows as the columns of the products:
// neurons are rows of the result, and its row 8j + 4h + c (held by lane half
// h) is neuron 2 (16 m + 4 j + c) + h of block m.  Result register 4j + c of
// block m is then neuron k = 2s + h, s = 16 m + 4 j + c: exactly the operand
// that k-step s of the next layer takes from that lane.
typedef float v16f __attribute__((ext_vector_type(16)));

__device__ __forceinline__ int neuron_of(int row, int m) {
    return 2 * (16 * m + 4 * (row >> 3) + (row & 3)) + ((row >> 2) & 1);
}

// Operands of the first layer: lane l holds row l % 32, k = 2s + l / 32.
__device__ __forceinline__ void load_w1(const float* __restrict__ theta, int lane, float (&w1)[2][3]) {
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int s = 0; s < 3; ++s)
            w1[m][s] = theta[OFF_W1 + neuron_of(lane & 31, m) * DIN + 2 * s + (lane >> 5)];
}

// Bias of this lane's result registers (b: 64 floats in LDS).
__device__ __forceinline__ v16f bias_regs(const float* b, int m, int h) {
    v16f v;
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = b[2 * (16 * m + i) + h];
    return v;
}

// First layer of 32 rows: h1[m][i] = relu of neuron 2 (16 m + i) + h.
__device__ __forceinline__ void layer1(const float (&x)[DIN], const float (&w1)[2][3], const float* b1, int h,
                                       v16f (&h1)[2]) {
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        v16f a = bias_regs(b1, m, h);
#pragma unroll
        for (int s = 0; s < 3; ++s)
            a = __builtin_amdgcn_mfma_f32_32x32x2f32(w1[m][s], h ? x[2 * s + 1] : x[2 * s], a, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 16; ++i) h1[m][i] = fmaxf(a[i], 0.0f);
    }
}

// Sums of v[q] over each half-wave's 32 lanes; lane l returns that of
// register l % 32.  At every level a lane keeps the registers whose index has
// its lane bit and adds the partner's.
template <int N>
__device__ __forceinline__ float half_wave_sums(const float (&v)[N], int lane) {
    if constexpr (N == 1) {
        return v[0];
    } else {
        float u[N / 2];
#pragma unroll
        for (int q = 0; q < N / 2; ++q) {
            const float lo = v[q], hi = v[q + N / 2];
            const bool up = (lane & (N / 2)) != 0;
            u[q] = (up ? hi : lo) + __shfl_xor(up ? lo : hi, N / 2, kWave);
        }
        return half_wave_sums(u, lane);
    }
}

__global__ __launch_bounds__(kBlock, 2) void k_mlp_fwd(const float* __restrict__ V, const int64_t* voff,
                                                      const int64_t* nrows, const Frame* frames,
                                                      const float* __restrict__ theta, RowItems items,
                                                      float* __restrict__ partial /*[items][H]*/) {
    __shared__ float b1[H], b2[H];
    __shared__ float hs[kBlock / kWave][H];
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave, h = lane >> 5;
    if (threadIdx.x < H) {
        b1[threadIdx.x] = theta[OFF_B1 + threadIdx.x];
        b2[threadIdx.x] = theta[OFF_B2 + threadIdx.x];
    }
    float w1[2][3], w2[2][32];
    load_w1(theta, lane, w1);
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        const float4* row = reinterpret_cast<const float4*>(theta + OFF_W2 + neuron_of(lane & 31, m) * H);
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const float4 v = row[q];
            w2[m][2 * q] = h ? v.y : v.x;
            w2[m][2 * q + 1] = h ? v.w : v.z;
        }
    }
    __syncthreads();
    for (int it = blockIdx.x; it < items.count; it += gridDim.x) {
        const int t = items.inst[it];
        const int64_t n = nrows[t];
        // a wave's 64 rows in two halves; their sums are added as a butterfly over
        // 64 lanes would add them (the halves first)
        float sum[32];
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int64_t i = items.start[it] + kWave * w + 32 * half + (lane & 31);
            const bool live = i < n;
            float x[DIN];
#pragma unroll
            for (int k = 0; k < DIN; ++k) x[k] = 0.0f;
            if (live) feature_row(V + voff[t], i, frames[t], x);
            v16f h1[2];
            layer1(x, w1, b1, h, h1);
            v16f a[2] = {bias_regs(b2, 0, h), bias_regs(b2, 1, h)};
#pragma unroll
            for (int s = 0; s < 32; ++s)
#pragma unroll
                for (int m = 0; m < 2; ++m)
                    a[m] = __builtin_amdgcn_mfma_f32_32x32x2f32(w2[m][s], h1[s / 16][s % 16], a[m], 0, 0, 0);
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int q = 0; q < 16; ++q) {
                    const float v = live ? fmaxf(a[m][q], 0.0f) : 0.0f;
                    sum[16 * m + q] = half ? sum[16 * m + q] + v : v;
                }
        }
        hs[w][2 * (lane & 31) + h] = half_wave_sums(sum, lane);
        __syncthreads();
        if (threadIdx.x < H) {
            float v = 0.0f;
            for (int q = 0; q < kBlock / kWave; ++q) v += hs[q][threadIdx.x];
            partial[(size_t)it * H + threadIdx.x] = v;
        }
        __syncthreads();
    }
}

// Mean embedding per instance from its items' partial sums (items of one
// instance are consecutive).  kPoolGroups groups of H threads each add a
// contiguous run of the items (in item order, sixteen loads in flight); the
// group sums are then added in group order.
constexpr int kPoolGroups = 16;

__global__ __launch_bounds__(H * kPoolGroups) void k_pool(const float* __restrict__ partial, const int32_t* first_item,
                                                          const int64_t* nrows, int count, float* __restrict__ mvec) {
    __shared__ float gsum[kPoolGroups][H];
    const int t = blockIdx.x;
    const int o = threadIdx.x % H, grp = threadIdx.x / H;
    if (t >= count) return;                  // the same in every thread of the block
    const int first = first_item[t], end = first_item[t + 1];
    const int per = (end - first + kPoolGroups - 1) / kPoolGroups;
    int it = min(end, first + grp * per);
    const int stop = min(end, it + per);
    float v = 0.0f;
    for (; it + 16 <= stop; it += 16) {
        float p[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) p[u] = partial[(size_t)(it + u) * H + o];
#pragma unroll
        for (int u = 0; u < 16; ++u) v += p[u];
    }
    for (; it < stop; ++it) v += partial[(size_t)it * H + o];
    gsum[grp][o] = v;
    __syncthreads();
    if (grp == 0) {
        float sum = 0.0f;
        for (int g = 0; g < kPoolGroups; ++g) sum += gsum[g][o];
        mvec[(size_t)t * H + o] = sum / (float)nrows[t];
    }
}

// Head: mixture parameters of one instance.
struct Mixture {
    float mu[NC][DIN];
    float logpi[NC];
    float kappa[NC];
    float logc[NC];
    float nrm[NC];
};

__device__ void head(const float* theta, const float* m, Mixture& mx, float* y /*[OUT]*/) {
    for (int o = threadIdx.x; o < OUT; o += blockDim.x) {
        float a = theta[OFF_B3 + o];
        const float4* row = reinterpret_cast<const float4*>(theta + OFF_W3 + o * H);
#pragma unroll 8
        for (int q = 0; q < H / 4; ++q) {
            const float4 v = row[q];
            a = fmaf(v.x, m[4 * q], a);
            a = fmaf(v.y, m[4 * q + 1], a);
            a = fmaf(v.z, m[4 * q + 2], a);
            a = fmaf(v.w, m[4 * q + 3], a);
        }
        y[o] = a;
    }
    __syncthreads();
    if (threadIdx.x < NC) {
        const int k = threadIdx.x;
        float nrm = 0.0f;
        for (int d = 0; d < DIN; ++d) nrm += y[k * (DIN + 2) + d] * y[k * (DIN + 2) + d];
        nrm = sqrtf(nrm);
        mx.nrm[k] = nrm;
        for (int d = 0; d < DIN; ++d) mx.mu[k][d] = y[k * (DIN + 2) + d] / nrm;
        const float kap = expf(y[k * (DIN + 2) + DIN + 1]);
        mx.kappa[k] = kap;
        mx.logc[k] = log_vmf_norm(kap);
    }
    __syncthreads();
    if (threadIdx.x < kWave) {   // log-softmax of the logits, terms added in component order
        const float a = threadIdx.x < NC ? y[threadIdx.x * (DIN + 2) + DIN] : -INFINITY;
        float amax = a;
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off, kWave));
        const float e = expf(a - amax);
        float se = 0.0f;
#pragma unroll
        for (int k = 0; k < NC; ++k) se += __shfl(e, k, kWave);
        if (threadIdx.x < NC) mx.logpi[threadIdx.x] = a - (amax + logf(se));
    }
    __syncthreads();
}

// Per instance: loss, d loss / d y, d loss / d m (for the row backward), and
// this instance's share of dW3, db3.  One block of 256 threads.
__global__ __launch_bounds__(kBlock) void k_head_loss(const float* __restrict__ theta,
                                                     const float* __restrict__ mvec,
                                                     const float* __restrict__ target /*[count][6] canonical c**/,
                                                     int K, float* __restrict__ loss,
                                                     float* __restrict__ dmvec, float* __restrict__ gW3 /*[count][OUT*H+OUT]*/) {
    __shared__ Mixture mx;
    __shared__ float y[OUT], dy[OUT], m[H];
    __shared__ float lg[256][NC + 1];   // K <= 255 rotations
    __shared__ float Q[NC], Xb[NC][DIN];
    const int t = blockIdx.x;
    if (threadIdx.x < H) m[threadIdx.x] = mvec[(size_t)t * H + threadIdx.x];
    __syncthreads();
    head(theta, m, mx, y);
    const float* c = target + (size_t)t * DIN;
    // log(pi_k) + log f_k(omega^r c*) for every rotation r and component k
    for (int e = threadIdx.x; e < K * NC; e += kBlock) {
        const int r = e / NC, k = e % NC;
        const float ang = 6.283185307179586f * (float)r / (float)K;
        const float cs = cosf(ang), sn = sinf(ang);
        float dot = 0.0f;
        for (int j = 0; j < 3; ++j) {
            const float xr = cs * c[2 * j] - sn * c[2 * j + 1];
            const float xi = sn * c[2 * j] + cs * c[2 * j + 1];
            dot += mx.mu[k][2 * j] * xr + mx.mu[k][2 * j + 1] * xi;
        }
        lg[r][k] = mx.logpi[k] + mx.logc[k] + mx.kappa[k] * dot;
    }
    __syncthreads();
    // log-sum-exp over all entries: thread maxima and sums, then over the block
    __shared__ float lse_s, wred[kBlock / kWave];
    const int wv = threadIdx.x / kWave;
    float mxv = -INFINITY;
    for (int e = threadIdx.x; e < K * NC; e += kBlock) mxv = fmaxf(mxv, lg[e / NC][e % NC]);
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) mxv = fmaxf(mxv, __shfl_xor(mxv, off, kWave));
    if ((threadIdx.x & (kWave - 1)) == 0) wred[wv] = mxv;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kBlock / kWave; ++q) mxv = fmaxf(mxv, wred[q]);
    __syncthreads();
    float se = 0.0f;
    for (int e = threadIdx.x; e < K * NC; e += kBlock) se += expf(lg[e / NC][e % NC] - mxv);
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) se += __shfl_xor(se, off, kWave);
    if ((threadIdx.x & (kWave - 1)) == 0) wred[wv] = se;
    __syncthreads();
    if (threadIdx.x == 0) {
        float tot = 0.0f;
        for (int q = 0; q < kBlock / kWave; ++q) tot += wred[q];
        lse_s = mxv + logf(tot);
        loss[t] = -(lse_s - logf((float)K));
    }
    __syncthreads();
    // posterior q_{rk}: component mass Q_k and weighted mean X̄_k
    if (threadIdx.x < NC) {
        const int k = threadIdx.x;
        float qk = 0.0f, xb[DIN] = {0};
        for (int r = 0; r < K; ++r) {
            const float q = expf(lg[r][k] - lse_s);
            qk += q;
            const float ang = 6.283185307179586f * (float)r / (float)K;
            const float cs = cosf(ang), sn = sinf(ang);
            for (int j = 0; j < 3; ++j) {
                xb[2 * j] += q * (cs * c[2 * j] - sn * c[2 * j + 1]);
                xb[2 * j + 1] += q * (sn * c[2 * j] + cs * c[2 * j + 1]);
            }
        }
        Q[k] = qk;
        for (int d = 0; d < DIN; ++d) Xb[k][d] = xb[d];
    }
    __syncthreads();
    if (threadIdx.x < NC) {
        const int k = threadIdx.x;
        const float kap = mx.kappa[k];
        float mux = 0.0f;
        for (int d = 0; d < DIN; ++d) mux += mx.mu[k][d] * Xb[k][d];
        const float dkappa = -(Q[k] * (-mean_resultant(kap)) + mux);
        dy[k * (DIN + 2) + DIN + 1] = dkappa * kap;
        dy[k * (DIN + 2) + DIN] = -Q[k] + expf(mx.logpi[k]);
        float dmu[DIN], proj = 0.0f;
        for (int d = 0; d < DIN; ++d) {
            dmu[d] = -kap * Xb[k][d];
            proj += dmu[d] * mx.mu[k][d];
        }
        for (int d = 0; d < DIN; ++d) dy[k * (DIN + 2) + d] = (dmu[d] - proj * mx.mu[k][d]) / mx.nrm[k];
    }
    __syncthreads();
    float* g = gW3 + (size_t)t * (OUT * H + OUT);
    for (int e = threadIdx.x; e < OUT * H; e += kBlock) g[e] = dy[e / H] * m[e % H];
    for (int o = threadIdx.x; o < OUT; o += kBlock) g[OUT * H + o] = dy[o];
    if (threadIdx.x < H) {
        float a = 0.0f;
        for (int o = 0; o < OUT; ++o) a = fmaf(theta[OFF_W3 + o * H + threadIdx.x], dy[o], a);
        dmvec[(size_t)t * H + threadIdx.x] = a;
    }
}

// Row backward.  A wave takes tiles of kRowTile = 32 rows (a contiguous run of
// the tile list) and keeps the weight gradients of all of them in registers;
// the eight waves of a block are added once at the end into partial[block].
// All three products run on the matrix core in FP32 like the forward pass:
//   layer 2 (recomputed) and D1 = W2^T D2 (* relu'): operands straight from the
//     previous product's registers, weights in lane order in LDS;
//   dW2 = D2 A1^T over the rows: D2 is relu' times one value per neuron, so its
//     operand is that value masked by a bit of the neuron's row mask (the
//     ballots of the signs); A1 is turned through LDS.
// dW1 and db1 (six columns) are vector FMAs, lane = neuron.  The vector form
// read two LDS operands per FMA and wrote 18 KB of partial sums per 64 rows
// (mini-batch of 354,000 rows: 453 us, now 114; the reduction of the partials
// 32 -> 5 us); its FP32 products take 62 us at the matrix-core rate.
constexpr int kBwdBlock = 512, kBwdWaves = kBwdBlock / kWave;
constexpr int kBwdBlocks = 256;            // one block per CU (102 KB of LDS)
constexpr int NG = H * DIN + H + H * H + H;

struct BwdLds {
    float4 wf[2][8][kWave], wb[2][8][kWave];   // operands of layer 2 and of D1: [block][step / 4][lane]
    float a[kBwdWaves][kRowTile][H + 1];       // A1, then D1 of a wave's tile
    float x[kBwdWaves][kRowTile][8];           // features
    unsigned mask[kBwdWaves][H];               // row masks of the neurons of layer 2
    float dh[kBwdWaves][H];                    // d loss / d h2 of the wave's instance
    float b1[H], b2[H];
};
static_assert(sizeof(BwdLds) <= 160 * 1024, "one block per CU");

// Compiler fence between LDS writes and reads of other lanes of the same wave
// (the LDS serves a wave's accesses in order).
__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__global__ __launch_bounds__(kBwdBlock, 2) void k_mlp_bwd(const float* __restrict__ V, const int64_t* voff,
                                                         const int64_t* nrows, const Frame* frames,
                                                         const float* __restrict__ theta,
                                                         const float* __restrict__ dmvec, RowItems items, int per_wave,
                                                         float* __restrict__ partial) {
    __shared__ BwdLds L;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave, h = lane >> 5, col = lane & 31;
    for (int e = tid; e < 2 * 8 * kWave; e += kBwdBlock) {
        const int l = e & (kWave - 1), q = (e / kWave) & 7, m = e / (8 * kWave), o = neuron_of(l & 31, m);
        float f[4], g[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int k = 2 * (4 * q + c) + (l >> 5);
            f[c] = theta[OFF_W2 + o * H + k];          // layer 2: rows are neurons, k-step s is input 2s + h
            g[c] = theta[OFF_W2 + k * H + o];          // D1: rows are inputs, k-step s is neuron 2s + h
        }
        L.wf[m][q][l] = make_float4(f[0], f[1], f[2], f[3]);
        L.wb[m][q][l] = make_float4(g[0], g[1], g[2], g[3]);
    }
    if (tid < H) {
        L.b1[tid] = theta[OFF_B1 + tid];
        L.b2[tid] = theta[OFF_B2 + tid];
    }
    float w1[2][3];
    load_w1(theta, lane, w1);
    __syncthreads();

    v16f gw2[2][2];                            // dW2: neurons 32 M .., inputs 32 N ..
    float gw1[DIN], gb1 = 0.0f, gb2[2] = {0.0f, 0.0f};
#pragma unroll
    for (int M = 0; M < 2; ++M)
#pragma unroll
        for (int N = 0; N < 2; ++N)
#pragma unroll
            for (int i = 0; i < 16; ++i) gw2[M][N][i] = 0.0f;
#pragma unroll
    for (int k = 0; k < DIN; ++k) gw1[k] = 0.0f;

    // a += weights (LDS, lane order) times the registers of a previous product
    auto product = [&](const float4 (&wt)[2][8][kWave], const v16f (&in)[2], v16f (&a)[2]) {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const float4 w0 = wt[0][q][lane], w1q = wt[1][q][lane];
            const float wv[2][4] = {{w0.x, w0.y, w0.z, w0.w}, {w1q.x, w1q.y, w1q.z, w1q.w}};
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int m = 0; m < 2; ++m)
                    a[m] = __builtin_amdgcn_mfma_f32_32x32x2f32(wv[m][c], in[q / 4][4 * (q % 4) + c], a[m], 0, 0, 0);
        }
    };
    const int it0 = (blockIdx.x * kBwdWaves + w) * per_wave, it1 = min(items.count, it0 + per_wave);
    int cur = -1;
    float dl[2] = {0.0f, 0.0f};                // d loss / d h2 of neurons col and 32 + col
    for (int it = it0; it < it1; ++it) {
        const int t = __builtin_amdgcn_readfirstlane(items.inst[it]);
        const int64_t n = nrows[t];
        if (t != cur) {
            cur = t;
            wave_fence();
            L.dh[w][lane] = dmvec[(size_t)t * H + lane] / (float)n;   // mean pooling
            wave_fence();
            dl[0] = L.dh[w][col];
            dl[1] = L.dh[w][32 + col];
        }
        const int64_t i = items.start[it] + col;
        const bool live = i < n;
        float x[DIN];
#pragma unroll
        for (int k = 0; k < DIN; ++k) x[k] = 0.0f;
        if (live) feature_row(V + voff[t], i, frames[t], x);
        if (h == 0) {
#pragma unroll
            for (int k = 0; k < DIN; ++k) L.x[w][col][k] = x[k];
        }
        v16f h1[2], d2[2];
        layer1(x, w1, L.b1, h, h1);
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                h1[m][q] = live ? h1[m][q] : 0.0f;
                L.a[w][col][2 * (16 * m + q) + h] = h1[m][q];
            }
        v16f a[2] = {bias_regs(L.b2, 0, h), bias_regs(L.b2, 1, h)};
        product(L.wf, h1, a);
#pragma unroll
        for (int m = 0; m < 2; ++m) {
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                const bool on = live && a[m][q] > 0.0f;
                const unsigned long long rows = __ballot(on);   // low half: neuron 2s, high half: 2s + 1
                L.mask[w][2 * (16 * m + q) + h] = h ? (unsigned)(rows >> 32) : (unsigned)rows;
                d2[m][q] = on ? L.dh[w][2 * (16 * m + q) + h] : 0.0f;
            }
        }
        wave_fence();
        // dW2 and db2
        unsigned bits[2];
#pragma unroll
        for (int M = 0; M < 2; ++M) {
            bits[M] = L.mask[w][32 * M + col];
            gb2[M] = fmaf((float)__popc(bits[M]), dl[M], gb2[M]);
            bits[M] >>= h;
        }
#pragma unroll
        for (int s = 0; s < kRowTile / 2; ++s) {        // rows 2s, 2s + 1
            float dv[2], av[2];
#pragma unroll
            for (int M = 0; M < 2; ++M) {
                const int on = ((int)(bits[M] << (31 - 2 * s))) >> 31;
                dv[M] = __int_as_float(__float_as_int(dl[M]) & on);
                av[M] = L.a[w][2 * s + h][32 * M + col];
            }
#pragma unroll
            for (int M = 0; M < 2; ++M)
#pragma unroll
                for (int N = 0; N < 2; ++N)
                    gw2[M][N] = __builtin_amdgcn_mfma_f32_32x32x2f32(dv[M], av[N], gw2[M][N], 0, 0, 0);
        }
        wave_fence();
        // D1 over A1's place
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int q = 0; q < 16; ++q) a[m][q] = 0.0f;
        product(L.wb, d2, a);
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int q = 0; q < 16; ++q) L.a[w][col][2 * (16 * m + q) + h] = h1[m][q] > 0.0f ? a[m][q] : 0.0f;
        wave_fence();
        // dW1, db1: lane = neuron
#pragma unroll 4
        for (int r = 0; r < kRowTile; ++r) {
            const float d = L.a[w][r][lane];
            gb1 += d;
#pragma unroll
            for (int k = 0; k < DIN; ++k) gw1[k] = fmaf(d, L.x[w][r][k], gw1[k]);
        }
        wave_fence();
    }

    // the block's waves: half of them at a time hand their sums to the others
    static_assert(sizeof(float) * NG * (kBwdWaves / 2) <= sizeof(BwdLds), "wave sums fit");
    float* hand = reinterpret_cast<float*>(&L);
    auto each = [&](auto f) {                  // (entry of partial, register, held by this lane)
#pragma unroll
        for (int M = 0; M < 2; ++M)
#pragma unroll
            for (int N = 0; N < 2; ++N)
#pragma unroll
                for (int q = 0; q < 16; ++q) {
                    const int o = 32 * M + 8 * (q / 4) + 4 * h + q % 4;
                    float v = gw2[M][N][q];
                    f(H * DIN + H + o * H + 32 * N + col, v, true);
                    gw2[M][N][q] = v;
                }
#pragma unroll
        for (int k = 0; k < DIN; ++k) f(lane * DIN + k, gw1[k], true);
        f(H * DIN + lane, gb1, true);
#pragma unroll
        for (int M = 0; M < 2; ++M) f(H * DIN + H + H * H + 32 * M + col, gb2[M], h == 0);
    };
    for (int half = kBwdWaves / 2; half > 0; half >>= 1) {
        __syncthreads();
        if (w >= half && w < 2 * half)
            each([&](int e, float& v, bool mine) { if (mine) hand[(w - half) * NG + e] = v; });
        __syncthreads();
        if (w < half)
            each([&](int e, float& v, bool mine) { if (mine) v += hand[w * NG + e]; });
    }
    if (w == 0) {
        float* out = partial + (size_t)blockIdx.x * NG;
        each([&](int e, float& v, bool mine) { if (mine) out[e] = v; });
    }
}

// grad[p] = (1/B) * (sum over row items of the MLP partials + sum over
// instances of the head partials), fixed order.
// Gradient = (sum of the row-tile partials of the MLP parameters, sum of
// the per-instance head partials) / count, in two fixed-order levels:
// chunk c of the partials -> gpart[c][p], then the chunks in order.
constexpr int kGradChunks = 64;

__global__ void k_grad_partial(const float* __restrict__ mlp_partial, int nitems,
                               const float* __restrict__ head_partial, int count,
                               float* __restrict__ gpart) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    const int c = blockIdx.y;
    if (p >= NP) return;
    float a = 0.0f;
    if (p < NG) {
        const int per = (nitems + kGradChunks - 1) / kGradChunks;
        const int lo = c * per, hi = min(nitems, lo + per);
        for (int it = lo; it < hi; ++it) a += mlp_partial[(size_t)it * NG + p];
    } else {
        const int q = p - NG;
        const int per = (count + kGradChunks - 1) / kGradChunks;
        const int lo = c * per, hi = min(count, lo + per);
        for (int t = lo; t < hi; ++t) a += head_partial[(size_t)t * (OUT * H + OUT) + q];
    }
    gpart[(size_t)c * NP + p] = a;
}

__global__ void k_grad_reduce(const float* __restrict__ gpart, int count, float* __restrict__ grad) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= NP) return;
    float a = 0.0f;
    for (int c = 0; c < kGradChunks; ++c) a += gpart[(size_t)c * NP + p];
    grad[p] = a / (float)count;
}

__global__ void k_adam(float* __restrict__ theta, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, float lr, float b1, float b2, float eps, float c1, float c2) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= NP) return;
    const float gp = g[p];
    const float mp = b1 * m[p] + (1.0f - b1) * gp;
    const float vp = b2 * v[p] + (1.0f - b2) * gp * gp;
    m[p] = mp;
    v[p] = vp;
    theta[p] -= lr * (mp / c1) / (sqrtf(vp / c2) + eps);
}

// ---------------------------------------------------------------- sampling
__device__ __forceinline__ float u01(uint32_t x) { return ((float)(x >> 9) + 0.5f) * 0x1p-23f; }

struct Rng {             // Philox-driven stream of uniforms for one sample
    uint64_t seed;
    uint32_t inst, s;
    uint32_t blk;
    uint32_t buf[4];
    int used;
    __device__ float next() {
        if (used == 4) {
            const U4 o = philox4x32_10(U4{s, 0x5EEDu, inst, 0x40000000u | blk},
                                       (uint32_t)seed, (uint32_t)(seed >> 32));
            buf[0] = o.x; buf[1] = o.y; buf[2] = o.z; buf[3] = o.w;
            ++blk;
            used = 0;
        }
        return u01(buf[used++]);
    }
    __device__ float normal() {
        const float a = next(), b = next();
        return sqrtf(-2.0f * logf(a)) * cospif(2.0f * b);
    }
    __device__ float gamma25() {   // Gamma(2) + Gamma(1/2) = Gamma(5/2)
        const float z = normal();
        return -logf(next() * next()) + 0.5f * z * z;
    }
};

// One thread per proposed direction.  Index s is uniform (the plain stream's
// direction s) when s % period == 0 with period = round(1/uniform_fraction),
// otherwise drawn from the mixture: component by its weight, w by Wood's
// rejection, a uniform tangent direction; c = G c_can.
__global__ __launch_bounds__(kBlock) void k_sample(const float* __restrict__ theta, const float* __restrict__ mvec,
                                                  const Frame* frames, int64_t S, uint64_t seed, uint32_t inst,
                                                  int period, float* __restrict__ dirs) {
    __shared__ Mixture mx;
    __shared__ float y[OUT], m[H];
    if (threadIdx.x < H) m[threadIdx.x] = mvec[threadIdx.x];
    __syncthreads();
    head(theta, m, mx, y);
    const Frame f = frames[0];
    for (int64_t s = blockIdx.x * (int64_t)kBlock + threadIdx.x; s < S; s += (int64_t)gridDim.x * kBlock) {
        float c[6];
        if (period > 0 && s % period == 0) {
            direction_f32<3>(seed, (uint64_t)s, inst, c);
        } else {
            Rng rng{seed, inst, (uint32_t)s, 0u, {0, 0, 0, 0}, 4};
            const float u = rng.next();
            int k = 0;
            float cum = expf(mx.logpi[0]);
            while (k < NC - 1 && u > cum) {
                ++k;
                cum += expf(mx.logpi[k]);
            }
            const float kap = mx.kappa[k];
            const float b = 5.0f / (2.0f * kap + sqrtf(4.0f * kap * kap + 25.0f));
            const float x0 = (1.0f - b) / (1.0f + b);
            const float cc = kap * x0 + 5.0f * logf(1.0f - x0 * x0);
            float w = 1.0f;
            for (int a = 0; a < kMaxRetry; ++a) {
                const float g1 = rng.gamma25(), g2 = rng.gamma25();
                const float z = g1 / (g1 + g2);
                const float ww = (1.0f - (1.0f + b) * z) / (1.0f - (1.0f - b) * z);
                const float uu = rng.next();
                if (kap * ww + 5.0f * logf(1.0f - x0 * ww) - cc >= logf(uu)) {
                    w = ww;
                    break;
                }
            }
            float tv[6], dot = 0.0f;
            for (int d = 0; d < 6; ++d) {
                tv[d] = rng.normal();
                dot += tv[d] * mx.mu[k][d];
            }
            float nt = 0.0f;
            for (int d = 0; d < 6; ++d) {
                tv[d] -= dot * mx.mu[k][d];
                nt += tv[d] * tv[d];
            }
            nt = nt > 0.0f ? 1.0f / sqrtf(nt) : 0.0f;
            const float sw = sqrtf(fmaxf(0.0f, 1.0f - w * w));
            float xc[6];
            for (int d = 0; d < 6; ++d) xc[d] = w * mx.mu[k][d] + sw * tv[d] * nt;
            // c = G c_can
            float nrm = 0.0f;
            for (int a2 = 0; a2 < 3; ++a2) {
                float re = 0.0f, im = 0.0f;
                for (int b2 = 0; b2 < 3; ++b2) {
                    const float gr = (float)f.g[2 * (3 * a2 + b2)], gi = (float)f.g[2 * (3 * a2 + b2) + 1];
                    re += gr * xc[2 * b2] - gi * xc[2 * b2 + 1];
                    im += gr * xc[2 * b2 + 1] + gi * xc[2 * b2];
                }
                c[2 * a2] = re;
                c[2 * a2 + 1] = im;
                nrm += re * re + im * im;
            }
            const float inv = 1.0f / sqrtf(nrm);
            for (int d = 0; d < 6; ++d) c[d] *= inv;
        }
        for (int d = 0; d < 6; ++d) dirs[s * 6 + d] = c[d];
    }
}

// Canonical targets: c_can = G^H c* (unit), written as 6 floats.
__global__ void k_targets(const float* __restrict__ cstar, const Frame* frames, int count,
                          float* __restrict__ out) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= count) return;
    const Frame f = frames[t];
    float nrm = 0.0f, o[6];
    for (int b = 0; b < 3; ++b) {
        float re = 0.0f, im = 0.0f;
        for (int a = 0; a < 3; ++a) {
            const float gr = (float)f.g[2 * (3 * a + b)], gi = -(float)f.g[2 * (3 * a + b) + 1];
            const float cr = cstar[t * 6 + 2 * a], ci = cstar[t * 6 + 2 * a + 1];
            re += gr * cr - gi * ci;
            im += gr * ci + gi * cr;
        }
        o[2 * b] = re;
        o[2 * b + 1] = im;
        nrm += re * re + im * im;
    }
    const float inv = 1.0f / sqrtf(nrm);
    for (int d = 0; d < 6; ++d) out[t * 6 + d] = o[d] * inv;
}

}  // namespace
}  // namespace lrqo

// ---------------------------------------------------------------- C ABI
struct lrqo_proposal {
    int device;
    int K;
    float* theta = nullptr;   // device parameters
    float* m = nullptr;       // Adam first moment
    float* v = nullptr;       // Adam second moment
    float* grad = nullptr;
    int64_t step = 0;
    // per-call scratch (grown on demand)
    void* scratch = nullptr;
    size_t scratch_bytes = 0;
};

namespace {

using lrqo::fail;

lrqo_status ensure_scratch(lrqo_proposal* p, size_t bytes) {
    if (bytes <= p->scratch_bytes) return LRQO_OK;
    if (p->scratch) {
        LRQO_HIP(hipDeviceSynchronize());
        LRQO_HIP(hipFree(p->scratch));
        p->scratch = nullptr;
        p->scratch_bytes = 0;
    }
    if (hipMalloc(&p->scratch, bytes) != hipSuccess) {
        (void)hipGetLastError();
        p->scratch = nullptr;
        return fail(LRQO_ENOMEM, "proposal scratch allocation failed");
    }
    p->scratch_bytes = bytes;
    return LRQO_OK;
}

struct RowPlan {
    std::vector<int32_t> inst;
    std::vector<int64_t> start;
    std::vector<int32_t> first;   // first item of each instance (+ end)
};

void plan_rows(int count, const int64_t* n, int tile, RowPlan& rp) {
    rp.inst.clear();
    rp.start.clear();
    rp.first.assign(count + 1, 0);
    for (int t = 0; t < count; ++t) {
        rp.first[t] = (int32_t)rp.inst.size();
        for (int64_t s = 0; s < n[t]; s += tile) {
            rp.inst.push_back(t);
            rp.start.push_back(s);
        }
    }
    rp.first[count] = (int32_t)rp.inst.size();
}

// The host-to-device data of one call in one copy: its pieces are carved one
// after another, so their device offsets (alignment padding included) lay
// out one host image of the whole range.
struct Upload {
    char* base = nullptr;
    std::vector<char> img;
    template <class T>
    T* take(lrqo::Carve& cv, const T* src, size_t count) {
        T* d = cv.take<T>(count);
        if (!base) base = reinterpret_cast<char*>(d);
        const size_t off = (size_t)(reinterpret_cast<char*>(d) - base), bytes = sizeof(T) * count;
        if (img.size() < off + bytes) img.resize(off + bytes);
        if (bytes) std::memcpy(img.data() + off, src, bytes);
        return d;
    }
    lrqo_status send(hipStream_t st) {
        using namespace lrqo;
        if (base && !img.empty())
            LRQO_HIP(hipMemcpyAsync(base, img.data(), img.size(), hipMemcpyHostToDevice, st));
        return LRQO_OK;
    }
};

// Shared by training and inference: frames, pooled embeddings.
struct FwdBufs {
    int64_t* voff;
    int64_t* n;
    lrqo::Frame* frames;
    int32_t* inst;
    int64_t* start;
    int32_t* first;
    float* partial;
    float* mvec;
    double* fwork;              // frame stages' partial sums
    int fsplits;
};

// b's descriptors (offsets, sizes, the row plan) are on the device already.
lrqo_status run_embed(lrqo_proposal* P, const float* V, int count, const RowPlan& rp, FwdBufs& b, hipStream_t st) {
    using namespace lrqo;
    launch_frames(V, b.voff, b.n, count, b.fsplits, P->K, b.frames, b.fwork, st);
    LRQO_HIP(hipGetLastError());
    RowItems items{b.inst, b.start, (int32_t)rp.inst.size()};
    // two blocks a CU (174 VGPRs), which keep the weights for all their items
    hipLaunchKernelGGL(k_mlp_fwd, dim3((unsigned)std::min<size_t>(rp.inst.size(), 512)), dim3(kBlock), 0, st, V, b.voff, b.n,
                       b.frames, P->theta, items, b.partial);
    LRQO_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_pool, dim3(count), dim3(H * kPoolGroups), 0, st, b.partial, b.first, b.n, count, b.mvec);
    LRQO_HIP(hipGetLastError());
    return LRQO_OK;
}

}  // namespace

extern "C" {

int32_t lrqo_proposal_param_count(void) { return lrqo::NP; }

lrqo_status lrqo_proposal_create(const double* init, int32_t K, lrqo_proposal** out) {
    using namespace lrqo;
    clear_error();
    if (!init || !out) return fail(LRQO_EINVAL, "null pointer argument");
    if (K < 2 || K > LRQO_MAX_K) return fail(LRQO_EINVAL, "K must be in [2, 255]");
    auto* P = new lrqo_proposal();
    P->K = K;
    if (hipGetDevice(&P->device) != hipSuccess) {
        delete P;
        return fail(LRQO_EDEVICE, "hipGetDevice failed");
    }
    std::vector<float> h(NP);
    for (int i = 0; i < NP; ++i) h[i] = (float)init[i];
    if (hipMalloc(&P->theta, sizeof(float) * NP) != hipSuccess || hipMalloc(&P->m, sizeof(float) * NP) != hipSuccess ||
        hipMalloc(&P->v, sizeof(float) * NP) != hipSuccess || hipMalloc(&P->grad, sizeof(float) * NP) != hipSuccess) {
        (void)hipGetLastError();
        lrqo_proposal_destroy(P);
        return fail(LRQO_ENOMEM, "proposal allocation failed");
    }
    LRQO_HIP(hipMemcpy(P->theta, h.data(), sizeof(float) * NP, hipMemcpyHostToDevice));
    LRQO_HIP(hipMemset(P->m, 0, sizeof(float) * NP));
    LRQO_HIP(hipMemset(P->v, 0, sizeof(float) * NP));
    LRQO_HIP(hipMemset(P->grad, 0, sizeof(float) * NP));
    *out = P;
    return LRQO_OK;
}

lrqo_status lrqo_proposal_destroy(lrqo_proposal* P) {
    if (!P) return LRQO_OK;
    (void)hipDeviceSynchronize();
    if (P->theta) (void)hipFree(P->theta);
    if (P->m) (void)hipFree(P->m);
    if (P->v) (void)hipFree(P->v);
    if (P->grad) (void)hipFree(P->grad);
    if (P->scratch) (void)hipFree(P->scratch);
    delete P;
    return LRQO_OK;
}

lrqo_status lrqo_proposal_get_state(lrqo_proposal* P, float* theta, float* m, float* v, int64_t* step) {
    using namespace lrqo;
    clear_error();
    if (!P || !theta) return fail(LRQO_EINVAL, "null pointer argument");
    LRQO_HIP(hipDeviceSynchronize());
    LRQO_HIP(hipMemcpy(theta, P->theta, sizeof(float) * NP, hipMemcpyDeviceToHost));
    if (m) LRQO_HIP(hipMemcpy(m, P->m, sizeof(float) * NP, hipMemcpyDeviceToHost));
    if (v) LRQO_HIP(hipMemcpy(v, P->v, sizeof(float) * NP, hipMemcpyDeviceToHost));
    if (step) *step = P->step;
    return LRQO_OK;
}

lrqo_status lrqo_proposal_set_state(lrqo_proposal* P, const float* theta, const float* m, const float* v,
                                    int64_t step) {
    using namespace lrqo;
    clear_error();
    if (!P || !theta) return fail(LRQO_EINVAL, "null pointer argument");
    if (step < 0) return fail(LRQO_EINVAL, "step must be >= 0");
    LRQO_HIP(hipMemcpy(P->theta, theta, sizeof(float) * NP, hipMemcpyHostToDevice));
    if (m) LRQO_HIP(hipMemcpy(P->m, m, sizeof(float) * NP, hipMemcpyHostToDevice));
    if (v) LRQO_HIP(hipMemcpy(P->v, v, sizeof(float) * NP, hipMemcpyHostToDevice));
    P->step = step;
    return LRQO_OK;
}

lrqo_status lrqo_proposal_train_step(lrqo_proposal* P, const float* V, int32_t count, const int64_t* v_offset,
                                     const int64_t* n, const float* targets, float lr, int32_t update,
                                     double* mean_loss, float* grad_out) {
    using namespace lrqo;
    clear_error();
    if (!P || !V || !v_offset || !n || !targets) return fail(LRQO_EINVAL, "null pointer argument");
    if (count < 1 || count > 65536) return fail(LRQO_EINVAL, "count must be in [1, 65536]");
    if (!(lr >= 0.0f) || lr > 1.0f) return fail(LRQO_EINVAL, "lr must be in [0, 1]");
    for (int t = 0; t < count; ++t)
        if (n[t] < 1 || n[t] > (1 << 24) || v_offset[t] < 0) return fail(LRQO_EINVAL, "bad n or v_offset");
    if (!is_device_pointer(V)) return fail(LRQO_EINVAL, "V is not device memory");
    RowPlan fp, bp;
    plan_rows(count, n, kBlock, fp);
    plan_rows(count, n, kRowTile, bp);
    // tiles of a wave and blocks of the backward pass
    const int tiles = (int)bp.inst.size();
    const int per_wave = (tiles + kBwdBlocks * kBwdWaves - 1) / (kBwdBlocks * kBwdWaves);
    const int bwd_blocks = (tiles + per_wave * kBwdWaves - 1) / (per_wave * kBwdWaves);
    CarveSize cs;
    cs.add<int64_t>(count);                  // uploaded: offsets, sizes,
    cs.add<int64_t>(count);
    cs.add<int32_t>(fp.inst.size());         // forward row plan,
    cs.add<int64_t>(fp.start.size());
    cs.add<int32_t>(count + 1);
    cs.add<float>((size_t)count * 6);        // host targets,
    cs.add<int32_t>(bp.inst.size());         // backward row plan
    cs.add<int64_t>(bp.start.size());
    cs.add<Frame>(count);
    cs.add<float>(fp.inst.size() * H);
    cs.add<float>((size_t)count * H);        // m
    cs.add<float>((size_t)count * H);        // dm
    cs.add<float>((size_t)count * 6);        // canonical targets
    cs.add<float>(count);                    // loss
    cs.add<float>((size_t)count * (OUT * H + OUT));
    cs.add<float>((size_t)bwd_blocks * NG);
    cs.add<float>((size_t)kGradChunks * NP);
    const int fsplits = frame_splits(count, *std::max_element(n, n + count));
    cs.add<double>(frame_work(count, fsplits));
    LRQO_TRY(ensure_scratch(P, cs.bytes));
    Carve cv(P->scratch);
    FwdBufs b{};
    Upload up;
    b.voff = up.take(cv, v_offset, count);
    b.n = up.take(cv, n, count);
    b.inst = up.take(cv, fp.inst.data(), fp.inst.size());
    b.start = up.take(cv, fp.start.data(), fp.start.size());
    b.first = up.take(cv, fp.first.data(), fp.first.size());
    float* tin = up.take(cv, targets, (size_t)count * 6);
    int32_t* inst_b = up.take(cv, bp.inst.data(), bp.inst.size());
    int64_t* start_b = up.take(cv, bp.start.data(), bp.start.size());
    b.frames = cv.take<Frame>(count);
    b.partial = cv.take<float>(fp.inst.size() * H);
    b.mvec = cv.take<float>((size_t)count * H);
    float* dm = cv.take<float>((size_t)count * H);
    float* tcan = cv.take<float>((size_t)count * 6);
    float* loss = cv.take<float>(count);
    float* headp = cv.take<float>((size_t)count * (OUT * H + OUT));
    float* mlpp = cv.take<float>((size_t)bwd_blocks * NG);
    float* gpart = cv.take<float>((size_t)kGradChunks * NP);
    b.fwork = cv.take<double>(frame_work(count, fsplits));
    b.fsplits = fsplits;
    hipStream_t st = current_stream();
    LRQO_TRY(up.send(st));
    LRQO_TRY(run_embed(P, V, count, fp, b, st));
    hipLaunchKernelGGL(k_targets, dim3((count + 255) / 256), dim3(256), 0, st, tin, b.frames, count, tcan);
    hipLaunchKernelGGL(k_head_loss, dim3(count), dim3(kBlock), 0, st, P->theta, b.mvec, tcan, P->K, loss, dm, headp);
    LRQO_HIP(hipGetLastError());
    RowItems items{inst_b, start_b, (int32_t)bp.inst.size()};
    hipLaunchKernelGGL(k_mlp_bwd, dim3((unsigned)bwd_blocks), dim3(kBwdBlock), 0, st, V, b.voff, b.n,
                       b.frames, P->theta, dm, items, per_wave, mlpp);
    LRQO_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_grad_partial, dim3((NP + 255) / 256, kGradChunks), dim3(256), 0, st, mlpp,
                       bwd_blocks, headp, count, gpart);
    hipLaunchKernelGGL(k_grad_reduce, dim3((NP + 255) / 256), dim3(256), 0, st, gpart, count, P->grad);
    LRQO_HIP(hipGetLastError());
    if (update) {
        P->step += 1;
        const float b1 = 0.9f, b2 = 0.999f;
        const float c1 = 1.0f - powf(b1, (float)P->step), c2 = 1.0f - powf(b2, (float)P->step);
        hipLaunchKernelGGL(k_adam, dim3((NP + 255) / 256), dim3(256), 0, st, P->theta, P->grad, P->m, P->v, lr, b1,
                           b2, 1e-8f, c1, c2);
        LRQO_HIP(hipGetLastError());
    }
    std::vector<float> hl(count);
    LRQO_HIP(hipMemcpyAsync(hl.data(), loss, sizeof(float) * count, hipMemcpyDeviceToHost, st));
    if (grad_out) LRQO_HIP(hipMemcpyAsync(grad_out, P->grad, sizeof(float) * NP, hipMemcpyDeviceToHost, st));
    LRQO_HIP(hipStreamSynchronize(st));
    if (mean_loss) {
        double s = 0.0;
        for (float x : hl) s += x;
        *mean_loss = s / count;
    }
    return LRQO_OK;
}

lrqo_status lrqo_proposal_sample(lrqo_proposal* P, const float* V, int64_t n, int64_t S, uint64_t seed,
                                 uint32_t instance, float uniform_fraction, float* dirs) {
    using namespace lrqo;
    clear_error();
    if (!P || !V || !dirs) return fail(LRQO_EINVAL, "null pointer argument");
    if (n < 1 || n > (1 << 24)) return fail(LRQO_EINVAL, "n must be in [1, 2^24]");
    if (S < 1 || S > (int64_t)0xFFFFFFFFll) return fail(LRQO_EINVAL, "S must be in [1, 2^32-1]");
    if (!(uniform_fraction >= 0.0f && uniform_fraction <= 1.0f))
        return fail(LRQO_EINVAL, "uniform_fraction must be in [0, 1]");
    if (!is_device_pointer(V) || !is_device_pointer(dirs)) return fail(LRQO_EINVAL, "V and dirs must be device memory");
    RowPlan fp;
    const int64_t zero = 0;
    plan_rows(1, &n, kBlock, fp);
    CarveSize cs;
    cs.add<int64_t>(1);                      // uploaded: offset, size, row plan
    cs.add<int64_t>(1);
    cs.add<int32_t>(fp.inst.size());
    cs.add<int64_t>(fp.start.size());
    cs.add<int32_t>(2);
    cs.add<Frame>(1);
    cs.add<float>(fp.inst.size() * H);
    cs.add<float>(H);
    const int fsplits = frame_splits(1, n);
    cs.add<double>(frame_work(1, fsplits));
    LRQO_TRY(ensure_scratch(P, cs.bytes));
    Carve cv(P->scratch);
    FwdBufs b{};
    Upload up;
    b.voff = up.take(cv, &zero, 1);
    b.n = up.take(cv, &n, 1);
    b.inst = up.take(cv, fp.inst.data(), fp.inst.size());
    b.start = up.take(cv, fp.start.data(), fp.start.size());
    b.first = up.take(cv, fp.first.data(), fp.first.size());
    b.frames = cv.take<Frame>(1);
    b.partial = cv.take<float>(fp.inst.size() * H);
    b.mvec = cv.take<float>(H);
    b.fwork = cv.take<double>(frame_work(1, fsplits));
    b.fsplits = fsplits;
    hipStream_t st = current_stream();
    LRQO_TRY(up.send(st));
    LRQO_TRY(run_embed(P, V, 1, fp, b, st));
    const int period = uniform_fraction > 0.0f ? std::max(1, (int)lrintf(1.0f / uniform_fraction)) : 0;
    const unsigned blocks = (unsigned)std::min<int64_t>((S + kBlock - 1) / kBlock, 4096);
    hipLaunchKernelGGL(k_sample, dim3(blocks), dim3(kBlock), 0, st, P->theta, b.mvec, b.frames, S, seed, instance,
                       period, dirs);
    LRQO_HIP(hipGetLastError());
    LRQO_HIP(hipStreamSynchronize(st));
    return LRQO_OK;
}

lrqo_status lrqo_proposal_frame(lrqo_proposal* P, const float* V, int64_t n, double* frame_out) {
    using namespace lrqo;
    clear_error();
    if (!P || !V || !frame_out) return fail(LRQO_EINVAL, "null pointer argument");
    if (n < 1 || n > (1 << 24)) return fail(LRQO_EINVAL, "n must be in [1, 2^24]");
    if (!is_device_pointer(V)) return fail(LRQO_EINVAL, "V is not device memory");
    const int fsplits = frame_splits(1, n);
    CarveSize cs;
    cs.add<int64_t>(2);
    cs.add<Frame>(1);
    cs.add<double>(frame_work(1, fsplits));
    LRQO_TRY(ensure_scratch(P, cs.bytes));
    Carve cv(P->scratch);
    int64_t* d = cv.take<int64_t>(2);
    Frame* fr = cv.take<Frame>(1);
    double* work = cv.take<double>(frame_work(1, fsplits));
    const int64_t h[2] = {0, n};
    hipStream_t st = current_stream();
    LRQO_HIP(hipMemcpyAsync(d, h, sizeof h, hipMemcpyHostToDevice, st));
    launch_frames(V, d, d + 1, 1, fsplits, P->K, fr, work, st);
    LRQO_HIP(hipGetLastError());
    Frame hf;
    LRQO_HIP(hipMemcpyAsync(&hf, fr, sizeof hf, hipMemcpyDeviceToHost, st));
    LRQO_HIP(hipStreamSynchronize(st));
    for (int e = 0; e < 18; ++e) frame_out[e] = hf.g[e];
    frame_out[18] = hf.s;
    return LRQO_OK;
}

}  // extern "C"
