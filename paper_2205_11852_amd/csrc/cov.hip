// Sample covariances over mocks and the linear construction (Sect. 2.2, 2.3),
// plus the positive-definiteness check of the result (Sect. 3).
//
//   mean (float64, two passes)  ->  deviations  ->  Cov_e = D_e^T D_e / (N-1)
//   for the three estimates e = (D,R1), (D,R2), (D,R1uR2)
//   ->  C^a = (Cov_0 + Cov_1)/2, C^b = Cov_2,
//       A = (M_b C^b - M_a C^a)/(M_b - M_a), B = M_a M_b (C^a - C^b)/(M_b - M_a)
//       (Eq. CovAB; 2C^b - C^a and 2 M_a (C^a - C^b) at M_b = 2 M_a),
//       C = A + B/M                                    (float64)
//   ->  Cholesky and eigenvalue extremes of each block of C (float64).
//
// The products D^T D run as float64 MFMA (v_mfma_f64_16x16x4) or float32 MFMA
// (v_mfma_f32_32x32x2f32) with float32 accumulation, by default over chunks
// of 256 mocks whose partial sums are added in float64 (LC_ACC32: over all
// mocks in float32).
#include <algorithm>
#include <cfloat>
#include <chrono>
#include <cmath>
#include <new>
#include <vector>

#include "lc_internal.hpp"

namespace lc {

// ---------------------------------------------------------------------------
// mean and deviations
// ---------------------------------------------------------------------------
static int nblocks(int64_t n, int threads, int cap = 4096) {
    return int(std::max<int64_t>(1, std::min<int64_t>((n + threads - 1) / threads, cap)));
}

constexpr int kMeanRows = 64;

// partial[c][j] = sum of xi[n][j] over rows n of chunk c (j < 3P)
__global__ void k_mean_partial(const double* __restrict__ xi, int64_t n_mock, int64_t W3,
                               double* __restrict__ partial) {
    const int64_t j = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
    if (j >= W3) return;
    const int64_t n0 = int64_t(blockIdx.y) * kMeanRows;
    const int64_t n1 = min(n0 + kMeanRows, n_mock);
    double s = 0.0;
    for (int64_t n = n0; n < n1; n++) s += xi[n * W3 + j];
    partial[int64_t(blockIdx.y) * W3 + j] = s;
}

__global__ void k_mean_final(const double* __restrict__ partial, int64_t nchunk, int64_t W3, int64_t n_mock,
                             double* __restrict__ mean) {
    const int64_t j = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
    if (j >= W3) return;
    double s = 0.0;
    for (int64_t c = 0; c < nchunk; c++) s += partial[c * W3 + j];
    mean[j] = s / double(n_mock);
}

// dev32[e][n][p] (ld = Ppad, Npad rows, zero padded) = float(xi - mean)
__global__ void k_dev32(const double* __restrict__ xi, const double* __restrict__ mean, int64_t n_mock,
                        int64_t P, int64_t ne, int64_t Npad, int64_t Ppad, float* __restrict__ dev) {
    const int64_t tot = ne * Npad * Ppad;
    for (int64_t t = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; t < tot;
         t += int64_t(gridDim.x) * blockDim.x) {
        const int64_t p = t % Ppad;
        const int64_t r = t / Ppad;
        const int64_t n = r % Npad;
        const int64_t e = r / Npad;
        float v = 0.0f;
        if (n < n_mock && p < P) v = float(xi[n * ne * P + e * P + p] - mean[e * P + p]);
        dev[t] = v;
    }
}

// ---------------------------------------------------------------------------
// SYRK, float64: C = D^T D / (N - 1) over lower-triangle tiles of 64 x 64,
// four waves of 32 x 32, each 2 x 2 blocks of v_mfma_f64_16x16x4 (operand
// layout: lane l supplies A[i = l % 16][k = l / 16] and B[k = l / 16][j =
// l % 16]; register r of lane l holds D[i = l / 16 + 4 r][j = l % 16]).  The
// deviations are formed while a slab of 16 mocks is staged, and the next
// slab's loads are in flight over the products.  What bounds short vectors is
// blocks: 540 elements give 45 tiles, so the mocks are split over gridDim.z
// as well and the parts summed in order (k_syrk_sum).  3000 mocks of 540 x 3:
// 0.80 ms from float64 VALU products of a stored copy of the deviations,
// 0.175 ms here; error against extended precision 1.5e-15 then, 1.6e-16 in
// eight parts.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void tri_tile(int t, int& ti, int& tj) {
    // t enumerates (ti, tj) with tj <= ti
    ti = int((sqrt(8.0 * t + 1.0) - 1.0) * 0.5);
    while ((ti + 1) * (ti + 2) / 2 <= t) ti++;
    while (ti * (ti + 1) / 2 > t) ti--;
    tj = t - ti * (ti + 1) / 2;
}

typedef double f64x4 __attribute__((ext_vector_type(4)));
constexpr int kST = 64;          // tile
constexpr int kSK = 16;          // mocks per slab
constexpr int kSLd = kST + 16;   // row stride in LDS: the two rows a half wave reads lie in different banks

// Element (i, j) of tile (ti, tj) held in register q of thread t.
__device__ __forceinline__ void syrk64_at(int q, int t, int& i, int& j) {
    const int lane = t & 63, wid = t >> 6, u = q >> 3, v = (q >> 2) & 1, r = q & 3;
    i = (wid >> 1) * 32 + 16 * u + (lane >> 4) + 4 * r;
    j = (wid & 1) * 32 + 16 * v + (lane & 15);
}

// x: element p of estimate e of mock n at x[n ld + e P + p].  split: mocks per
// gridDim.z part (a multiple of kSK); part != NULL: raw sums go there.
__global__ __launch_bounds__(256) void k_syrk64(const double* __restrict__ x, int64_t ld,
                                                const double* __restrict__ mean, int64_t n_mock, int64_t P,
                                                int64_t split, double denom, double* __restrict__ part,
                                                double* __restrict__ cov) {
    __shared__ double As[2][kSK][kSLd];
    __shared__ double Bs[2][kSK][kSLd];
    const int e = blockIdx.y;
    int ti, tj;
    tri_tile(blockIdx.x, ti, tj);
    const int64_t i0 = int64_t(ti) * kST, j0 = int64_t(tj) * kST;
    const int64_t nb = int64_t(blockIdx.z) * split, ne = min(nb + split, n_mock);
    // this thread stages column c of the tile, mocks k4, k4 + 4, ... of a slab
    const int c = threadIdx.x & 63, k4 = threadIdx.x >> 6;
    const bool ai = i0 + c < P, bj = j0 + c < P;
    const double* xa = x + e * P + (ai ? i0 + c : 0);
    const double* xb = x + e * P + (bj ? j0 + c : 0);
    const double ma = ai ? mean[e * P + i0 + c] : 0.0, mb = bj ? mean[e * P + j0 + c] : 0.0;
    double pa[kSK / 4], pb[kSK / 4];
    auto load = [&](int64_t n0) {
#pragma unroll
        for (int q = 0; q < kSK / 4; q++) {
            const int64_t n = n0 + k4 + 4 * q;
            pa[q] = ai && n < ne ? xa[n * ld] - ma : 0.0;
            pb[q] = bj && n < ne ? xb[n * ld] - mb : 0.0;
        }
    };
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int wr = (wid >> 1) * 32, wc = (wid & 1) * 32, lc = lane & 15, lk = lane >> 4;
    f64x4 acc[2][2] = {};
    load(nb);
    int buf = 0;
    for (int64_t n0 = nb; n0 < ne; n0 += kSK, buf ^= 1) {
#pragma unroll
        for (int q = 0; q < kSK / 4; q++) {
            As[buf][k4 + 4 * q][c] = pa[q];
            Bs[buf][k4 + 4 * q][c] = pb[q];
        }
        __syncthreads();  // (the other buffer was read before the last barrier)
        load(n0 + kSK);
#pragma unroll
        for (int k = 0; k < kSK; k += 4) {
            double a[2], b[2];
#pragma unroll
            for (int u = 0; u < 2; u++) {
                a[u] = As[buf][k + lk][wr + 16 * u + lc];
                b[u] = Bs[buf][k + lk][wc + 16 * u + lc];
            }
#pragma unroll
            for (int u = 0; u < 2; u++)
#pragma unroll
                for (int v = 0; v < 2; v++)
                    acc[u][v] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b[v], acc[u][v], 0, 0, 0);
        }
    }
    const int64_t tile = (int64_t(blockIdx.z) * gridDim.y + e) * gridDim.x + blockIdx.x;
    double* C = cov + int64_t(e) * P * P;
#pragma unroll
    for (int q = 0; q < 16; q++) {
        const double s = acc[q >> 3][(q >> 2) & 1][q & 3];
        if (part) {
            part[(tile * 16 + q) * 256 + threadIdx.x] = s;
            continue;
        }
        int il, jl;
        syrk64_at(q, threadIdx.x, il, jl);
        const int64_t i = i0 + il, j = j0 + jl;
        if (i < P && j < P) {
            C[i * P + j] = s / denom;
            if (ti != tj) C[j * P + i] = s / denom;
        }
    }
}

// Sums the nz parts of every tile in order.  PREC 64: k_syrk64's tiles of 16
// registers a thread; 32: k_syrk32's of 64.
template <int PREC>
__global__ __launch_bounds__(256) void k_syrk_sum(const double* __restrict__ part, int nz, int64_t P, double denom,
                                                  double* __restrict__ cov);

// ---------------------------------------------------------------------------
// SYRK, float32 MFMA: 128x128 tile per block, 2x2 waves of 64x64,
// each wave 2x2 blocks of v_mfma_f32_32x32x2f32.
// Operand layout of the 32x32x2 instruction (wave64): lane l supplies
// A[i = l%32][k = l/32] and B[k = l/32][j = l%32]; accumulator register r of
// lane l holds D[i = 8*(r/4) + 4*(l/32) + r%4][j = l%32].
// ---------------------------------------------------------------------------
typedef float f32x16 __attribute__((ext_vector_type(16)));
constexpr int kMT = 128;    // tile
constexpr int kKT = 32;     // rows per LDS slab
constexpr int kKC = 256;    // rows per float32 accumulation chunk

__device__ __forceinline__ void syrk32_at(int q, int t, int& i, int& j) {
    const int lane = t & 63, wid = t >> 6, a = q >> 5, b = (q >> 4) & 1, r = q & 15;
    i = (wid >> 1) * 64 + a * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
    j = (wid & 1) * 64 + b * 32 + (lane & 31);
}

// kc: rows summed in the float32 accumulators before they are added into
// the float64 ones (a multiple of kKT; Npad or more: float32 throughout).
// split: rows per gridDim.z part, a multiple of kc; part != NULL: the parts'
// raw sums go there (k_syrk_sum adds them).  A slab's loads are in flight
// over the products of the one before it, and two blocks fit on a CU (the
// float64 accumulators leave room for no more; with one, 1.77 ms).  5000
// mocks of 2120 x 3: 1.62 ms with 459 blocks and a slab's loads waited for,
// 1.26 ms and 0.08 ms for the sums in two parts here.
__global__ __launch_bounds__(256, 2) void k_syrk32(const float* __restrict__ dev, int64_t Npad, int64_t Ppad,
                                                int64_t P, int64_t kc, int64_t split, double denom,
                                                double* __restrict__ part, double* __restrict__ cov) {
    __shared__ __align__(16) float As[kKT][kMT];
    __shared__ __align__(16) float Bs[kKT][kMT];
    const int e = blockIdx.y;
    int ti, tj;
    tri_tile(blockIdx.x, ti, tj);
    const int64_t i0 = int64_t(ti) * kMT, j0 = int64_t(tj) * kMT;
    const float* D = dev + int64_t(e) * Npad * Ppad;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int wr = wid >> 1, wc = wid & 1;
    const int li = lane & 31, lk = lane >> 5;
    f32x16 acc[2][2];
    double dacc[2][2][16];
    for (int a = 0; a < 2; a++)
        for (int b = 0; b < 2; b++) {
            for (int r = 0; r < 16; r++) {
                acc[a][b][r] = 0.0f;
                dacc[a][b][r] = 0.0;
            }
        }
    const int64_t nb = int64_t(blockIdx.z) * split, ne = min(nb + split, Npad);
    // this thread stages columns c4 .. c4 + 3 of rows k8, k8 + 8, ...
    const int c4 = (threadIdx.x & 31) * 4, k8 = threadIdx.x >> 5;
    float4 va[kKT / 8], vb[kKT / 8];
    auto load = [&](int64_t n0) {
#pragma unroll
        for (int q = 0; q < kKT / 8; q++) {
            const float* row = D + (n0 + k8 + 8 * q) * Ppad + c4;
            va[q] = *reinterpret_cast<const float4*>(row + i0);
            vb[q] = *reinterpret_cast<const float4*>(row + j0);
        }
    };
    load(nb);
    int64_t since = 0;
    for (int64_t n0 = nb; n0 < ne; n0 += kKT) {
#pragma unroll
        for (int q = 0; q < kKT / 8; q++) {
            *reinterpret_cast<float4*>(&As[k8 + 8 * q][c4]) = va[q];
            *reinterpret_cast<float4*>(&Bs[k8 + 8 * q][c4]) = vb[q];
        }
        __syncthreads();
        if (n0 + kKT < ne) load(n0 + kKT);
#pragma unroll
        for (int ks = 0; ks < kKT; ks += 2) {
            float a0 = As[ks + lk][wr * 64 + li];
            float a1 = As[ks + lk][wr * 64 + 32 + li];
            float b0 = Bs[ks + lk][wc * 64 + li];
            float b1 = Bs[ks + lk][wc * 64 + 32 + li];
            acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, b0, acc[0][0], 0, 0, 0);
            acc[0][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, b1, acc[0][1], 0, 0, 0);
            acc[1][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, b0, acc[1][0], 0, 0, 0);
            acc[1][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, b1, acc[1][1], 0, 0, 0);
        }
        __syncthreads();
        since += kKT;
        if (since == kc || n0 + kKT >= ne) {
            for (int a = 0; a < 2; a++)
                for (int b = 0; b < 2; b++)
                    for (int r = 0; r < 16; r++) {
                        dacc[a][b][r] += double(acc[a][b][r]);
                        acc[a][b][r] = 0.0f;
                    }
            since = 0;
        }
    }
    const int64_t tile = (int64_t(blockIdx.z) * gridDim.y + e) * gridDim.x + blockIdx.x;
    double* C = cov + int64_t(e) * P * P;
#pragma unroll
    for (int q = 0; q < 64; q++) {
        const double s = dacc[q >> 5][(q >> 4) & 1][q & 15];
        if (part) {
            part[(tile * 64 + q) * 256 + threadIdx.x] = s;
            continue;
        }
        int il, jl;
        syrk32_at(q, threadIdx.x, il, jl);
        const int64_t i = i0 + il, j = j0 + jl;
        if (i < P && j < P) {
            const double v = s / denom;
            C[i * P + j] = v;
            if (ti != tj) C[j * P + i] = v;
        }
    }
}

template <int PREC>
__global__ __launch_bounds__(256) void k_syrk_sum(const double* __restrict__ part, int nz, int64_t P, double denom,
                                                  double* __restrict__ cov) {
    constexpr int NQ = PREC == 64 ? 16 : 64, T = PREC == 64 ? kST : kMT;
    const int e = blockIdx.y;
    int ti, tj;
    tri_tile(blockIdx.x, ti, tj);
    double* C = cov + int64_t(e) * P * P;
    const int64_t zs = int64_t(gridDim.y) * gridDim.x * NQ * 256;
    for (int q = blockIdx.z; q < NQ; q += gridDim.z) {
        const double* src = part + ((int64_t(e) * gridDim.x + blockIdx.x) * NQ + q) * 256 + threadIdx.x;
        double s = src[0];
        for (int z = 1; z < nz; z++) s += src[z * zs];
        int il, jl;
        if (PREC == 64) syrk64_at(q, threadIdx.x, il, jl);
        else syrk32_at(q, threadIdx.x, il, jl);
        const int64_t i = int64_t(ti) * T + il, j = int64_t(tj) * T + jl;
        if (i < P && j < P) {
            const double v = s / denom;
            C[i * P + j] = v;
            if (ti != tj) C[j * P + i] = v;
        }
    }
}

// Parts the mocks are split into: about four blocks per CU where whole tiles
// give fewer than two, each part a whole number of `unit` rows and at least
// four of them, at most 16 parts.  (595 tiles of 200 mocks: 49 + 16 us in two
// parts and their sum, 50 us whole.)
static int64_t syrk_split(int64_t rows, int64_t unit, int64_t blocks, int n_cu, int& nz) {
    const int64_t units = (rows + unit - 1) / unit;
    const int64_t want = blocks >= 2 * n_cu ? 1 : std::min<int64_t>({4 * n_cu / blocks, units / 4, 16});
    const int64_t per = (units + std::max<int64_t>(want, 1) - 1) / std::max<int64_t>(want, 1);
    nz = int((units + per - 1) / per);
    return per * unit;
}

// cov[e] = the sample covariance of estimate e of ne, in float64.
static lc_status syrk_fp64(DeviceCtx* ctx, const double* x, const double* mean, int64_t N, int64_t P, int ne,
                           double denom, double* cov, hipStream_t s) {
    const int64_t T = (P + kST - 1) / kST, nt = T * (T + 1) / 2;
    int nz;
    const int64_t split = syrk_split(N, kSK, nt * ne, ctx->n_cu, nz);
    DevBuf<double> part;
    if (nz > 1) LC_TRY(part.alloc(size_t(nz) * ne * nt * kST * kST, s));
    k_syrk64<<<dim3(unsigned(nt), ne, nz), 256, 0, s>>>(x, ne * P, mean, N, P, split, denom, part.get(), cov);
    if (nz > 1) k_syrk_sum<64><<<dim3(unsigned(nt), ne, 4), 256, 0, s>>>(part.get(), nz, P, denom, cov);
    return LC_OK;
}

// The same from float32 deviations and MFMA products.
static lc_status syrk_fp32(DeviceCtx* ctx, const double* x, const double* mean, int64_t N, int64_t P, int ne,
                           bool acc32, double denom, double* cov, hipStream_t s) {
    const int64_t Npad = (N + kKT - 1) / kKT * kKT;
    const int64_t Ppad = (P + kMT - 1) / kMT * kMT;
    DevBuf<float> dev;
    LC_TRY(dev.alloc(size_t(ne * Npad * Ppad), s));
    k_dev32<<<nblocks(ne * Npad * Ppad, 256, 65536), 256, 0, s>>>(x, mean, N, P, ne, Npad, Ppad, dev.get());
    const int64_t T = Ppad / kMT, nt = T * (T + 1) / 2;
    int nz = 1;
    int64_t split = Npad;
    if (!acc32) split = syrk_split(Npad, kKC, nt * ne, ctx->n_cu, nz);
    DevBuf<double> part;
    if (nz > 1) LC_TRY(part.alloc(size_t(nz) * ne * nt * kMT * kMT, s));
    k_syrk32<<<dim3(unsigned(nt), ne, nz), 256, 0, s>>>(dev.get(), Npad, Ppad, P, acc32 ? INT64_MAX : int64_t(kKC),
                                                        split, denom, part.get(), cov);
    if (nz > 1) k_syrk_sum<32><<<dim3(unsigned(nt), ne, 16), 256, 0, s>>>(part.get(), nz, P, denom, cov);
    return LC_OK;
}

// ---------------------------------------------------------------------------
// linear construction (float64)
// ---------------------------------------------------------------------------
__global__ void k_combine(const double* __restrict__ cov, int64_t PP, double m_a, double m_b, double M, int m_inf,
                          double* __restrict__ A, double* __restrict__ B, double* __restrict__ C) {
#pragma clang fp contract(off)
    // Eq. CovAB: A = (M_b C^b - M_a C^a)/(M_b - M_a), B = M_a M_b/(M_b - M_a) (C^a - C^b);
    // at M_b = 2 M_a (Eq. LCdef) the forms 2 C^b - C^a and 2 M_a (C^a - C^b)
    // are used as written (the general quotient would round differently
    // unless M_a is a power of two)
    const double dm = m_b - m_a;
    const bool paper = (m_b == 2.0 * m_a);
    const double kb = paper ? 2.0 * m_a : (m_a * m_b) / dm;
    for (int64_t t = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; t < PP;
         t += int64_t(gridDim.x) * blockDim.x) {
        const double ca = 0.5 * (cov[t] + cov[PP + t]);
        const double cb = cov[2 * PP + t];
        const double a = paper ? 2.0 * cb - ca : (m_b * cb - m_a * ca) / dm;
        const double b = kb * (ca - cb);
        A[t] = a;
        B[t] = b;
        C[t] = m_inf ? a : a + b / M;
    }
}

// ---------------------------------------------------------------------------
// Frobenius norms for the float32-vs-float64 report
// ---------------------------------------------------------------------------
__global__ void k_frob(const double* __restrict__ x, const double* __restrict__ y, int64_t n,
                       double* __restrict__ part) {
    __shared__ double sd[256], sy[256];
    double d = 0.0, s = 0.0;
    for (int64_t t = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; t < n; t += int64_t(gridDim.x) * blockDim.x) {
        const double df = x[t] - y[t];
        d += df * df;
        s += y[t] * y[t];
    }
    sd[threadIdx.x] = d;
    sy[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) {
            sd[threadIdx.x] += sd[threadIdx.x + o];
            sy[threadIdx.x] += sy[threadIdx.x + o];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x] = sd[0];
        part[2 * blockIdx.x + 1] = sy[0];
    }
}

// ---------------------------------------------------------------------------
// check: copy a diagonal block, Cholesky, Householder tridiagonalisation,
// bisection on the tridiagonal for the extreme eigenvalues and the number of
// negative ones.  Work matrix: n x n row-major, ld = n.
// ---------------------------------------------------------------------------
struct CheckFlags {
    int nan_seen;
    int chol_fail;
};

__global__ void k_copy_block(const double* __restrict__ C, int64_t P, int64_t off, int64_t n,
                             double* __restrict__ W, CheckFlags* fl) {
    for (int64_t t = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; t < n * n; t += int64_t(gridDim.x) * blockDim.x) {
        const int64_t i = t / n, j = t % n;
        const double v = C[(off + i) * P + off + j];
        W[t] = v;
        if (v != v) fl->nan_seen = 1;
    }
}

__global__ void k_zero_flags(CheckFlags* fl, int n) {
    if (int(threadIdx.x) < n) {
        fl[threadIdx.x].nan_seen = 0;
        fl[threadIdx.x].chol_fail = 0;
    }
}

// Cholesky factorisation of the lower triangle, 32 columns at a time: a panel
// launch, then the trailing update.  The chain of panels bounds it, so a
// panel is one launch of single waves: every block factors the 32 x 32
// diagonal block for itself (row i in lane i's registers, the column's other
// elements through readlane) and with the same broadcast elements solves 64
// rows below it, one per lane: 20 us, where a launch for the diagonal block
// (one thread forming each pivot) took 46 us and one for the rows 52 us.  The
// update is a contraction over the panel's 32 columns and runs on the matrix
// cores: 13 us, 24 us before.  2000 rows: 8.0 ms before, 2.1 ms now.  Square
// roots and quotients are the correctly rounded ones (the hardware's estimate of
// 1 / sqrt and two Newton steps in their place: 17 us, errors of an ulp or two,
// and a NaN from an infinite pivot).
constexpr int kNB = 32;

__device__ __forceinline__ double readlane_f64(double x, int l) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), l),
                            __builtin_amdgcn_readlane(__double2loint(x), l));
}

// Columns [k0, k0 + nb) of L from the updated W: the rows below the diagonal
// block, 64 per block.  Every block reads the diagonal block, and blocks start
// at any time (one after another where other work holds the CUs), so none may
// store its factor over it: the factor stays in registers, and nothing after
// this launch reads the diagonal block again.
// FULL: nb = 32; the last panel may be narrower and has no rows below it.
template <bool FULL>
__global__ __launch_bounds__(64) void k_potrf_panel(double* __restrict__ W, int64_t n, int64_t k0, int nb,
                                                    CheckFlags* fl) {
    if (fl->chol_fail || fl->nan_seen) return;
    const int lane = threadIdx.x;
    // row `lane` of the diagonal block (lanes 32 to 63 repeat it; rows and
    // columns past nb: identity)
    const int li = lane & (kNB - 1);
    double r[kNB], x[kNB];
    const double* const own = W + (k0 + (FULL || li < nb ? li : 0)) * n + k0;
#pragma unroll
    for (int c = 0; c < kNB; c++) r[c] = FULL || (li < nb && c < nb) ? own[c] : (li == c ? 1.0 : 0.0);
    // this lane's row below (past the last one, the last one again)
    const int64_t row = k0 + kNB + blockIdx.x * int64_t(64) + lane;
    double* const dst = W + (row < n ? row : n - 1) * n + k0;
#pragma unroll
    for (int c = 0; c < kNB; c++) x[c] = FULL ? dst[c] : 0.0;
    bool bad = false;
#pragma unroll
    for (int j = 0; j < kNB; j++) {
        if (!FULL && j >= nb) continue;  // (identity)
        const double d = readlane_f64(r[j], j);
        bad |= !(d > 0.0);
        const double s = sqrt(d);
        const double l = r[j] / s;
        r[j] = l;
        x[j] /= s;
#pragma unroll
        for (int c = j + 1; c < kNB; c++) {
            const double lc = readlane_f64(l, c);
            r[c] -= l * lc;
            x[c] -= x[j] * lc;
        }
    }
    if (bad) {  // the same in every block
        if (blockIdx.x == 0 && lane == 0) fl->chol_fail = 1;
        return;
    }
    if (FULL && row < n) {
#pragma unroll
        for (int c = 0; c < kNB; c++) dst[c] = x[c];
    }
}

// Trailing update of the lower triangle: A22 -= L21 L21^T, for a full panel
// of 32 columns.  64 x 64 tiles, four waves of 32 x 32, each 2 x 2 blocks of
// v_mfma_f64_16x16x4: lane l supplies A[i = l % 16][k = l / 16] and
// B[k = l / 16][j = l % 16]; register r of lane l holds
// D[i = l / 16 + 4 r][j = l % 16].
__global__ __launch_bounds__(256) void k_potrf_update(double* __restrict__ W, int64_t n, int64_t k0,
                                                      const CheckFlags* fl) {
    if (fl->chol_fail || fl->nan_seen) return;
    __shared__ double Li[64][kNB + 1];
    __shared__ double Lj[64][kNB + 1];
    const int64_t base = k0 + kNB;
    int ti, tj;
    tri_tile(blockIdx.x, ti, tj);
    const int64_t i0 = base + int64_t(ti) * 64, j0 = base + int64_t(tj) * 64;
    for (int t = threadIdx.x; t < 64 * kNB; t += 256) {
        const int r = t / kNB, q = t % kNB;
        Li[r][q] = (i0 + r < n) ? W[(i0 + r) * n + k0 + q] : 0.0;
        Lj[r][q] = (j0 + r < n) ? W[(j0 + r) * n + k0 + q] : 0.0;
    }
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int wr = (wid >> 1) * 32, wc = (wid & 1) * 32, lc = lane & 15, lk = lane >> 4;
    __syncthreads();
    f64x4 acc[2][2] = {};
#pragma unroll
    for (int q = 0; q < kNB; q += 4) {
        double a[2], b[2];
#pragma unroll
        for (int u = 0; u < 2; u++) {
            a[u] = Li[wr + 16 * u + lc][q + lk];
            b[u] = Lj[wc + 16 * u + lc][q + lk];
        }
#pragma unroll
        for (int u = 0; u < 2; u++)
#pragma unroll
            for (int v = 0; v < 2; v++)
                acc[u][v] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b[v], acc[u][v], 0, 0, 0);
    }
#pragma unroll
    for (int u = 0; u < 2; u++)
#pragma unroll
        for (int v = 0; v < 2; v++)
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const int64_t i = i0 + wr + 16 * u + lk + 4 * r, j = j0 + wc + 16 * v + lc;
                if (i < n && j <= i) W[i * n + j] -= acc[u][v][r];
            }
}

// Sum of x over the block (every thread gets the total).
// Wave sums by butterfly shuffles, then one exchange of the per-wave sums
// through `red` (blockDim.x a multiple of 64, at most 1024): two barriers.
__device__ __forceinline__ double block_sum(double x, double* red) {
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
    const int nw = int(blockDim.x >> 6);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
    __syncthreads();
    double r = 0.0;
    for (int w = 0; w < nw; w++) r += red[w];
    __syncthreads();
    return r;
}

// Householder tridiagonalisation of the symmetric block, one launch per
// column k = 0 .. n-3.  Step k reflects row k of the trailing matrix onto
// alpha e1 (v = x - alpha e1, tau = 2 / v.v), forms p = tau A22 v and the
// rank-2 update A22 -= v w^T + w v^T with w = p - K v, K = (tau/2) v.p.
// The launch for column k applies the update of column k-1 as it goes:
// every wave updates its own row of A22(k) while reading it (and writes it
// back), and every block updates row k on the fly from the old row and
// step k-1's v and p, so no block waits for another.  Indices of the
// pending update run over A22(k-1), whose row and column 0 are row and
// column k of W.
struct HhPending {
    const double* v;        // [m + 1] Householder vector of step k-1 (NULL: none pending)
    const double* p;        // [m + 1] tau A v of step k-1
    const double* tau;
    const double* vp_part;  // partial sums of v.p, n1 of them
    int64_t n1;
};

// K of the pending update: the same ordered reduction in every block.
__device__ __forceinline__ double hh_pending_k(const HhPending& q, double* red) {
    double s = 0.0;
    for (int64_t i = threadIdx.x; i < q.n1; i += blockDim.x) s += q.vp_part[i];
    const double t = block_sum(s, red);
    return q.v ? 0.5 * *q.tau * t : 0.0;
}

// element (i, j) of A22(k-1) with the pending update applied
__device__ __forceinline__ double hh_apply(double a, const HhPending& q, double K, int64_t i, int64_t j) {
    if (!q.v) return a;
    const double wi = q.p[i] - K * q.v[i], wj = q.p[j] - K * q.v[j];
    return a - (q.v[i] * wj + wi * q.v[j]);
}

// The pending update's v and w at index i (zero when none is pending).
struct HhVW {
    double v, w;
};
__device__ __forceinline__ HhVW hh_vw(const HhPending& q, double K, int64_t i) {
    if (!q.v) return HhVW{0.0, 0.0};
    const double v = q.v[i];
    return HhVW{v, q.p[i] - K * v};
}

// Reflection of x onto alpha e1 from its first element and the squares of the
// others, summed apart from its own: elements below 1e-8 of the first one
// would vanish in the rounding of |x|^2, and with them the coupling they carry.
struct HhReflect {
    double e;     // the off-diagonal entry: alpha, or x0 where there is nothing to reflect
    double v0;    // v = (v0, x1, x2, ...)
    double tau;
    bool trivial;
};
__device__ __forceinline__ HhReflect hh_reflect(double x0, double rest2) {
    const double nrm = sqrt(x0 * x0 + rest2);
    const double alpha = x0 > 0 ? -nrm : nrm;
    const double v0 = x0 - alpha, vnorm2 = rest2 + v0 * v0;
    const bool trivial = !(rest2 > 0.0) || !(vnorm2 >= DBL_MIN);  // (2 / vnorm2 stays finite)
    // (a NaN among the others, from infinities, shows in e)
    return HhReflect{trivial ? x0 + 0.0 * rest2 : alpha, v0, trivial ? 0.0 : 2.0 / vnorm2, trivial};
}

constexpr int kHhRows = 4;  // rows of A22 per k_hh_column block

// WAVES waves per row: 4 while the trailing matrix is large (more loads in
// flight), 1 once it is small (the launch's fixed cost dominates).  Every
// load that does not depend on the pending update's K (the partial sums
// that give K, this thread's share of row k for the norm, this lane's share
// of its row of A22 with row k beside it, the pending v and p there) is
// issued before the first barrier and held in registers, so a launch waits
// on memory once instead of three times in a row; elements beyond the held
// ones (a trailing matrix wider than the block for the norm, 2 x 256 or
// 4 x 64 per lane for the product, so that two 1024-thread blocks still fit
// on a CU) are read afterwards, the product's two per lane at a time with
// both loads issued before either store (four at a time spill registers).
template <int WAVES>
__global__ __launch_bounds__(64 * kHhRows * WAVES)
__attribute__((amdgpu_waves_per_eu(WAVES == 4 ? 8 : 4))) void k_hh_column(double* __restrict__ W, int64_t n,
                                                                          int64_t k, HhPending q,
                                                   double* __restrict__ v, double* __restrict__ tau,
                                                   double* __restrict__ d, double* __restrict__ e,
                                                   double* __restrict__ pv, double* __restrict__ vp_part) {
    constexpr int NT = 64 * kHhRows * WAVES;   // threads
    constexpr int NPF = 1;                     // row-k elements per thread held for the norm
    constexpr int RPF = WAVES == 4 ? 2 : 4;    // row elements per lane held for the product
    constexpr int64_t RST = 64 * WAVES;        // stride of a lane's row elements
    constexpr int CH = 2;                      // row elements per load group after the held ones
    __shared__ double red[kHhRows * WAVES];
    __shared__ double wsum[kHhRows * WAVES];
    const int64_t m = n - k - 1;
    const bool pend = q.v != nullptr;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t r = blockIdx.x * int64_t(kHhRows) + wv / WAVES;
    const int64_t jl = int64_t(wv % WAVES) * 64 + lane;
    const bool rowok = r < m;
    // row k beyond the diagonal, old values; its updated value at j is
    // x_j = row[j] - (v_0 w_{j+1} + w_0 v_{j+1}) (pending update, index 0)
    const double* row = W + k * n + k + 1;
    double* ar = W + (k + 1 + (rowok ? r : 0)) * n + k + 1;
    auto pv_at = [&](int64_t i) { return pend ? q.v[i] : 0.0; };
    auto pp_at = [&](int64_t i) { return pend ? q.p[i] : 0.0; };
    // --- loads independent of K
    double kp = 0.0;
    if (pend)
        for (int64_t i = threadIdx.x; i < q.n1; i += NT) kp += q.vp_part[i];
    const double tau_prev = pend ? *q.tau : 0.0;
    const double zv = pv_at(0), zp = pp_at(0);
    const double x0r = row[0], x0v = pv_at(1), x0p = pp_at(1);
    const double yv = rowok ? pv_at(r + 1) : 0.0, yp = rowok ? pp_at(r + 1) : 0.0;
    double nr[NPF], nv[NPF], np[NPF];
#pragma unroll
    for (int t = 0; t < NPF; t++) {
        const int64_t j = threadIdx.x + int64_t(t) * NT;
        const bool ok = j < m;
        nr[t] = ok ? row[j] : 0.0;
        nv[t] = ok ? pv_at(j + 1) : 0.0;
        np[t] = ok ? pp_at(j + 1) : 0.0;
    }
    double ra[RPF], rr[RPF], rv[RPF], rp[RPF];
#pragma unroll
    for (int t = 0; t < RPF; t++) {
        const int64_t j = jl + int64_t(t) * RST;
        const bool ok = rowok && j < m;
        ra[t] = ok ? ar[j] : 0.0;
        rr[t] = ok ? row[j] : 0.0;
        rv[t] = ok ? pv_at(j + 1) : 0.0;
        rp[t] = ok ? pp_at(j + 1) : 0.0;
    }
    // --- K of the pending update: the same ordered reduction in every block
    const double K = pend ? 0.5 * tau_prev * block_sum(kp, red) : 0.0;
    const double zw = zp - K * zv;
    // updated row k at j from the old value and the pending v, p at j + 1
    auto xk = [&](double rj, double vj, double pj) { return pend ? rj - (zv * (pj - K * vj) + zw * vj) : rj; };
    double s = 0.0;
#pragma unroll
    for (int t = 0; t < NPF; t++) {
        const double x = xk(nr[t], nv[t], np[t]);
        s += t == 0 && threadIdx.x == 0 ? 0.0 : x * x;
    }
#pragma unroll 2
    for (int64_t j = threadIdx.x + int64_t(NPF) * NT; j < m; j += NT) {
        const double x = xk(row[j], pv_at(j + 1), pp_at(j + 1));
        s += x * x;
    }
    const HhReflect h = hh_reflect(xk(x0r, x0v, x0p), block_sum(s, red));
    const bool trivial = h.trivial;
    const double v0 = h.v0, t = h.tau;
    if (blockIdx.x == 0) {
        for (int64_t i = threadIdx.x; i < m; i += NT)
            v[i] = trivial ? 0.0 : (i == 0 ? v0 : xk(row[i], pv_at(i + 1), pp_at(i + 1)));
        if (threadIdx.x == 0) {
            // diagonal entry k: the old one less 2 v_0 w_0 of the pending update
            d[k] = pend ? W[k * n + k] - 2.0 * zv * zw : W[k * n + k];
            e[k] = h.e;
            *tau = t;
        }
    }
    // p_r = tau sum_j A22[r][j] v_j, WAVES waves per row (kHhRows rows per
    // block) taking 64 columns in turn; the row is brought up to date
    // (pending update, index r + 1) as it is read and written back
    const double yw = yp - K * yv;
    double acc = 0.0;
    if (rowok) {
#pragma unroll
        for (int tt = 0; tt < RPF; tt++) {
            const int64_t j = jl + int64_t(tt) * RST;
            if (j < m) {
                const double cw = rp[tt] - K * rv[tt];
                double a = ra[tt];
                if (pend) {
                    a = a - (yv * cw + yw * rv[tt]);
                    ar[j] = a;
                }
                acc += a * (j == 0 ? v0 : xk(rr[tt], rv[tt], rp[tt]));
            }
        }
        // the rest in groups of CH elements whose loads are all issued
        // before the group's stores (same order of the sum)
        for (int64_t j0 = jl + int64_t(RPF) * RST; j0 < m; j0 += CH * RST) {
            double ca[CH], cr[CH], cv[CH], cp[CH];
#pragma unroll
            for (int u = 0; u < CH; u++) {
                const int64_t j = j0 + int64_t(u) * RST;
                const bool ok = j < m;
                ca[u] = ok ? ar[j] : 0.0;
                cr[u] = ok ? row[j] : 0.0;
                cv[u] = ok ? pv_at(j + 1) : 0.0;
                cp[u] = ok ? pp_at(j + 1) : 0.0;
            }
#pragma unroll
            for (int u = 0; u < CH; u++) {
                const int64_t j = j0 + int64_t(u) * RST;
                if (j < m) {
                    const double cw = cp[u] - K * cv[u];
                    double a = ca[u];
                    if (pend) {
                        a = a - (yv * cw + yw * cv[u]);
                        ar[j] = a;
                    }
                    acc += a * (j == 0 ? v0 : xk(cr[u], cv[u], cp[u]));
                }
            }
        }
        for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
    }
    if (lane == 0) wsum[wv] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double b = 0.0;
        for (int i = 0; i < kHhRows; i++) {
            const int64_t ri = blockIdx.x * int64_t(kHhRows) + i;
            if (ri >= m) break;
            double a = 0.0;
            for (int w = 0; w < WAVES; w++) a += wsum[WAVES * i + w];
            const double p = trivial ? 0.0 : t * a;
            pv[ri] = p;
            b += trivial ? 0.0 : p * (ri == 0 ? v0 : xk(row[ri], pv_at(ri + 1), pp_at(ri + 1)));
        }
        vp_part[blockIdx.x] = b;
    }
}

// ---------------------------------------------------------------------------
// Householder tridiagonalisation in one launch, for up to kTrRows kTrMaxBlocks
// rows.  A launch per column (above) is bound by the launch itself and by
// reading and writing the trailing matrix; here the matrix never leaves the
// registers.  Block b holds rows b, b + B, b + 2 B, ... (kTrRows of them, so
// every block keeps work until the end), thread t columns t + 512 u of each
// of them, and with them elements t + 512 u of v, w and the current row: the
// rank-2 update and the product A22 v need no other thread's data but the
// rows' own v and w.  At the end of a column a block publishes, for each of
// its rows r, p_r and the element A[r][k+1] of the next row to reflect (A is
// symmetric), and every block forms the same v, K and w from them.  What
// bounds a column is this exchange between all blocks, there and back, and
// three barriers in each: 2.2 us a column with 15 blocks, 3.0 us with 68 and
// 3.8 us with 250, where the reads of the exchange add up (2000 rows: 24.4 ms
// in a launch per column, 7.6 ms here; 540 rows: 3.5 and 1.6 ms; 120 rows:
// 0.65 and 0.27 ms).
//
// The exchange: slots hold kTrEmpty until a value is there, so a value is its
// own flag and a reader polls the values themselves (agent-scope relaxed
// accesses, which go to the point where the XCDs meet).  Three buffers take
// turns: a block publishes step k only after it has read all of step k-1, so
// once a block has read all of step k-1, everyone is done with step k-2, and
// the block empties its own slots of that buffer, which takes step k+1; its
// stores have completed before its next publication.
//
// Blocks that are not all resident at once (other work holds the CUs) would
// wait for each other; every wait is bounded by `spin` polls, after which the
// block raises *gave_up and ends; the others follow at their own bounds, those
// that start later at once, and the caller goes through the columns launch by
// launch.  (A look at *gave_up between polls: 2.27 ms in place of 1.93 for 540
// rows.)
// ---------------------------------------------------------------------------
constexpr int kTrThreads = 512;
constexpr int kTrRows = 8;
constexpr int kTrMaxBlocks = 256;
constexpr int kColumnUs = 12;    // a launch per column takes about this long per row
// Polls of a wait, about 1.2 us each: no longer than the columns would take.
constexpr int kTrSpinRow = 10, kTrSpinMin = 1000;
constexpr unsigned long long kTrEmpty = 0x7FF4DEAD5EED0001ull;  // a NaN no operation returns

// x plus the lane's neighbour under a DPP control (0 where there is none)
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ double dpp_add(double x) {
    const int lo = __double2loint(x), hi = __double2hiint(x);
    const int l2 = __builtin_amdgcn_update_dpp(0, lo, CTRL, ROWS, 0xF, true);
    const int h2 = __builtin_amdgcn_update_dpp(0, hi, CTRL, ROWS, 0xF, true);
    return x + __hiloint2double(h2, l2);
}

// Sum over the wave (valid in lane 63).
__device__ __forceinline__ double wave_sum63(double x) {
    x = dpp_add<0x111>(x);        // row_shr:1
    x = dpp_add<0x112>(x);        // row_shr:2
    x = dpp_add<0x114>(x);        // row_shr:4
    x = dpp_add<0x118>(x);        // row_shr:8
    x = dpp_add<0x142, 0xA>(x);   // row_bcast:15 into rows 1 and 3
    x = dpp_add<0x143, 0xC>(x);   // row_bcast:31 into rows 2 and 3
    return x;
}

// Sum over the lane's group of eight.
__device__ __forceinline__ double octet_sum(double x) {
    x = dpp_add<0xB1>(x);    // quad_perm [1, 0, 3, 2]
    x = dpp_add<0x4E>(x);    // quad_perm [2, 3, 0, 1]
    return dpp_add<0x141>(x);  // row_half_mirror
}

// a + b with the upper half (H 32) or odd rows of 16 (H 16) of a exchanged
// for the lower half or even rows of b: sums of a in the lanes that kept it,
// of b in the others.
template <int H>
__device__ __forceinline__ double swap_add(double a, double b) {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const unsigned al = __double2loint(a), ah = __double2hiint(a), bl = __double2loint(b), bh = __double2hiint(b);
    u2 l, h;
    if (H == 32) {
        l = __builtin_amdgcn_permlane32_swap(al, bl, false, false);
        h = __builtin_amdgcn_permlane32_swap(ah, bh, false, false);
    } else {
        l = __builtin_amdgcn_permlane16_swap(al, bl, false, false);
        h = __builtin_amdgcn_permlane16_swap(ah, bh, false, false);
    }
    return __hiloint2double(int(h[0]), int(l[0])) + __hiloint2double(int(h[1]), int(l[1]));
}

// Wave sums of eight values: lane l returns the sum of acc[l >> 3].
__device__ __forceinline__ double wave_sum8(const double (&acc)[kTrRows], int lane) {
    double u[4], t[2];
#pragma unroll
    for (int i = 0; i < 4; i++) u[i] = swap_add<32>(acc[i], acc[i + 4]);
#pragma unroll
    for (int i = 0; i < 2; i++) t[i] = swap_add<16>(u[i], u[i + 2]);
    const bool up = (lane & 8) != 0;
    const double y = up ? t[1] : t[0], z = up ? t[0] : t[1];
    const int zl = __builtin_amdgcn_update_dpp(0, __double2loint(z), 0x128, 0xF, 0xF, true);  // row_ror:8
    const int zh = __builtin_amdgcn_update_dpp(0, __double2hiint(z), 0x128, 0xF, 0xF, true);
    return octet_sum(y + __hiloint2double(zh, zl));
}

__device__ __forceinline__ void tr_put(unsigned long long* q, unsigned long long v) {
    __hip_atomic_store(q, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long tr_get(const unsigned long long* q) {
    return __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__global__ void k_tr_empty(unsigned long long* __restrict__ q, int64_t n, int* __restrict__ gave_up) {
    for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x)
        q[i] = kTrEmpty;
    if (blockIdx.x == 0 && threadIdx.x == 0) *gave_up = 0;
}

// E columns per thread (n <= 512 E).  C: the block at (off, off) of a matrix
// of row length P.  q: [3][2][n] slots (p, then the next row's elements).
// spin = 0: every block gives up at its first column.
// Element i of a thread's column c < k (reflected already) is kept zero.
template <int E>
__global__ __launch_bounds__(kTrThreads, 1) void k_tridiag(const double* __restrict__ C, int64_t P, int64_t off, int n,
                                                           const CheckFlags* fl, unsigned long long* __restrict__ q,
                                                           int spin, int* __restrict__ gave_up,
                                                           double* __restrict__ d, double* __restrict__ e) {
    constexpr int R = kTrRows, NW = kTrThreads / 64;
    __shared__ double red[2][NW];     // wave sums of v.p and of |x|^2 past its first element
    __shared__ double sums[NW][R];    // wave sums of the rows' products
    __shared__ double rv[R], rw[R];   // v and w at the block's rows
    __shared__ double rnext[R];       // A[r][k+1] at the block's rows
    __shared__ double at_k[3], at_k1; // v, p and A[k][k] at k; x at k + 1
    __shared__ int failed;
    if (fl->nan_seen || __hip_atomic_load(gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b = blockIdx.x, B = gridDim.x;
    const int rlast = b + (n - 1 - b) / B * B;  // the block's last row
    double a[R][E], v[E];
    int own[E];  // this thread's columns that are rows of this block: which one, or -1
#pragma unroll
    for (int u = 0; u < E; u++) {
        const int c = tid + u * kTrThreads;
        own[u] = (c < n && c % B == b) ? c / B : -1;
        v[u] = 0.0;
#pragma unroll
        for (int i = 0; i < R; i++) {
            const int r = b + i * B;
            a[i][u] = (r < n && c < n) ? C[(off + r) * P + off + c] : 0.0;
        }
    }
    // the first row to reflect, with no update pending
    const int myrow = b + tid * B;  // (tid < R) the row whose slots this thread fills first
    unsigned long long* const q0 = q;
    const int64_t step_words = 2 * int64_t(n);
    if (tid < R && myrow < n) {
        tr_put(q0 + 2 * step_words + myrow, 0ull);
        tr_put(q0 + 2 * step_words + n + myrow,
               (unsigned long long)__double_as_longlong(C[(off + myrow) * P + off]));
    }
    if (tid == 0) failed = 0;
    double tau = 0.0;
    int buf = 2;  // buffer of step k - 1
    __syncthreads();
    for (int k = 0; k + 1 < n; k++) {
        if (rlast <= k) return;  // none of the block's rows is left (row n - 1's block stays)
        const int buf_next = buf == 2 ? 0 : buf + 1;          // step k's
        const int buf_old = buf_next == 2 ? 0 : buf_next + 1;  // step k - 2's, which step k + 1 takes
        unsigned long long* const qp = q0 + buf * step_words;
        double w[E], x[E];
        {
            unsigned long long sp[E], sa[E];
            // (a first look that comes too early costs another round trip: 2000,
            // 540 and 120 rows 9.7, 2.2 and 0.37 ms without this pause, 7.6, 1.6
            // and 0.27 ms with it; a few blocks exchange sooner)
            if (B > 4) __builtin_amdgcn_s_sleep(8);
            bool ok = true;
#pragma unroll
            for (int u = 0; u < E; u++) {
                const int c = tid + u * kTrThreads;
                sp[u] = sa[u] = 0ull;
                if (c >= k && c < n) {
                    sp[u] = tr_get(qp + c);
                    sa[u] = tr_get(qp + n + c);
                }
            }
            for (int polls = 0;; polls++) {
                ok = true;
#pragma unroll
                for (int u = 0; u < E; u++) ok = ok && sp[u] != kTrEmpty && sa[u] != kTrEmpty;
                if (ok || polls >= spin) break;
#pragma unroll
                for (int u = 0; u < E; u++) {
                    const int c = tid + u * kTrThreads;
                    if (sp[u] == kTrEmpty) sp[u] = tr_get(qp + c);
                    if (sa[u] == kTrEmpty) sa[u] = tr_get(qp + n + c);
                }
            }
            if (!ok || spin == 0) failed = 1;
#pragma unroll
            for (int u = 0; u < E; u++) {
                w[u] = __longlong_as_double((long long)sp[u]);  // p for now
                x[u] = __longlong_as_double((long long)sa[u]);  // the row before the pending update
            }
        }
        double s = 0.0;
#pragma unroll
        for (int u = 0; u < E; u++) {
            s += v[u] * w[u];
            if (tid + u * kTrThreads == k) {
                at_k[0] = v[u];
                at_k[1] = w[u];
                at_k[2] = x[u];
            }
        }
        s = wave_sum63(s);
        if (lane == 63) red[0][wv] = s;
        __syncthreads();
        if (failed) {
            if (tid == 0) __hip_atomic_store(gave_up, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return;
        }
        if (tid < R && myrow < n) {
            tr_put(q0 + buf_old * step_words + myrow, kTrEmpty);
            tr_put(q0 + buf_old * step_words + n + myrow, kTrEmpty);
        }
        // the pending update's K and w, and row k brought up to date
        double K = 0.0;
#pragma unroll
        for (int i = 0; i < NW; i++) K += red[0][i];
        K *= 0.5 * tau;
        const double vk = at_k[0], wk = at_k[1] - K * vk;
        s = 0.0;
#pragma unroll
        for (int u = 0; u < E; u++) {
            const int c = tid + u * kTrThreads;
            w[u] -= K * v[u];
            x[u] = c > k && c < n ? x[u] - (vk * w[u] + wk * v[u]) : 0.0;
            s += c == k + 1 ? 0.0 : x[u] * x[u];
            if (c == k + 1) at_k1 = x[u];
            if (own[u] >= 0) {
                rv[own[u]] = v[u];
                rw[own[u]] = w[u];
            }
        }
        s = wave_sum63(s);
        if (lane == 63) red[1][wv] = s;
        __syncthreads();
        double rest2 = 0.0;
#pragma unroll
        for (int i = 0; i < NW; i++) rest2 += red[1][i];
        const HhReflect h = hh_reflect(at_k1, rest2);
        const bool trivial = h.trivial;
        const double v0 = h.v0;
        tau = h.tau;
        if (rlast == n - 1 && tid == 0) {
            d[k] = at_k[2] - 2.0 * vk * wk;
            e[k] = h.e;
        }
        double acc[R];
#pragma unroll
        for (int i = 0; i < R; i++) acc[i] = 0.0;
#pragma unroll
        for (int u = 0; u < E; u++) {
            const int c = tid + u * kTrThreads;
            const double vn = trivial ? 0.0 : (c == k + 1 ? v0 : x[u]);
#pragma unroll
            for (int i = 0; i < R; i++) {
                a[i][u] -= rv[i] * w[u] + rw[i] * v[u];
                acc[i] += a[i][u] * vn;
            }
            if (c == k + 1) {
#pragma unroll
                for (int i = 0; i < R; i++) rnext[i] = a[i][u];
            }
            v[u] = vn;
        }
        s = wave_sum8(acc, lane);
        if ((lane & 7) == 0) sums[wv][lane >> 3] = s;
        __syncthreads();
        if (wv == 0) {
            const int i = lane >> 3, r = b + i * B;
            const double p = octet_sum(sums[lane & 7][i]);
            // the emptied slots before the new values
            __builtin_amdgcn_s_waitcnt(0);
            if ((lane & 7) == 0 && r > k && r < n) {
                unsigned long long* const qn = q0 + buf_next * step_words;
                tr_put(qn + r, (unsigned long long)__double_as_longlong(trivial ? 0.0 : tau * p));
                tr_put(qn + n + r, (unsigned long long)__double_as_longlong(rnext[i]));
            }
        }
        buf = buf_next;
    }
    if (rlast == n - 1) {
#pragma unroll
        for (int u = 0; u < E; u++)
            if (tid + u * kTrThreads == n - 1) {
                const int il = (n - 1) / B;
#pragma unroll
                for (int i = 0; i < R; i++)
                    if (i == il) d[n - 1] = a[i][u];
            }
    }
}

// The last 2 x 2 block (rows n-2, n-1 = indices 0, 1 of the pending update's
// A22) gives the last diagonal and off-diagonal entries.  One block.
__global__ void k_hh_tail(const double* __restrict__ W, int64_t n, HhPending q, double* __restrict__ d,
                          double* __restrict__ e) {
    __shared__ double red[256];
    const double K = hh_pending_k(q, red);
    if (threadIdx.x != 0) return;
    if (n >= 2) {
        d[n - 2] = hh_apply(W[(n - 2) * n + n - 2], q, K, 0, 0);
        e[n - 2] = hh_apply(W[(n - 1) * n + n - 2], q, K, 1, 0);
    }
    d[n - 1] = hh_apply(W[(n - 1) * n + n - 1], q, K, n >= 2 ? 1 : 0, n >= 2 ? 1 : 0);
}

// Eigenvalue counts of the tridiagonal (d, e), scaled by a power of two to a
// spectrum within [-4, 4].  de: pairs (d_i, e_{i-1}^2), i < n, with e_{-1} = 0.
//
// sturm_count: the number of eigenvalues below x is the number of sign changes
// in the sequence of leading principal minors p_i = (d_i - x) p_{i-1} -
// e_{i-1}^2 p_{i-2} (Givens' Sturm sequence): one fused multiply-add on the
// critical path of a step, where the quotients p_i / p_{i-1} need a float64
// division.  Every fourth step both minors are scaled by a power of two, so
// they neither overflow nor underflow: a step shrinks them by 2^-220 at most,
// since squares of off-diagonals below kMinE2 are staged as kMinE2.  A diagonal
// equal to x counts as below it (kTie).  The two move the eigenvalues by less
// than kSturmError, an ulp of those beyond kSturmSmall.
//
// sturm_quotients: the same from the quotients, without those two: the sign of
// an eigenvalue near zero, however graded the matrix (1 beside 1e-31).  A
// quotient below DBL_MIN counts as negative.
constexpr double kMinE2 = 0x1p-220, kTie = 0x1p-100, kSturmError = 0x1p-98, kSturmSmall = 0x1p-46;

__device__ __forceinline__ int sturm_count(const double2* de, int64_t n, double x) {
    double p1 = 1.0, p2 = 0.0;  // p_{i-1}, p_{i-2}
    int c = 0;
    auto step = [&](int64_t i) {
        const double2 v = de[i];
        const double p = fma((v.x - x) - kTie, p1, -(v.y * p2));
        c += int(unsigned(__double2hiint(p) ^ __double2hiint(p1)) >> 31);
        p2 = p1;
        p1 = p;
    };
    int64_t i = 0;
    for (; i + 4 <= n; i += 4) {
#pragma unroll
        for (int u = 0; u < 4; u++) step(i + u);
        const int ex = -__builtin_amdgcn_frexp_exp(fmax(fabs(p1), fabs(p2)));
        p1 = __builtin_amdgcn_ldexp(p1, ex);
        p2 = __builtin_amdgcn_ldexp(p2, ex);
    }
    for (; i < n; i++) step(i);
    return c;
}

__device__ __noinline__ int sturm_quotients(const double2* de, int64_t n, double x) {
    double q = 1.0;
    int c = 0;
    for (int64_t i = 0; i < n; i++) {
        const double2 v = de[i];
        q = (v.x - x) - v.y / q;
        if (fabs(q) < DBL_MIN) q = -DBL_MIN;
        c += q < 0.0 ? 1 : 0;
    }
    return c;
}

// out: [0] min eig, [1] max eig, [2] count below 0 (as double).  Three
// blocks work at once: block 0 bisects for the smallest eigenvalue, block 1
// for the largest (kBisectThreads counts per round, one wave per SIMD: a
// round is bound by the serial recurrence of one count, a step of which
// takes about 30 cycles), block 2 counts the eigenvalues below 0.  Up to
// kBisectLds entries are read from LDS, more from the global scratch `de`
// (3 n pairs).  2000 rows: 2.3 ms with quotients, 0.6 ms here; 540 rows: 0.77
// and 0.16 ms.
constexpr int kBisectThreads = 256;
constexpr int64_t kBisectLds = 3072;  // 48 KB of LDS for the pairs
__global__ __launch_bounds__(kBisectThreads) void k_bisect(const double* __restrict__ d, const double* __restrict__ e,
                                                           int64_t n, const CheckFlags* fl, double2* __restrict__ de_g,
                                                           double* __restrict__ out) {
    __shared__ double red_lo[kBisectThreads / 64], red_hi[kBisectThreads / 64];
    __shared__ int first_s[kBisectThreads / 64];
    __shared__ double2 de_l[kBisectLds];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    constexpr int NW = kBisectThreads / 64;
    // Gershgorin bounds
    double lo = DBL_MAX, hi = -DBL_MAX;
    bool bad = fl->nan_seen != 0;
    for (int64_t i = tid; i < n; i += kBisectThreads) {
        const double r = (i > 0 ? fabs(e[i - 1]) : 0.0) + (i + 1 < n ? fabs(e[i]) : 0.0);
        bad |= !(fabs(d[i]) + r <= DBL_MAX);
        lo = fmin(lo, d[i] - r);
        hi = fmax(hi, d[i] + r);
    }
    for (int o = 32; o > 0; o >>= 1) {
        lo = fmin(lo, __shfl_xor(lo, o));
        hi = fmax(hi, __shfl_xor(hi, o));
    }
    if (lane == 0) {
        red_lo[wv] = lo;
        red_hi[wv] = hi;
    }
    if (__syncthreads_or(bad)) {
        if (tid == 0) out[blockIdx.x] = blockIdx.x == 2 ? -1.0 : __builtin_nan("");
        return;
    }
    for (int w = 0; w < NW; w++) {
        lo = fmin(lo, red_lo[w]);
        hi = fmax(hi, red_hi[w]);
    }
    const double span = fmax(fabs(lo), fabs(hi));
    if (span == 0.0) {  // a zero matrix
        if (tid == 0) out[blockIdx.x] = blockIdx.x == 2 ? double(n) : 0.0;
        return;
    }
    const int ex = -__builtin_amdgcn_frexp_exp(span);
    const bool staged = n <= kBisectLds;
    double2* de = staged ? de_l : de_g + int64_t(blockIdx.x) * n;
    auto stage = [&](double floor) {
        for (int64_t i = tid; i < n; i += kBisectThreads) {
            const double o = i > 0 ? __builtin_amdgcn_ldexp(e[i - 1], ex) : 0.0;
            de[i] = make_double2(__builtin_amdgcn_ldexp(d[i], ex), i > 0 ? fmax(o * o, floor) : 0.0);
        }
        __syncthreads();
    };
    stage(blockIdx.x == 2 ? 0.0 : kMinE2);
    auto count = [&](double x) { return staged ? sturm_count(de_l, n, x) : sturm_count(de, n, x); };
    if (blockIdx.x == 2) {
        if (tid == 0) out[2] = double(sturm_quotients(de, n, 0.0));
        return;
    }
    // block 0: smallest x with count(x) >= 1; block 1: smallest x with count(x) >= n
    lo = __builtin_amdgcn_ldexp(lo, ex) - 2.0 * DBL_EPSILON * n;
    hi = __builtin_amdgcn_ldexp(hi, ex) + 2.0 * DBL_EPSILON * n;
    const int target = blockIdx.x == 0 ? 1 : int(n);
    // cuts [lo, hi] at the points of all threads, in increasing order; below(x):
    // at least target eigenvalues lie below x
    auto cut = [&](auto&& point, auto&& below) {
        // bracket: the first point above the eigenvalue, and the one before it
        const unsigned long long at = __builtin_amdgcn_ballot_w64(below(point(tid)));
        if (lane == 0) first_s[wv] = at ? 64 * wv + __builtin_ctzll(at) : kBisectThreads;
        __syncthreads();
        int q = kBisectThreads;
        for (int w = 0; w < NW; w++) q = min(q, first_s[w]);
        __syncthreads();
        const double nlo = q > 0 ? fmax(lo, point(q - 1)) : lo;
        const double nhi = q < kBisectThreads ? fmin(hi, point(q)) : hi;
        lo = nlo;
        hi = nhi;
    };
    auto even = [&](int t) { return lo + (hi - lo) * double(t + 1) / double(kBisectThreads + 1); };
    auto size = [&] { return fmax(fabs(lo), fabs(hi)); };
    auto done = [&] { return hi - lo <= 2.0 * DBL_EPSILON * size(); };
    auto small = [&] { return size() < kSturmSmall && hi - lo < 0x1p8 * kSturmError; };
    for (int it = 0; it < 14 && !done() && !small(); it++) cut(even, [&](double x) { return count(x) >= target; });
    if (!done() && small()) {
        // near zero, where the minors' error begins to show, the quotients take
        // over; a bracket around zero is first cut at +-m 2^(-7 t), which
        // leaves a sign and a few octaves
        stage(0.0);
        lo -= kSturmError;
        hi += kSturmError;
        auto below = [&](double x) { return sturm_quotients(de, n, x) >= target; };
        if (lo < 0.0 && hi > 0.0) {
            const double m = size();
            cut([&](int t) {
                return t < kBisectThreads / 2 ? -__builtin_amdgcn_ldexp(m, -7 * t)
                                              : __builtin_amdgcn_ldexp(m, -7 * (kBisectThreads - 1 - t));
            }, below);
        }
        if (lo < 0.0 && hi > 0.0) lo = hi = 0.0;  // within 2^-900 of it
        for (int it = 0; it < 12 && !done(); it++) cut(even, below);
    }
    if (tid == 0) out[blockIdx.x] = __builtin_amdgcn_ldexp(0.5 * (lo + hi), -ex);
}

// Tridiagonalisation with one launch per column, on a fresh copy W of the
// block.
static void tridiag_columns(const double* C, int64_t P, int64_t off, int64_t n, double* W, CheckFlags* fl,
                            double* const (&v)[2], double* const (&pv)[2], double* const (&vpp)[2], double* tau,
                            double* d, double* e, hipStream_t s) {
    k_copy_block<<<nblocks(n * n, 256), 256, 0, s>>>(C, P, off, n, W, fl);
    HhPending q{nullptr, nullptr, nullptr, nullptr, 0};
    for (int64_t k = 0; k + 2 < n; k++) {
        const int64_t m = n - k - 1;
        const int64_t n1 = (m + kHhRows - 1) / kHhRows;
        const int c = int(k & 1);
        if (m >= 256)
            k_hh_column<4><<<unsigned(n1), 64 * kHhRows * 4, 0, s>>>(W, n, k, q, v[c], tau + c, d, e, pv[c], vpp[c]);
        else
            k_hh_column<1><<<unsigned(n1), 64 * kHhRows, 0, s>>>(W, n, k, q, v[c], tau + c, d, e, pv[c], vpp[c]);
        q = HhPending{v[c], pv[c], tau + c, vpp[c], n1};
    }
    k_hh_tail<<<1, 256, 0, s>>>(W, n, q, d, e);
}

// A call's share of the blocks that this process has running in resident
// tridiagonalisations on the device, a CU each; given back when the call ends.
// Checks of several threads whose blocks do not fit on the card together would
// hold each other up (four of 2000 rows: up to 99 ms each until they gave up;
// a launch per column 55 ms; one after another 10 to 35 ms), so a call waits
// in line for its share, at most twice as long as its own columns would take.
class ResidentBlocks {
  public:
    explicit ResidentBlocks(DeviceCtx* ctx) : ctx_(ctx) {}
    ~ResidentBlocks() {
        if (!n_) return;
        {
            std::lock_guard<std::mutex> lk(ctx_->resident_mu);
            ctx_->resident_blocks -= n_;
        }
        ctx_->resident_cv.notify_all();
    }
    ResidentBlocks(const ResidentBlocks&) = delete;
    ResidentBlocks& operator=(const ResidentBlocks&) = delete;
    bool take(int n, std::chrono::microseconds wait) {
        std::unique_lock<std::mutex> lk(ctx_->resident_mu);
        std::list<const ResidentBlocks*>& line = ctx_->resident_line;
        try {
            line.push_back(this);
        } catch (const std::bad_alloc&) {
            return false;  // (the columns need no place in line)
        }
        const bool got = ctx_->resident_cv.wait_for(
            lk, wait, [&] { return line.front() == this && ctx_->resident_blocks + n <= ctx_->n_cu; });
        line.remove(this);
        if (got) ctx_->resident_blocks += n_ = n;
        lk.unlock();
        ctx_->resident_cv.notify_all();  // the next in line
        return got;
    }

  private:
    DeviceCtx* ctx_;
    int n_ = 0;
};

// Check one diagonal block [off, off+n) of C.  Writes chol_ok, n_neg, min, max.
// spin: polls a wait of the resident tridiagonalisation may take (kTrDefault:
// by the rows; kTrColumns: a launch per column instead); *gave_up (if given):
// it ran and gave up.
constexpr int kTrDefault = -1, kTrColumns = -2;
static lc_status check_block(const double* C, int64_t P, int64_t off, int64_t n, hipStream_t s, int spin,
                             int32_t* chol_ok, int32_t* n_neg, double* mn, double* mx, int32_t* gave_up_out) {
    if (gave_up_out) *gave_up_out = 0;
    if (n == 0) {  // an empty block: nothing to factor, no eigenvalues
        *chol_ok = 1;
        *n_neg = 0;
        *mn = *mx = NAN;
        return LC_OK;
    }
    DevBuf<double> Wb, auxb;
    DevBuf<CheckFlags> flb;
    LC_TRY(Wb.alloc(size_t(n * n), s));
    // (past kBisectLds rows the bisection's blocks keep their pairs there)
    const int64_t npair = n <= kBisectLds ? 0 : 3 * n;
    const int64_t naux = 8 * n + 32 + 2 * npair;
    LC_TRY(auxb.alloc(size_t(naux), s));
    LC_TRY(flb.alloc(1, s));
    double* W = Wb.get();
    double* aux = auxb.get();
    CheckFlags* fl = flb.get();
    k_zero_flags<<<1, 64, 0, s>>>(fl, 1);
    // two sets of Householder buffers: the launch for column k reads step
    // k-1's set while it fills its own
    double* const v[2] = {aux, aux + n};
    double* const pv[2] = {aux + 2 * n, aux + 3 * n};
    double* d = aux + 4 * n;
    double* e = aux + 5 * n;
    double* const vpp[2] = {aux + 6 * n, aux + 7 * n};  // partial sums of v.p, (n + 3)/4 each
    double* tau = aux + 8 * n;                           // [2]
    double* res = aux + 8 * n + 4;
    double2* const de = reinterpret_cast<double2*>(aux + 8 * n + 32);
    // Cholesky
    k_copy_block<<<nblocks(n * n, 256), 256, 0, s>>>(C, P, off, n, W, fl);
    for (int64_t k0 = 0; k0 < n; k0 += kNB) {
        const int nb = int(std::min<int64_t>(kNB, n - k0));
        const int64_t rest = n - k0 - nb;
        auto* panel = nb == kNB ? k_potrf_panel<true> : k_potrf_panel<false>;
        panel<<<unsigned(std::max<int64_t>(1, (rest + 63) / 64)), 64, 0, s>>>(W, n, k0, nb, fl);
        if (rest > 0) {
            const int64_t T = (rest + 63) / 64;
            k_potrf_update<<<unsigned(T * (T + 1) / 2), 256, 0, s>>>(W, n, k0, fl);
        }
    }
    // eigenvalues: tridiagonalise, bisect
    DevBuf<unsigned long long> slots;
    DeviceCtx* ctx;
    LC_TRY(get_ctx(&ctx));
    const int B = int((n + kTrRows - 1) / kTrRows);
    bool resident = spin != kTrColumns && B <= std::min(kTrMaxBlocks, ctx->n_cu) && n <= 4 * kTrThreads;
    ResidentBlocks held(ctx);
    if (resident) resident = held.take(B, std::chrono::microseconds(2 * kColumnUs * n));
    if (resident) {
        LC_TRY(slots.alloc(size_t(6 * n) + 1, s));
        int* const gave_up = reinterpret_cast<int*>(slots.get() + 6 * n);
        k_tr_empty<<<nblocks(6 * n, 256), 256, 0, s>>>(slots.get(), 6 * n, gave_up);
        if (spin == kTrDefault) spin = std::max(kTrSpinMin, kTrSpinRow * int(n));
        auto* kern = n <= kTrThreads ? k_tridiag<1> : n <= 2 * kTrThreads ? k_tridiag<2> : k_tridiag<4>;
        kern<<<unsigned(B), kTrThreads, 0, s>>>(C, P, off, int(n), fl, slots.get(), spin, gave_up, d, e);
    } else {
        tridiag_columns(C, P, off, n, W, fl, v, pv, vpp, tau, d, e, s);
    }
    k_bisect<<<3, kBisectThreads, 0, s>>>(d, e, n, fl, de, res);
    CheckFlags hf;
    double hr[3];
    int hg = 0;
    if (resident) LC_TRY_HIP(hipMemcpyAsync(&hg, slots.get() + 6 * n, sizeof hg, hipMemcpyDeviceToHost, s));
    LC_TRY_HIP(hipMemcpyAsync(&hf, fl, sizeof hf, hipMemcpyDeviceToHost, s));
    LC_TRY_HIP(hipMemcpyAsync(hr, res, sizeof hr, hipMemcpyDeviceToHost, s));
    LC_TRY_HIP(hipStreamSynchronize(s));
    if (gave_up_out) *gave_up_out = hg;
    if (hg) {
        // the blocks were not all resident: column by column instead
        tridiag_columns(C, P, off, n, W, fl, v, pv, vpp, tau, d, e, s);
        k_bisect<<<3, kBisectThreads, 0, s>>>(d, e, n, fl, de, res);
        LC_TRY_HIP(hipMemcpyAsync(hr, res, sizeof hr, hipMemcpyDeviceToHost, s));
        LC_TRY_HIP(hipStreamSynchronize(s));
    }
    *chol_ok = (!hf.nan_seen && !hf.chol_fail) ? 1 : 0;
    *n_neg = int32_t(hr[2]);
    *mn = hr[0];
    *mx = hr[1];
    return LC_OK;
}

// Both blocks [0, split) and [split, P) of C.
static lc_status check_blocks(const double* C, int64_t P, int64_t split, hipStream_t s, int spin, lc_cov_report* rep,
                              int32_t* gave_up) {
    for (int q = 0; q < 2; q++)
        LC_TRY(check_block(C, P, q ? split : 0, q ? P - split : split, s, spin, &rep->chol_ok[q], &rep->n_neg_eig[q],
                           &rep->min_eig[q], &rep->max_eig[q], gave_up ? gave_up + q : nullptr));
    return LC_OK;
}

// The sample covariances of the three estimates, the construction and the
// check; blocks [0, split) and [split, P) of C are checked separately.
static lc_status covariance_impl(const double* xi, int32_t n_mock, int64_t P, int64_t split, double m_a, double m_b,
                                 double M, int32_t precision, double* A, double* B, double* C, lc_cov_report* rep,
                                 hipStream_t s) {
    if (!(M > 0.0)) return fail(LC_ERR_INVALID, "M must be > 0 (or INFINITY)");
    const bool acc32 = (precision & LC_ACC32) != 0;
    precision &= ~LC_ACC32;
    if (precision != LC_FP64 && precision != LC_FP32_MFMA && precision != LC_FP32_MFMA_CHECKED)
        return fail(LC_ERR_INVALID, "precision = %d is not LC_FP64 / LC_FP32_MFMA / LC_FP32_MFMA_CHECKED",
                    precision);
    if (acc32 && precision == LC_FP64) return fail(LC_ERR_INVALID, "LC_ACC32 needs a float32 MFMA precision");
    DeviceCtx* ctx;
    LC_TRY(get_ctx(&ctx));
    const int64_t N = n_mock;
    const int64_t PP = P * P;
    const int64_t W3 = 3 * P;
    const double denom = double(N - 1);
    const int m_inf = std::isinf(M) ? 1 : 0;
    DevBuf<double> meanb, partb, covb, Ab, Bb;
    LC_TRY(meanb.alloc(size_t(W3), s));
    const int64_t nchunk = (N + kMeanRows - 1) / kMeanRows;
    LC_TRY(partb.alloc(size_t(W3 * nchunk), s));
    LC_TRY(covb.alloc(size_t(3 * PP), s));
    if (!A) LC_TRY(Ab.alloc(size_t(PP), s));
    if (!B) LC_TRY(Bb.alloc(size_t(PP), s));
    double* mean = meanb.get();
    double* part = partb.get();
    double* cov = covb.get();
    double* Aw = A ? A : Ab.get();
    double* Bw = B ? B : Bb.get();
    {
        dim3 g(unsigned((W3 + 255) / 256), unsigned(nchunk));
        k_mean_partial<<<g, 256, 0, s>>>(xi, N, W3, part);
        k_mean_final<<<unsigned((W3 + 255) / 256), 256, 0, s>>>(part, nchunk, W3, N, mean);
    }
    auto run_fp64 = [&](double* covbuf) { return syrk_fp64(ctx, xi, mean, N, P, 3, denom, covbuf, s); };
    auto run_fp32 = [&](double* covbuf) { return syrk_fp32(ctx, xi, mean, N, P, 3, acc32, denom, covbuf, s); };
    if (precision == LC_FP64) {
        LC_TRY(run_fp64(cov));
    } else {
        LC_TRY(run_fp32(cov));
    }
    k_combine<<<nblocks(PP, 256, 65536), 256, 0, s>>>(cov, PP, m_a, m_b, M, m_inf, Aw, Bw, C);
    double rel[3] = {-1.0, -1.0, -1.0};
    if (precision == LC_FP32_MFMA_CHECKED) {
        DevBuf<double> A64, B64, C64, fpart;
        LC_TRY(A64.alloc(size_t(PP), s));
        LC_TRY(B64.alloc(size_t(PP), s));
        LC_TRY(C64.alloc(size_t(PP), s));
        const int nfb = 512;
        LC_TRY(fpart.alloc(size_t(2 * nfb * 3), s));
        LC_TRY(run_fp64(cov));
        k_combine<<<nblocks(PP, 256, 65536), 256, 0, s>>>(cov, PP, m_a, m_b, M, m_inf, A64.get(), B64.get(),
                                                          C64.get());
        k_frob<<<nfb, 256, 0, s>>>(C, C64.get(), PP, fpart.get());
        k_frob<<<nfb, 256, 0, s>>>(Aw, A64.get(), PP, fpart.get() + 2 * nfb);
        k_frob<<<nfb, 256, 0, s>>>(Bw, B64.get(), PP, fpart.get() + 4 * nfb);
        std::vector<double> h(2 * nfb * 3);
        LC_TRY_HIP(hipMemcpyAsync(h.data(), fpart.get(), sizeof(double) * h.size(), hipMemcpyDeviceToHost, s));
        A64.reset();
        B64.reset();
        C64.reset();
        fpart.reset();
        LC_TRY_HIP(hipStreamSynchronize(s));
        for (int q = 0; q < 3; q++) {
            double num = 0, den = 0;
            for (int bkt = 0; bkt < nfb; bkt++) {
                num += h[q * 2 * nfb + 2 * bkt];
                den += h[q * 2 * nfb + 2 * bkt + 1];
            }
            rel[q] = den > 0 ? std::sqrt(num / den) : (num > 0 ? INFINITY : 0.0);
        }
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(LC_ERR_HIP, "covariance launch failed: %s", hipGetErrorString(e));
    meanb.reset();
    partb.reset();
    covb.reset();
    if (rep) {
        rep->rel_frob_vs_fp64[0] = rel[0];
        rep->rel_frob_vs_fp64[1] = rel[1];
        rep->rel_frob_vs_fp64[2] = rel[2];
        LC_TRY(check_blocks(C, P, split, s, kTrDefault, rep, nullptr));
    }
    return LC_OK;
}

}  // namespace lc

using namespace lc;

extern "C" lc_status lc_covariance(const double* xi, int32_t n_mock, int32_t n_r, int32_t n_mu, int32_t m_a,
                                   double M, int32_t precision, double* A, double* B, double* C,
                                   lc_cov_report* rep, void* stream) {
    clear_error();
    if (!xi || !C) return fail(LC_ERR_INVALID, "xi and C must not be NULL");
    if (n_mock < 2) return fail(LC_ERR_INVALID, "n_mock = %d, need >= 2", n_mock);
    if (n_r < 1 || n_mu < 1 || n_mu > LC_MAX_NMU || int64_t(n_r) * n_mu > LC_MAX_BINS)
        return fail(LC_ERR_INVALID, "bad n_r = %d / n_mu = %d", n_r, n_mu);
    if (m_a < 1) return fail(LC_ERR_INVALID, "m_a = %d, must be >= 1", m_a);
    const int64_t nb0 = int64_t(n_r) * n_mu;
    return covariance_impl(xi, n_mock, nb0 + 3 * int64_t(n_r), nb0, double(m_a), 2.0 * double(m_a), M, precision, A,
                           B, C, rep, (hipStream_t)stream);
}

extern "C" lc_status lc_covariance_general(const double* xi, int32_t n_mock, int32_t P, int32_t n_split, double m_a,
                                           double m_b, double M, int32_t precision, double* A, double* B, double* C,
                                           lc_cov_report* rep, void* stream) {
    clear_error();
    if (!xi || !C) return fail(LC_ERR_INVALID, "xi and C must not be NULL");
    if (n_mock < 2) return fail(LC_ERR_INVALID, "n_mock = %d, need >= 2", n_mock);
    if (P < 1 || P > 4 * LC_MAX_BINS) return fail(LC_ERR_INVALID, "P = %d out of range", P);
    if (n_split < 0 || n_split > P) return fail(LC_ERR_INVALID, "n_split = %d outside [0, P = %d]", n_split, P);
    if (!(m_a > 0.0) || !(m_b > m_a) || !std::isfinite(m_b))
        return fail(LC_ERR_INVALID, "need 0 < m_a < m_b < infinity (got %g, %g)", m_a, m_b);
    return covariance_impl(xi, n_mock, P, n_split, m_a, m_b, M, precision, A, B, C, rep, (hipStream_t)stream);
}

extern "C" lc_status lc_sample_covariance(const double* x, int32_t n_mock, int32_t P, int32_t precision, double* C,
                                          void* stream) {
    clear_error();
    if (!x || !C) return fail(LC_ERR_INVALID, "x and C must not be NULL");
    if (n_mock < 2) return fail(LC_ERR_INVALID, "n_mock = %d, need >= 2", n_mock);
    if (P < 1 || P > 4 * LC_MAX_BINS) return fail(LC_ERR_INVALID, "P = %d out of range", P);
    const bool acc32 = (precision & LC_ACC32) != 0;
    precision &= ~LC_ACC32;
    if (precision != LC_FP64 && precision != LC_FP32_MFMA)
        return fail(LC_ERR_INVALID, "precision = %d is not LC_FP64 / LC_FP32_MFMA", precision);
    if (acc32 && precision == LC_FP64) return fail(LC_ERR_INVALID, "LC_ACC32 needs LC_FP32_MFMA");
    DeviceCtx* ctx;
    LC_TRY(get_ctx(&ctx));
    hipStream_t s = (hipStream_t)stream;
    const int64_t N = n_mock, PL = P;
    const double denom = double(N - 1);
    DevBuf<double> meanb, partb;
    LC_TRY(meanb.alloc(size_t(PL), s));
    const int64_t nchunk = (N + kMeanRows - 1) / kMeanRows;
    LC_TRY(partb.alloc(size_t(PL * nchunk), s));
    double* mean = meanb.get();
    double* part = partb.get();
    {
        dim3 g(unsigned((PL + 255) / 256), unsigned(nchunk));
        k_mean_partial<<<g, 256, 0, s>>>(x, N, PL, part);
        k_mean_final<<<unsigned((PL + 255) / 256), 256, 0, s>>>(part, nchunk, PL, N, mean);
    }
    if (precision == LC_FP64) {
        LC_TRY(syrk_fp64(ctx, x, mean, N, PL, 1, denom, C, s));
    } else {
        LC_TRY(syrk_fp32(ctx, x, mean, N, PL, 1, acc32, denom, C, s));
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(LC_ERR_HIP, "covariance launch failed: %s", hipGetErrorString(e));
    return LC_OK;
}

// Testing (not part of lc.h): the check alone, of a device matrix C, with the
// wait bound of its resident tridiagonalisation: spin > 0 polls; 0, it gives up
// at its first column; -1, as lc_covariance; -2, a launch per column.
// gave_up: HOST [2], per block.
extern "C" lc_status lc_testing_check(const double* C, int32_t P, int32_t n_split, int32_t spin, lc_cov_report* rep,
                                      int32_t* gave_up, void* stream) {
    clear_error();
    if (!C || !rep || !gave_up) return fail(LC_ERR_INVALID, "NULL argument");
    if (P < 1 || P > 4 * LC_MAX_BINS || n_split < 0 || n_split > P || spin < kTrColumns)
        return fail(LC_ERR_INVALID, "P = %d, n_split = %d or spin = %d out of range", P, n_split, spin);
    for (double& r : rep->rel_frob_vs_fp64) r = -1.0;
    return check_blocks(C, P, n_split, (hipStream_t)stream, spin, rep, gave_up);
}
