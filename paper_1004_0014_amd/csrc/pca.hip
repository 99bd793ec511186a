// PCA training of the motion model on the GPU (section 2.1, eq. (1); section
// 3: PCA over the N-1 DVFs between the reference phase and the other
// phases).  For J training DVFs d_j [3][N]:
//   mean  = (1/J) sum_j d_j
//   U     = the K leading left singular vectors of the centred 3N x J matrix
//           [d_1 - mean, ..., d_J - mean], unit norm, each flipped so that its
//           largest-magnitude entry (the first within 1e-5 of it) is positive
//   w_train[j][k] = <U_k, d_j - mean>.
// One streaming pass forms the raw Gram matrix G_ij = <d_i, d_j> in FP64; the
// centred Gram follows exactly in J x J algebra; a cyclic Jacobi eigen-solve
// on the host gives V and the singular values; a second streaming pass writes
// the mean and U_k = sum_j V_jk (d_j - mean) / sigma_k.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "host.h"

using namespace pcr;

namespace {

constexpr int kMaxJ = 16;
constexpr int kMaxPairs = kMaxJ * (kMaxJ + 1) / 2;
constexpr int kMaxChunks = 4096;     // of the field pass

// Raw Gram matrix of the J fields (upper triangle, FP64 per-block partials,
// stored pair-major for the final sum: partials[p * blocks + block]).  Bound
// by HBM once the next element's J loads are in flight while this one's
// products are formed (the 2 P registers of the sums leave four waves a SIMD,
// too few to hide a load each by themselves): 9 fields of 3 x 6.55 M values,
// 708 MB, 163 -> 153 us (4.6 TB/s) by events around the pass; in a kernel trace
// of single calls, 164 us.
template <int J>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(J <= 9 ? 4 : 1))) k_gram(const float* __restrict__ d, size_t E,
                                              double* __restrict__ partials)
{
    constexpr int P = J * (J + 1) / 2;
    double acc[P];
#pragma unroll
    for (int p = 0; p < P; ++p) acc[p] = 0.0;
    const size_t step = (size_t)gridDim.x * 256;
    size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
    float next[J];
    if (e < E) {
#pragma unroll
        for (int j = 0; j < J; ++j) next[j] = d[(size_t)j * E + e];
    }
    while (e < E) {
        double v[J];
#pragma unroll
        for (int j = 0; j < J; ++j) {
            // (opaque, or the wait for the next element moves up to its loads)
            asm volatile("" : "+v"(next[j]));
            v[j] = (double)next[j];
        }
        e += step;
        // (past the end: the last element again, not used)
        const size_t en = e < E ? e : E - 1;
#pragma unroll
        for (int j = 0; j < J; ++j) next[j] = d[(size_t)j * E + en];
        int p = 0;
#pragma unroll
        for (int i = 0; i < J; ++i)
#pragma unroll
            for (int j = i; j < J; ++j) acc[p++] += v[i] * v[j];
    }
    __shared__ double red[4][P];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int p = 0; p < P; ++p) {
        double s = acc[p];
        for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
        if (lane == 0) red[wv][p] = s;
    }
    __syncthreads();
    for (int p = threadIdx.x; p < P; p += 256)
        partials[(size_t)p * gridDim.x + blockIdx.x] = red[0][p] + red[1][p] + red[2][p] + red[3][p];
}

struct Coef {
    float v[kMaxJ * 8];   // V_jk / sigma_k
};

// Words of the training's device scratch that start at zero: the final sum's
// arrival count, and per field the guess of its sign (see k_sign_guess) and
// whether the guess has to be turned round.
struct SignState {
    unsigned arrived, pad;
    unsigned guess[8], flip[8];
};

// The sign rule needs a field's largest entry, which is known only after the
// field is written; turning it round then costs another pass over it.  A sample
// of the field (4096 values, evenly spread) guesses the sign beforehand: guess[k] = the
// largest sampled |u| (bits, shifted up) with its sign in the lowest bit.  A
// wrong guess only costs that pass.
template <int J>
__global__ void __launch_bounds__(256) k_sign_guess(const float* __restrict__ d, size_t E, int K, Coef c,
                                                    SignState* __restrict__ st)
{
    const size_t n = (size_t)gridDim.x * 256, i = (size_t)blockIdx.x * 256 + threadIdx.x;
    const size_t e = E / n * i + E % n * i / n;   // spread evenly over the field
    float v[J], s = 0.f;
#pragma unroll
    for (int j = 0; j < J; ++j) v[j] = d[(size_t)j * E + e];
#pragma unroll
    for (int j = 0; j < J; ++j) s += v[j];
    const float m = s / (float)J;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        if (k < K) {
            float u = 0.f;
#pragma unroll
            for (int j = 0; j < J; ++j) u = fmaf(c.v[j * 8 + k], v[j] - m, u);
            unsigned key = (__float_as_uint(fabsf(u)) << 1) | (u < 0.f ? 1u : 0u);
            for (int off = 32; off > 0; off >>= 1) key = max(key, (unsigned)__shfl_xor((int)key, off));
            if ((threadIdx.x & 63) == 0) atomicMax(&st->guess[k], key);
        }
    }
}

// mean and U_k = s_k sum_j (V_jk / sigma_k) (d_j - mean), s_k the guessed
// sign, and each block's max |U_k|: bmax[k * blocks + block].  A block takes
// one contiguous chunk of the field, four values a thread and step (fields
// of odd length leave the next one unaligned: the wide accesses ask for 4
// bytes).  Bound by HBM; the chunks go from the fields' ends backwards, so
// that those the Gram pass read last are still in the Infinity Cache.  708 MB
// read and 315 MB written in 190 -> 184 us (5.6 TB/s).
template <int J>
__global__ void __launch_bounds__(256) k_pca_fields(const float* __restrict__ d, size_t E, size_t chunk, int K,
                                                    Coef c, const SignState* __restrict__ st,
                                                    float* __restrict__ mean, float* __restrict__ U,
                                                    float* __restrict__ bmax)
{
    struct Vec {
        float v[4];
    };
    const unsigned b = gridDim.x - 1 - blockIdx.x;
    const size_t c0 = (size_t)b * chunk, c1 = min(E, c0 + chunk);
    float mx[8], sg[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        mx[k] = 0.f;
        sg[k] = k < K && (st->guess[k] & 1u) ? -1.f : 1.f;
    }
    auto point = [&](const float (&v)[J], float& m, float (&u)[8]) {
        float s = 0.f;
#pragma unroll
        for (int j = 0; j < J; ++j) s += v[j];
        m = s / (float)J;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            if (k < K) {
                float t = 0.f;
#pragma unroll
                for (int j = 0; j < J; ++j) t = fmaf(c.v[j * 8 + k], v[j] - m, t);
                u[k] = sg[k] * t;
                mx[k] = fmaxf(mx[k], fabsf(t));
            }
        }
    };
    for (size_t e = c0 + threadIdx.x * 4; e < c1; e += 1024) {
        if (e + 4 <= c1) {
            Vec v[J], m, o[8];
#pragma unroll
            for (int j = 0; j < J; ++j) __builtin_memcpy(&v[j], d + (size_t)j * E + e, sizeof(Vec));
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float w[J], u[8];
#pragma unroll
                for (int j = 0; j < J; ++j) w[j] = v[j].v[i];
                point(w, m.v[i], u);
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    if (k < K) o[k].v[i] = u[k];
            }
            __builtin_memcpy(mean + e, &m, sizeof(Vec));
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (k < K) __builtin_memcpy(U + (size_t)k * E + e, &o[k], sizeof(Vec));
        } else {
            for (size_t x = e; x < c1; ++x) {
                float w[J], m, u[8];
#pragma unroll
                for (int j = 0; j < J; ++j) w[j] = d[(size_t)j * E + x];
                point(w, m, u);
                mean[x] = m;
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    if (k < K) U[(size_t)k * E + x] = u[k];
            }
        }
    }
    __shared__ float red[4][8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        if (k < K) {
            float m = mx[k];
            for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_down(m, off, 64));
            if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][k] = m;
        }
    }
    __syncthreads();
    if ((int)threadIdx.x < K) {
        const int k = threadIdx.x;
        bmax[(size_t)k * gridDim.x + b] = fmaxf(fmaxf(red[0][k], red[1][k]), fmaxf(red[2][k], red[3][k]));
    }
}

// One block per field: its largest magnitude from the chunks' maxima, the
// first chunk that reaches (1 - 1e-5) of it (a tolerance well above FP32
// rounding, so near-ties of symmetric fields resolve alike in FP32 and FP64),
// and there the first such entry, which has to be positive: flip[k] = 1 if it
// is not.  sign_host[k] = the sign of the field against V's.
__global__ void __launch_bounds__(1024) k_sign_pick(const float* __restrict__ U, size_t E, size_t chunk,
                                                    const float* __restrict__ bmax, int nb,
                                                    SignState* __restrict__ st, double* __restrict__ sign_host)
{
    __shared__ float wm[16];
    __shared__ int first_chunk;
    __shared__ unsigned long long first;
    const int k = blockIdx.x, t = threadIdx.x;
    const float* bm = bmax + (size_t)k * nb;
    float v[kMaxChunks / 1024], m = 0.f;
#pragma unroll
    for (int i = 0; i < kMaxChunks / 1024; ++i) v[i] = bm[min(t + 1024 * i, nb - 1)];
#pragma unroll
    for (int i = 0; i < kMaxChunks / 1024; ++i) m = fmaxf(m, v[i]);
    for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
    if ((t & 63) == 0) wm[t >> 6] = m;
    if (t == 0) {
        first_chunk = nb;
        first = ~0ull;
    }
    __syncthreads();
    for (int i = 0; i < 16; ++i) m = fmaxf(m, wm[i]);
    const float thr = m * (1.0f - 1e-5f);
#pragma unroll
    for (int i = 0; i < kMaxChunks / 1024; ++i)
        if (t + 1024 * i < nb && v[i] >= thr) atomicMin(&first_chunk, t + 1024 * i);
    __syncthreads();
    const size_t c0 = (size_t)first_chunk * chunk, c1 = min(E, c0 + chunk);
    const float* u = U + (size_t)k * E;
    for (size_t e0 = c0 + t; e0 < c1; e0 += 8192) {
        float w[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) w[i] = u[min(e0 + 1024 * i, E - 1)];
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (e0 + 1024 * i < c1 && fabsf(w[i]) >= thr) atomicMin(&first, (unsigned long long)(e0 + 1024 * i));
    }
    __syncthreads();
    if (t == 0) {
        const bool neg = first < E && u[first] < 0.f;
        st->flip[k] = neg ? 1u : 0u;
        const bool guessed = st->guess[k] & 1u;
        __hip_atomic_store(&sign_host[k], guessed != neg ? -1.0 : 1.0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// turns the fields round whose guess was wrong
__global__ void __launch_bounds__(256) k_flip(float* __restrict__ U, size_t E, const SignState* __restrict__ st)
{
    const int k = blockIdx.y;
    if (!st->flip[k]) return;
    for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < E; e += (size_t)gridDim.x * 256)
        U[(size_t)k * E + e] = -U[(size_t)k * E + e];
}

// Cyclic Jacobi eigen-decomposition of a symmetric n x n matrix (row-major):
// A is overwritten; on exit lam[i] = eigenvalues, V (row-major) the
// eigenvectors in columns.
void jacobi_eigen(std::vector<double>& A, int n, std::vector<double>& lam, std::vector<double>& V)
{
    V.assign((size_t)n * n, 0.0);
    for (int i = 0; i < n; ++i) V[(size_t)i * n + i] = 1.0;
    for (int sweep = 0; sweep < 100; ++sweep) {
        double off = 0.0, tot = 0.0;
        for (int i = 0; i < n; ++i)
            for (int j = 0; j < n; ++j) {
                tot += A[(size_t)i * n + j] * A[(size_t)i * n + j];
                if (i != j) off += A[(size_t)i * n + j] * A[(size_t)i * n + j];
            }
        if (off <= 1e-30 * tot) break;
        for (int p = 0; p < n; ++p)
            for (int q = p + 1; q < n; ++q) {
                double apq = A[(size_t)p * n + q];
                if (apq == 0.0) continue;
                double app = A[(size_t)p * n + p], aqq = A[(size_t)q * n + q];
                double theta = (aqq - app) / (2.0 * apq);
                double t = (theta >= 0 ? 1.0 : -1.0) / (std::fabs(theta) + std::sqrt(theta * theta + 1.0));
                double c = 1.0 / std::sqrt(t * t + 1.0), s = t * c;
                for (int k = 0; k < n; ++k) {   // A <- J^T A J, rows/cols p, q
                    double akp = A[(size_t)k * n + p], akq = A[(size_t)k * n + q];
                    A[(size_t)k * n + p] = c * akp - s * akq;
                    A[(size_t)k * n + q] = s * akp + c * akq;
                }
                for (int k = 0; k < n; ++k) {
                    double apk = A[(size_t)p * n + k], aqk = A[(size_t)q * n + k];
                    A[(size_t)p * n + k] = c * apk - s * aqk;
                    A[(size_t)q * n + k] = s * apk + c * aqk;
                }
                for (int k = 0; k < n; ++k) {
                    double vkp = V[(size_t)k * n + p], vkq = V[(size_t)k * n + q];
                    V[(size_t)k * n + p] = c * vkp - s * vkq;
                    V[(size_t)k * n + q] = s * vkp + c * vkq;
                }
            }
    }
    lam.resize(n);
    for (int i = 0; i < n; ++i) lam[i] = A[(size_t)i * n + i];
}

// Device and host scratch of the training, kept per thread (about 1.2 MB: one
// allocation and one free a call took longer than the sums) and given back
// when the thread ends.
struct TrainScratch {
    DevBuf dev;
    HostBuf host;
    int host_dev = -1;            // device the host buffer was mapped for
    unsigned long long seq = 0;
    ~TrainScratch()
    {
        dev.release();
        host.release();
    }
};
thread_local TrainScratch train;

constexpr int kBlocks = 1024;        // of the Gram pass
constexpr int kPcaDone = kMaxPairs + 8;   // host slots: Gram sums, field signs, sequence number

template <int J>
pcr_status train_fields(const float* d, size_t E, int K, const Coef& c, float* mean, float* U, SignState* st,
                        float* bmax, hipStream_t s)
{
    size_t chunk = (E + kMaxChunks - 1) / kMaxChunks;
    chunk = (chunk + 1023) / 1024 * 1024;
    const int nb = (int)((E + chunk - 1) / chunk);
    const unsigned ns = (unsigned)std::min<size_t>((E + 255) / 256, 16);
    k_sign_guess<J><<<ns, 256, 0, s>>>(d, E, K, c, st);
    HIP_TRY(hipGetLastError());
    {
        PROF(PCA_FIELDS, s);
        k_pca_fields<J><<<nb, 256, 0, s>>>(d, E, chunk, K, c, st, mean, U, bmax);
        HIP_TRY(hipGetLastError());
    }
    k_sign_pick<<<K, 1024, 0, s>>>(U, E, chunk, bmax, nb, st, train.host.d + kMaxPairs);
    HIP_TRY(hipGetLastError());
    k_flip<<<dim3((unsigned)std::min<size_t>((E + 255) / 256, 2048), K), 256, 0, s>>>(U, E, st);
    HIP_TRY(hipGetLastError());
    return PCR_OK;
}

}  // namespace

extern "C" {

pcr_status pcr_pca_train(const pcr_grid* grid, int32_t J, const float* dvfs_dev, int32_t K,
                         float* mean_dev, float* U_dev, double* sing_host, double* w_train_host,
                         void* stream)
{
    PCR_TRY(check_grid(grid));
    if (J < 2 || J > kMaxJ) return fail(PCR_EINVAL, "J = %d must be in 2..%d", J, kMaxJ);
    if (K < 1 || K > 8 || K > J - 1) return fail(PCR_EINVAL, "K = %d must be in 1..min(8, J-1)", K);
    if (!dvfs_dev || !mean_dev || !U_dev) return fail(PCR_EINVAL, "NULL device pointer");
    hipStream_t s = (hipStream_t)stream;
    const size_t E = 3 * (size_t)grid->n[0] * grid->n[1] * grid->n[2];
    const int P = J * (J + 1) / 2;
    int dev;
    HIP_TRY(hipGetDevice(&dev));
    // scratch: the sign state, the chunks' maxima, the Gram partials
    constexpr size_t kState = 256, kMaxima = (size_t)8 * kMaxChunks * sizeof(float);
    static_assert(sizeof(SignState) <= kState, "sign state");
    PCR_TRY(train.dev.ensure(kState + kMaxima + (size_t)kBlocks * kMaxPairs * sizeof(double), dev, s));
    if (train.host_dev != dev) {
        train.host.release();
        train.host_dev = dev;
    }
    PCR_TRY(train.host.ensure(kPcaDone + 1));
    SignState* st = (SignState*)train.dev.p;
    float* bmax = (float*)((char*)train.dev.p + kState);
    double* part = (double*)((char*)train.dev.p + kState + kMaxima);
    HIP_TRY(launch_zero(st, kState, s));
    {
        PROF(PCA_GRAM, s);
        switch (J) {
#define PCR_G(n) case n: k_gram<n><<<kBlocks, 256, 0, s>>>(dvfs_dev, E, part); break;
            PCR_G(2) PCR_G(3) PCR_G(4) PCR_G(5) PCR_G(6) PCR_G(7) PCR_G(8) PCR_G(9)
            PCR_G(10) PCR_G(11) PCR_G(12) PCR_G(13) PCR_G(14) PCR_G(15) PCR_G(16)
#undef PCR_G
        }
        HIP_TRY(hipGetLastError());
    }
    unsigned long long* done = (unsigned long long*)(train.host.d + kPcaDone);
    const unsigned long long seq = ++train.seq;
    HIP_TRY(launch_reduce_publish(part, kBlocks, P, train.host.d, &st->arrived, done, seq, s));
    PCR_TRY(wait_published((const unsigned long long*)(train.host.p + kPcaDone), seq, s));
    const std::vector<double> Gu(train.host.p, train.host.p + P);
    // centred Gram: Gc_ij = G_ij - (r_i + r_j)/J + T/J^2
    std::vector<double> G((size_t)J * J), r(J, 0.0);
    for (int i = 0, p = 0; i < J; ++i)
        for (int j = i; j < J; ++j, ++p) G[(size_t)i * J + j] = G[(size_t)j * J + i] = Gu[p];
    double T = 0.0;
    for (int i = 0; i < J; ++i) {
        for (int j = 0; j < J; ++j) r[i] += G[(size_t)i * J + j];
        T += r[i];
    }
    std::vector<double> Gc((size_t)J * J);
    for (int i = 0; i < J; ++i)
        for (int j = 0; j < J; ++j) Gc[(size_t)i * J + j] = G[(size_t)i * J + j] - (r[i] + r[j]) / J + T / ((double)J * J);
    std::vector<double> lam, V;
    jacobi_eigen(Gc, J, lam, V);
    std::vector<int> order(J);
    for (int i = 0; i < J; ++i) order[i] = i;
    std::sort(order.begin(), order.end(), [&](int a, int b) { return lam[a] > lam[b]; });
    Coef c{};
    double sig[8];
    for (int k = 0; k < K; ++k) {
        sig[k] = std::sqrt(std::max(lam[order[k]], 0.0));
        if (!(sig[k] > 0.0)) return fail(PCR_EINVAL, "training DVFs have rank < K");
        for (int j = 0; j < J; ++j) c.v[j * 8 + k] = (float)(V[(size_t)j * J + order[k]] / sig[k]);
    }
    // the fields; sign rule: the first entry within 1e-5 of the largest
    // magnitude is positive
    switch (J) {
#define PCR_F(n) case n: PCR_TRY(train_fields<n>(dvfs_dev, E, K, c, mean_dev, U_dev, st, bmax, s)); break;
        PCR_F(2) PCR_F(3) PCR_F(4) PCR_F(5) PCR_F(6) PCR_F(7) PCR_F(8) PCR_F(9)
        PCR_F(10) PCR_F(11) PCR_F(12) PCR_F(13) PCR_F(14) PCR_F(15) PCR_F(16)
#undef PCR_F
    }
    HIP_TRY(hipStreamSynchronize(s));
    const double* sgn = train.host.p + kMaxPairs;
    // w_train[j][k] = <U_k, d_j - mean> = sign_k sigma_k V_jk
    for (int k = 0; k < K; ++k) {
        if (sing_host) sing_host[k] = sig[k];
        if (w_train_host)
            for (int j = 0; j < J; ++j) w_train_host[j * K + k] = sgn[k] * sig[k] * V[(size_t)j * J + order[k]];
    }
    return PCR_OK;
}

}  // extern "C"
