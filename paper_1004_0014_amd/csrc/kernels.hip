// HIP kernels for gfx950 (MI355X, CDNA4, wave64).
//
// Hot path of single-projection reconstruction under a PCA motion model
// (Li et al., section 2.2): per iteration compose the DVF, warp the
// reference image, ray-march the cone-beam projection, form the residual and
// return the cost and its gradient in w.
//
//  * Voxel passes (compose, warp, contraction) stream HBM: one thread per
//    voxel (composition: per four values), x-contiguous lanes,
//    structure-of-arrays fields.
//  * The ray march gathers from a zero-padded, channel-interleaved copy of
//    the warped image that stays resident in L2/MALL; each lane marches one
//    ray (or one segment of one) so a wave's taps fall in a compact 3-D
//    region; samples are clamped to the interpolant's support so no tap
//    needs a bounds check.
//  * Detector-wide and volume-wide sums accumulate in FP64: wave shuffles,
//    then LDS, then per-block partials, then one fixed-order final pass, so
//    every result is bitwise reproducible (no floating-point atomics in any
//    reduction).
#include <hip/hip_runtime.h>

#include <cmath>
#include <algorithm>
#include <climits>
#include <cstdint>
#include <cstdlib>
#include <type_traits>
#include <utility>

#include "pcr_internal.h"

namespace pcr {

// ------------------------------------------------------------ storage ----
struct bf16 {
    uint16_t bits;
};

template <typename R, typename S>
__device__ __forceinline__ R widen(S v);
template <> __device__ __forceinline__ float widen<float, float>(float v) { return v; }
template <> __device__ __forceinline__ double widen<double, float>(float v) { return v; }
template <> __device__ __forceinline__ float widen<float, double>(double v) { return (float)v; }
template <> __device__ __forceinline__ double widen<double, double>(double v) { return v; }
template <> __device__ __forceinline__ float widen<float, bf16>(bf16 v)
{
    return __uint_as_float((uint32_t)v.bits << 16);
}
template <> __device__ __forceinline__ double widen<double, bf16>(bf16 v)
{
    return (double)__uint_as_float((uint32_t)v.bits << 16);
}
template <> __device__ __forceinline__ float widen<float, _Float16>(_Float16 v) { return (float)v; }
template <> __device__ __forceinline__ double widen<double, _Float16>(_Float16 v) { return (double)(float)v; }

// C channels of type R, aligned to the largest power of two (at most 16
// bytes) that divides their size, so that arrays of cells have no padding
// (6 FP32 channels: 24-byte cells at 8-byte alignment).
template <typename R, int C>
struct alignas(((sizeof(R) * C) & (0 - sizeof(R) * C)) >= 16 ? 16 : ((sizeof(R) * C) & (0 - sizeof(R) * C))) Chan {
    R v[C];
};

template <typename T>
__device__ __forceinline__ T clampv(T x, T lo, T hi)
{
    return fmin(fmax(x, lo), hi);
}
__device__ __forceinline__ float clampv(float x, float lo, float hi) { return fminf(fmaxf(x, lo), hi); }

// ----------------------------------------------------------- reductions --
// Sum over the 64 lanes of a wave with the device library's wave reduction
// (a fixed DPP tree: the same order on every call, deterministic).
extern "C" __device__ __attribute__((const)) double __ockl_wfred_add_f64(double);
__device__ __forceinline__ double wave_sum(double v) { return __ockl_wfred_add_f64(v); }
extern "C" __device__ __attribute__((const)) float __ockl_wfred_min_f32(float);
__device__ __forceinline__ float wave_min(float v) { return __ockl_wfred_min_f32(v); }

// Sums over the wave of N doubles per lane (N a multiple of 4), in fewer
// exchanges than N separate sums: swapping the half waves of two registers
// and adding leaves one value's sums in each half, swapping the 16-lane rows
// of two such registers leaves four values in the rows of one; only N / 4
// registers then take the four steps within a row.  The sum of value
// i + (N/4) q ends in every lane of row q (lanes 16 q ..) of v[i].  A fixed
// order: deterministic.
__device__ __forceinline__ void swap_add(double& a, double b, bool rows)
{
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    union { double d; unsigned w[2]; } x{a}, y{b};
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const u2 r = rows ? __builtin_amdgcn_permlane16_swap(x.w[i], y.w[i], false, false)
                          : __builtin_amdgcn_permlane32_swap(x.w[i], y.w[i], false, false);
        x.w[i] = r.x;
        y.w[i] = r.y;
    }
    a = x.d + y.d;
}
template <int CTRL>
__device__ __forceinline__ double row_rot(double v)
{
    union { double d; int w[2]; } x{v};
    x.w[0] = __builtin_amdgcn_update_dpp(0, x.w[0], CTRL, 0xf, 0xf, false);
    x.w[1] = __builtin_amdgcn_update_dpp(0, x.w[1], CTRL, 0xf, 0xf, false);
    return x.d;
}
template <int N>
__device__ __forceinline__ void wave_sums(double (&v)[N])
{
    static_assert(N % 4 == 0, "N in quarters");
#pragma unroll
    for (int i = 0; i < N / 2; ++i) swap_add(v[i], v[i + N / 2], false);
#pragma unroll
    for (int i = 0; i < N / 4; ++i) swap_add(v[i], v[i + N / 4], true);
#pragma unroll
    for (int i = 0; i < N / 4; ++i) {
        v[i] += row_rot<0x128>(v[i]);   // row_ror:8, 4, 2, 1
        v[i] += row_rot<0x124>(v[i]);
        v[i] += row_rot<0x122>(v[i]);
        v[i] += row_rot<0x121>(v[i]);
    }
}
// Block (256 threads = 4 waves) sum of NM doubles per thread; thread t < nm
// writes dst[t * stride].  Only waves 0 .. nw-1 hold data (the others add
// nothing and skip their sums).  Fixed order: wave tree, then waves 0..nw-1.
// (16 moments: ~100 instructions against ~340 for 16 separate sums, which
// the block's other waves wait for.)
template <int NM>
__device__ __forceinline__ void block_sum_store(double (&m)[NM], int nm, double* dst, int stride,
                                                int nw = 4, bool through = false)
{
    constexpr int N = (NM + 3) / 4 * 4, Q = N / 4;
    __shared__ double red[4][N];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (wv < nw) {
        double v[N];
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = i < NM ? m[i] : 0.0;
        wave_sums(v);
        double s = v[0];
#pragma unroll
        for (int i = 1; i < Q; ++i) s = (lane & 15) == i ? v[i] : s;
        if ((lane & 15) < Q) red[wv][(lane >> 4) * Q + (lane & 15)] = s;
    }
    __syncthreads();
    if ((int)threadIdx.x < nm) {
        double s = red[0][threadIdx.x];
        for (int w2 = 1; w2 < nw; ++w2) s += red[w2][threadIdx.x];
        // (through: past this XCD's L2, for a block on another one)
        if (through)
            __hip_atomic_store(&dst[(size_t)threadIdx.x * stride], s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else dst[(size_t)threadIdx.x * stride] = s;
    }
}

// The ray segments' sums (and sample counts) into segment 0's thread of
// each ray (threads [0, rpb)); smem holds T (C + 1) words.  Afterwards
// only segment 0 holds data: the block's moments need only its waves.
template <int C, int T>
__device__ __forceinline__ void gather_segments(char* smem, int seg, int rpb, int sid, float (&acc)[C],
                                                int& nsamp)
{
    float* segbuf = (float*)smem;
    int* segn = (int*)(segbuf + T * C);
#pragma unroll
    for (int c = 0; c < C; ++c) segbuf[threadIdx.x * C + c] = acc[c];
    segn[threadIdx.x] = nsamp;
    __syncthreads();
    if (sid == 0)
        for (int s2 = 1; s2 < seg; ++s2) {
#pragma unroll
            for (int c = 0; c < C; ++c) acc[c] += segbuf[(threadIdx.x + s2 * rpb) * C + c];
            nsamp += segn[threadIdx.x + s2 * rpb];
        }
}

// Sum over the blocks of their partial sums, stored slot-major: part[m *
// nblocks + b] is slot m of block b.  out[0..nm) = sums of slots 0..nm-1;
// with extra >= 0 also out[nm] = the sum of slot `extra`.  One workgroup per
// output, 16 KB of loads in flight: a single workgroup for all of them was
// bound by what one CU can read (16 outputs of 3072 partials: 7.5 -> 4.5 us,
// 21 of 12288: 10 -> 4.3 us).  Thread t adds blocks t, t + 256, ... in order,
// then a fixed tree: deterministic.
// With done != null the sums are stored at system scope (through to memory);
// each workgroup waits for its store to complete and then counts itself in
// `arrived` (which wraps to zero at the last, so it is ready for the next
// launch), and the last one stores `seq` into *done with a system-scope
// release: a host polling *done in mapped memory sees the sums once it sees
// seq.  One release fence per launch, not one per workgroup.
__global__ void __launch_bounds__(256) k_reduce(const double* __restrict__ part, int nblocks, int nm,
                                                int extra, double* __restrict__ out, unsigned* arrived,
                                                unsigned long long* done, unsigned long long seq)
{
    __shared__ double red[4];
    const int o = blockIdx.x;
    const double* r = part + (size_t)(o < nm ? o : extra) * nblocks;
    double s = 0.0;
    for (int b0 = threadIdx.x; b0 < nblocks; b0 += 256 * 8) {
        // (past the end: the last block's partial, not added)
        double v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = r[min(b0 + 256 * i, nblocks - 1)];
#pragma unroll
        for (int i = 0; i < 8; ++i) s += b0 + 256 * i < nblocks ? v[i] : 0.0;
    }
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x != 0) return;
    s = ((red[0] + red[1]) + red[2]) + red[3];
    if (!done) {
        out[o] = s;
        return;
    }
    __hip_atomic_store(&out[o], s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __builtin_amdgcn_s_waitcnt(0);   // the store is complete
    asm volatile("" ::: "memory");
    if (atomicInc(arrived, gridDim.x - 1) == gridDim.x - 1)
        __hip_atomic_store(done, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

static hipError_t run_reduce(const double* part, int nblocks, int nm, int extra, double* out, hipStream_t s,
                             unsigned* arrived = nullptr, unsigned long long* done = nullptr,
                             unsigned long long seq = 0)
{
    k_reduce<<<nm + (extra >= 0 ? 1 : 0), 256, 0, s>>>(part, nblocks, nm, extra, out, arrived, done, seq);
    return hipGetLastError();
}

// The same sums at the end of the kernel that makes the partials, by its last
// block to arrive (256 threads; every block calls this after block_sum_store
// with `through`): where the blocks are few, a launch and the gap before it
// cost more than one block reading all partials.  The partials were stored
// past the L2s and each block waits for its own to complete before it counts
// itself, so no cache is written back (a device-wide fence per block made
// this slower than a second launch).  Only for NM + 1 <= 64 slots.
constexpr int kFusedSumBlocks = 512;
template <int NM>
__device__ __forceinline__ void last_block_sums(const double* part, int nm, int extra, double* out, unsigned* arrived,
                                                unsigned long long* done, unsigned long long seq)
{
    static_assert(NM + 1 <= 64, "slots stored by the first wave");
    __shared__ int last;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nb = gridDim.x;
    if (wv == 0) {
        __builtin_amdgcn_s_waitcnt(0);   // this wave's partials are stored
        asm volatile("" ::: "memory");
        if (lane == 0) last = atomicInc(arrived, (unsigned)nb - 1) == (unsigned)nb - 1;
    }
    __syncthreads();
    if (!last) return;
    constexpr int NO = (NM + 1 + 3) / 4;   // outputs a wave: wv, wv + 4, ...
    constexpr int QN = NM <= 14 ? 4 : 2;   // reads in flight for each, as registers allow
    const int nout = nm + 1;
    double s[NO];
#pragma unroll
    for (int i = 0; i < NO; ++i) s[i] = 0.0;
    for (int b0 = lane; b0 < nb; b0 += 64 * QN) {
        double v[NO][QN];
#pragma unroll
        for (int i = 0; i < NO; ++i) {
            const int o = min(wv + 4 * i, nout - 1);
            const double* r = part + (size_t)(o < nm ? o : extra) * nb;
#pragma unroll
            for (int q = 0; q < QN; ++q)
                v[i][q] = __hip_atomic_load(&r[min(b0 + 64 * q, nb - 1)], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
#pragma unroll
        for (int i = 0; i < NO; ++i)
#pragma unroll
            for (int q = 0; q < QN; ++q) s[i] += b0 + 64 * q < nb ? v[i][q] : 0.0;
    }
#pragma unroll
    for (int i = 0; i < NO; ++i) {
        const double t = wave_sum(s[i]);
        if (lane == 0 && wv + 4 * i < nout)
            __hip_atomic_store(&out[wv + 4 * i], t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(done, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// ------------------------------------------------------------ compose ----
// dvf = mean + sum_k w_k U_k over the E = 3 N values of a field (the components
// follow each other, so fields add value by value).  Four values a thread,
// every field's loads before the first sum: bound by HBM.  A field of odd
// length leaves the next one unaligned: the wide loads ask for the element's
// alignment only.  FP16 model, 255x251x99, K = 3: 82 -> 34 us (228 MB);
// FP32, 256x256x100: 81 -> 67 us (394 MB).
template <typename R, typename S, int K>
__global__ void __launch_bounds__(256) k_compose(const S* __restrict__ mean, const S* __restrict__ U, size_t E,
                                                 Chan<double, 8> w, R* __restrict__ dvf)
{
    constexpr int V = 4;
    struct Vec {
        S v[V];
    };
    const size_t e = ((size_t)blockIdx.x * 256 + threadIdx.x) * V;
    if (e >= E) return;
    if (e + V <= E) {
        Vec m, f[K];
        __builtin_memcpy(&m, mean + e, sizeof m);
#pragma unroll
        for (int k = 0; k < K; ++k) __builtin_memcpy(&f[k], U + (size_t)k * E + e, sizeof m);
        struct {
            R v[V];
        } o;
#pragma unroll
        for (int i = 0; i < V; ++i) {
            R x = widen<R>(m.v[i]);
#pragma unroll
            for (int k = 0; k < K; ++k) x += (R)w.v[k] * widen<R>(f[k].v[i]);
            o.v[i] = x;
        }
        __builtin_memcpy(dvf + e, &o, sizeof o);
    } else {
        for (size_t i = e; i < E; ++i) {
            R x = widen<R>(mean[i]);
#pragma unroll
            for (int k = 0; k < K; ++k) x += (R)w.v[k] * widen<R>(U[(size_t)k * E + i]);
            dvf[i] = x;
        }
    }
}

// --------------------------------------------------------------- warp ----
// x / s for a grid constant s, given rs = RN(1 / s): a product and one
// correction step (Markstein), the correctly rounded quotient of a normal
// result at a third of the instructions of a division.  Of an infinity (or
// of a product that overflows) the correction is NaN and the product stands.
template <typename R>
__device__ __forceinline__ R div_by(R x, R s, R rs)
{
    const R q = x * rs, c = fma(fma(-q, s, x), rs, q);
    return c == c ? c : q;
}

// Trilinear sample of an unpadded image at index-space point q, zero outside;
// optionally also the exact partial derivatives dT/dq (floor cell).  All taps
// are loaded before the first is used (a branch per tap made each wait for
// the one before): where every lane's cell lies inside the image, as four
// pairs along x, else by the lanes that reach it, at clamped indices and
// masked.
template <typename R, typename S, bool GRAD>
__device__ __forceinline__ R sample_f0(const S* __restrict__ f0, int nx, int ny, int nz,
                                       R qx, R qy, R qz, R* dT)
{
    qx = clampv(qx, (R)-2, (R)(nx + 1));
    qy = clampv(qy, (R)-2, (R)(ny + 1));
    qz = clampv(qz, (R)-2, (R)(nz + 1));
    R fx = floor(qx), fy = floor(qy), fz = floor(qz);
    int i0 = (int)fx, j0 = (int)fy, k0 = (int)fz;
    R ax = qx - fx, ay = qy - fy, az = qz - fz;
    R bx = (R)1 - ax, by = (R)1 - ay, bz = (R)1 - az;
    R c[2][2][2];
    const bool inside = (unsigned)i0 < (unsigned)(nx - 1) && (unsigned)j0 < (unsigned)(ny - 1) &&
                        (unsigned)k0 < (unsigned)(nz - 1);
    if (__all(inside)) {
        struct Pair {
            S a, b;
        } t[2][2];
        const S* base = f0 + ((size_t)i0 + (size_t)nx * ((size_t)j0 + (size_t)ny * k0));
#pragma unroll
        for (int dz = 0; dz < 2; ++dz)
#pragma unroll
            for (int dy = 0; dy < 2; ++dy)
                __builtin_memcpy(&t[dz][dy], base + ((size_t)nx * (dy + (size_t)ny * dz)), sizeof(Pair));
#pragma unroll
        for (int dz = 0; dz < 2; ++dz)
#pragma unroll
            for (int dy = 0; dy < 2; ++dy) {
                c[dz][dy][0] = widen<R>(t[dz][dy].a);
                c[dz][dy][1] = widen<R>(t[dz][dy].b);
            }
    } else {
        // (values alone: lanes whose cell lies outside altogether load nothing.
        // 100x90x80 moved by up to 200 mm 8.9 -> 6.0 us, 256x256x100 by noise of
        // 30 mm 186 -> 164 us.  With derivatives, the region that a solve warps
        // leaves out most of them.)
        const bool near = (unsigned)(i0 + 1) < (unsigned)(nx + 1) && (unsigned)(j0 + 1) < (unsigned)(ny + 1) &&
                          (unsigned)(k0 + 1) < (unsigned)(nz + 1);
        S t[2][2][2];
        if (GRAD || near) {
#pragma unroll
            for (int dz = 0; dz < 2; ++dz)
#pragma unroll
                for (int dy = 0; dy < 2; ++dy)
#pragma unroll
                    for (int dx = 0; dx < 2; ++dx) {
                        const int i = min(max(i0 + dx, 0), nx - 1), j = min(max(j0 + dy, 0), ny - 1),
                                  k = min(max(k0 + dz, 0), nz - 1);
                        t[dz][dy][dx] = f0[(size_t)i + (size_t)nx * ((size_t)j + (size_t)ny * k)];
                    }
        }
#pragma unroll
        for (int dz = 0; dz < 2; ++dz)
#pragma unroll
            for (int dy = 0; dy < 2; ++dy)
#pragma unroll
                for (int dx = 0; dx < 2; ++dx) {
                    const bool in = (unsigned)(i0 + dx) < (unsigned)nx && (unsigned)(j0 + dy) < (unsigned)ny &&
                                    (unsigned)(k0 + dz) < (unsigned)nz;
                    c[dz][dy][dx] = in ? widen<R>(t[dz][dy][dx]) : (R)0;
                }
    }
    R w00 = by * bz, w10 = ay * bz, w01 = by * az, w11 = ay * az;
    R val = w00 * (bx * c[0][0][0] + ax * c[0][0][1]) + w10 * (bx * c[0][1][0] + ax * c[0][1][1]) +
            w01 * (bx * c[1][0][0] + ax * c[1][0][1]) + w11 * (bx * c[1][1][0] + ax * c[1][1][1]);
    if (GRAD) {
        dT[0] = w00 * (c[0][0][1] - c[0][0][0]) + w10 * (c[0][1][1] - c[0][1][0]) +
                w01 * (c[1][0][1] - c[1][0][0]) + w11 * (c[1][1][1] - c[1][1][0]);
        dT[1] = bx * bz * (c[0][1][0] - c[0][0][0]) + ax * bz * (c[0][1][1] - c[0][0][1]) +
                bx * az * (c[1][1][0] - c[1][0][0]) + ax * az * (c[1][1][1] - c[1][0][1]);
        dT[2] = bx * by * (c[1][0][0] - c[0][0][0]) + ax * by * (c[1][0][1] - c[0][0][1]) +
                bx * ay * (c[1][1][0] - c[0][1][0]) + ax * ay * (c[1][1][1] - c[0][1][1]);
    }
    return val;
}

struct VoxGrid {
    int nx, ny, nz;
    double sp[3];
    double rd[3];   // 1 / sp, and 1 / (float)sp in FP32 (for div_by)
    float rf[3];
};
template <typename R>
__device__ __forceinline__ R by_spacing(R x, const VoxGrid& g, int a)
{
    if constexpr (std::is_same<R, float>::value) return div_by(x, (float)g.sp[a], g.rf[a]);
    else return div_by(x, (R)g.sp[a], (R)g.rd[a]);
}

// Displacement x = mean + sum_k w_k u_k and the fields u_k of one voxel: all
// loads first, then the sums.  Fields past the K-th (of KM) repeat the last
// one's loads (from the cache) and are replaced by zero.  O: type of the
// voxel's byte offset within a field.
template <typename R, typename S, int KM, typename O>
__device__ __forceinline__ void load_fields(const S* __restrict__ mean, const S* __restrict__ U, int K, size_t N,
                                            O off, const Chan<double, 8>& w, R (&x)[3], R (&u)[KM][3])
{
    S m[3], f[KM][3];
#pragma unroll
    for (int a = 0; a < 3; ++a) m[a] = *(const S*)((const char*)(mean + a * N) + off);
#pragma unroll
    for (int kk = 0; kk < KM; ++kk)
#pragma unroll
        for (int a = 0; a < 3; ++a)
            f[kk][a] = *(const S*)((const char*)(U + (size_t)(min(kk, K - 1) * 3 + a) * N) + off);
#pragma unroll
    for (int a = 0; a < 3; ++a) x[a] = widen<R>(m[a]);
#pragma unroll
    for (int kk = 0; kk < KM; ++kk)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            u[kk][a] = kk < K ? widen<R>(f[kk][a]) : (R)0;
            x[a] += (R)w.v[kk] * u[kk][a];
        }
}

// Standalone warp: f[v] = T[f0](v + dvf[v] / s).
template <typename R, typename S>
__global__ void __launch_bounds__(256) k_warp_plain(const S* __restrict__ f0,
                                                    const R* __restrict__ dvf, VoxGrid g,
                                                    R* __restrict__ f)
{
    int i = blockIdx.x * 64 + threadIdx.x, j = blockIdx.y * 4 + threadIdx.y, k = blockIdx.z;
    if (i >= g.nx || j >= g.ny) return;
    size_t N = (size_t)g.nx * g.ny * g.nz;
    size_t v = (size_t)i + (size_t)g.nx * ((size_t)j + (size_t)g.ny * k);
    const R x0 = dvf[v], x1 = dvf[N + v], x2 = dvf[2 * N + v];
    R qx = (R)i + by_spacing(x0, g, 0);
    R qy = (R)j + by_spacing(x1, g, 1);
    R qz = (R)k + by_spacing(x2, g, 2);
    f[v] = sample_f0<R, S, false>(f0, g.nx, g.ny, g.nz, qx, qy, qz, nullptr);
}

// Fused compose + warp (+ tangents) of one voxel: channel 0 = f, channels
// 1..K = h_k = sum_a (1/s_a) dT[f0]/dq_a u_k[a] (tangent), rest zero.  KM: most
// fields the instance takes.  (FP32 images stay below 2^31 bytes at 4 bytes a
// voxel or more, so a field's byte offsets fit 32 bits there.)
template <typename R, typename S, typename F, int C, bool TAN, int KM>
__device__ __forceinline__ Chan<R, C> warp_cell(const F* __restrict__ f0, const S* __restrict__ mean,
                                                const S* __restrict__ U, int K,
                                                const Chan<double, 8>& w, const VoxGrid& g, int i,
                                                int j, int k)
{
    using O = typename std::conditional<std::is_same<R, float>::value, unsigned, size_t>::type;
    const size_t N = (size_t)g.nx * g.ny * g.nz;
    const O off = ((O)i + (O)g.nx * ((O)j + (O)g.ny * (O)k)) * (O)sizeof(S);
    R x[3], u[KM][3];
    load_fields<R, S, KM, O>(mean, U, K, N, off, w, x, u);
    R qx = (R)i + by_spacing(x[0], g, 0);
    R qy = (R)j + by_spacing(x[1], g, 1);
    R qz = (R)k + by_spacing(x[2], g, 2);
    R dT[3];
    Chan<R, C> o;
#pragma unroll
    for (int c = 0; c < C; ++c) o.v[c] = (R)0;
    o.v[0] = sample_f0<R, F, TAN>(f0, g.nx, g.ny, g.nz, qx, qy, qz, dT);
    if constexpr (TAN) {
        R G0 = by_spacing(dT[0], g, 0), G1 = by_spacing(dT[1], g, 1), G2 = by_spacing(dT[2], g, 2);
#pragma unroll
        for (int kk = 0; kk < C - 1; ++kk)
            if (kk < K) o.v[kk + 1] = G0 * u[kk][0] + G1 * u[kk][1] + G2 * u[kk][2];
    }
    return o;
}

// Cell as stored: the compute type, or (H) FP16 of value * hs[c].
template <typename R, int C, bool H>
using CellOf = Chan<typename std::conditional<H, _Float16, R>::type, C>;
template <typename R, int C, bool H>
__device__ __forceinline__ CellOf<R, C, H> store_cell(const Chan<R, C>& o, const Chan<float, 8>& hs)
{
    if constexpr (!H) {
        return o;
    } else {
        CellOf<R, C, H> h;
#pragma unroll
        for (int c = 0; c < C; ++c) h.v[c] = (_Float16)((float)o.v[c] * hs.v[c]);
        return h;
    }
}

// Voxels [lo, hi) per axis that a launch computes.
struct VoxBox {
    int lo[3], hi[3];
};

// Blocks are dispatched round-robin over the 8 XCDs, each with its own L2.
// xcd_tile maps dispatch index b of nb to a logical index such that each XCD
// takes one contiguous run of logical indices (in order).
__device__ __forceinline__ int xcd_tile(int b, int nb)
{
    const int q = nb >> 3, rem = nb & 7, x = b & 7;
    return x * q + min(x, rem) + (b >> 3);
}

// x-fastest padded layout: a block per 256-voxel run along x, coalesced in x
// both ways (longer runs than 64 x 4 blocks: 49.5 against 57.7 us at paper
// scale).  FP32 at paper scale streams 297 MB (4.4 M voxels of 68 bytes) in
// 49 us, 6 TB/s with part of the model in the Infinity Cache; a BF16 model
// moves fewer bytes a load and was bound by the chain of waits until all of
// a voxel's loads went out together (load_fields, sample_f0): K = 4 at
// 256x256x128 102 -> 69 us, K = 5 at 512x512x160 520 -> 370 us (1.5 GB).
// (Ordering the runs by XCD, as the y-fastest tiles are, was 2-4 % slower here:
// in dispatch order the XCDs work on neighbouring rows at the same time and
// share their f0 taps through the Infinity Cache.)
template <typename R, typename S, typename F, int C, bool TAN, bool H, int KM>
__global__ void __launch_bounds__(256) k_warp_fused(const F* __restrict__ f0,
                                                    const S* __restrict__ mean,
                                                    const S* __restrict__ U, int K,
                                                    Chan<double, 8> w, VoxGrid g, int px, int py,
                                                    Chan<float, 8> hs, VoxBox b,
                                                    CellOf<R, C, H>* __restrict__ out)
{
    const int i = b.lo[0] + blockIdx.x * 256 + threadIdx.x, j = b.lo[1] + blockIdx.y;
    const int k = b.lo[2] + blockIdx.z;
    if (i >= b.hi[0] || j >= b.hi[1]) return;
    Chan<R, C> o = warp_cell<R, S, F, C, TAN, KM>(f0, mean, U, K, w, g, i, j, k);
    out[(size_t)(i + 1) + (size_t)px * ((size_t)(j + 1) + (size_t)py * (k + 1))] =
        store_cell<R, C, H>(o, hs);
}

// Width (x) of the y-fastest warp's tiles: the widest of 128, 64 or 32
// voxels whose 8-row tile of cells stays within about 8 KB of LDS, so that a
// block still finds room on a CU whose LDS the march's staging mostly holds
// (a serving engine runs both at once).
template <typename R, int C, bool H>
constexpr int yf_tile_x()
{
    constexpr int cb = (int)sizeof(CellOf<R, C, H>);
    return 8 * 128 * cb <= 8448 ? 128 : (8 * 64 * cb <= 8448 ? 64 : 32);
}

// y-fastest padded layout: a TX x 8 (x, y) tile per block, computed with
// x-contiguous reads (runs of 4 TX bytes of each field), staged in LDS and
// written as 8-cell runs along y.
template <typename R, typename S, typename F, int C, bool TAN, bool H, int KM>
__global__ void __launch_bounds__(256) k_warp_fused_yf(const F* __restrict__ f0,
                                                       const S* __restrict__ mean,
                                                       const S* __restrict__ U, int K,
                                                       Chan<double, 8> w, VoxGrid g, int px,
                                                       int py, Chan<float, 8> hs, VoxBox b,
                                                       int gx, int gy,
                                                       CellOf<R, C, H>* __restrict__ out)
{
    constexpr int TX = yf_tile_x<R, C, H>();
    __shared__ CellOf<R, C, H> tile[8][TX + 1];
    // tiles in XCD order: each XCD's L2 sees a contiguous band of tile rows,
    // so the f0 taps that neighbouring tiles share (displacements reach
    // several voxels) are fetched into one L2 (-7 % at 80-90 deg)
    const int lb = xcd_tile(blockIdx.x, gridDim.x);
    const int bx = lb % gx, rb = lb / gx;
    const int i0 = b.lo[0] + bx * TX, j0 = b.lo[1] + (rb % gy) * 8, k = b.lo[2] + rb / gy;
    const int t = threadIdx.x;
#pragma unroll
    for (int r = 0; r < TX / 32; ++r) {
        const int il = t % TX, jl = t / TX + (256 / TX) * r;
        const int i = i0 + il, j = j0 + jl;
        if (i < b.hi[0] && j < b.hi[1])
            tile[jl][il] = store_cell<R, C, H>(warp_cell<R, S, F, C, TAN, KM>(f0, mean, U, K, w, g, i, j, k), hs);
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < TX / 32; ++r) {
        const int jl = t & 7, il = (t >> 3) + 32 * r;
        const int i = i0 + il, j = j0 + jl;
        if (i < b.hi[0] && j < b.hi[1])
            out[(size_t)(j + 1) + (size_t)px * ((size_t)(i + 1) + (size_t)py * (k + 1))] = tile[jl][il];
    }
}

// The padded copy of a volume, zero borders included.  (A block takes more
// than one slice only of the longest grids, whose padded slices are more than
// a launch's blocks along z.)
template <typename R>
__global__ void __launch_bounds__(256) k_pad(const R* __restrict__ vol, VoxGrid g, R* __restrict__ pad)
{
    const int i = blockIdx.x * 64 + threadIdx.x, j = blockIdx.y * 4 + threadIdx.y;
    if (i >= g.nx + 3 || j >= g.ny + 3) return;
    for (int k = blockIdx.z; k < g.nz + 3; k += gridDim.z) {
        const bool in = (unsigned)(i - 1) < (unsigned)g.nx && (unsigned)(j - 1) < (unsigned)g.ny &&
                        (unsigned)(k - 1) < (unsigned)g.nz;
        pad[(size_t)i + (size_t)(g.nx + 3) * ((size_t)j + (size_t)(g.ny + 3) * k)] =
            in ? vol[(size_t)(i - 1) + (size_t)g.nx * ((size_t)(j - 1) + (size_t)g.ny * (k - 1))] : (R)0;
    }
}

__global__ void __launch_bounds__(256) k_zero16(uint4* __restrict__ p, size_t n16)
{
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    for (; i < n16; i += (size_t)gridDim.x * 256) p[i] = make_uint4(0, 0, 0, 0);
}

__global__ void __launch_bounds__(256) k_zero4(uint32_t* __restrict__ p, size_t n4)
{
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    for (; i < n4; i += (size_t)gridDim.x * 256) p[i] = 0u;
}

// ---------------------------------------------------------- ray march ----
template <typename R>
struct RaySeg {
    R q0[3];         // index-space point of sample 0
    R dq[3];         // index-space step per sample
    int first, end;  // the segment's samples
};

// One direction of the slab tests along a ray: the coordinate o + t d,
// with 1 / d and the offsets that fold the dilation into one FMA per bound:
// t = lo * inv + nlo is where the coordinate reaches lo - h, t = hi * inv + nhi
// where it reaches hi + h.  1 / d is the hardware reciprocal (1 ulp, far
// inside the half-cell slack of the dilation).  |d| < 1e-20 is taken as 1e-20
// (the coordinate moves by < 1e-16 index units over any ray): both bounds are
// then beyond the ray, on opposite sides if the coordinate lies between them.
struct SlabAxis {
    float inv, nlo, nhi;
    __device__ __forceinline__ void init(float o, float d, float h)
    {
        inv = __builtin_amdgcn_rcpf(copysignf(fmaxf(fabsf(d), 1e-20f), d));
        nlo = -(o + h) * inv;
        nhi = (h - o) * inv;
    }
    __device__ __forceinline__ void clip(float lo, float hi, float& ta, float& tb) const
    {
        const float t1 = fmaf(lo, inv, nlo), t2 = fmaf(hi, inv, nhi);
        ta = fmaxf(ta, fminf(t1, t2));
        tb = fminf(tb, fmaxf(t1, t2));
    }
};

// Narrows the box segment [tmin, tmax] of a ray (direction dq, index units
// per mm) to the hull of its intersections with the dilated slab regions:
// outside every one of them all of the ray's samples are exactly zero.  The
// bounds are evaluated in FP32: where a constraint binds, the rounding moves
// the cut point by ~1e-4 index units along that constraint's own axis,
// against the half-cell slack of the dilation.
__device__ __forceinline__ void refine_by_slabs(const RayGeom& g, const double dq[3], double& tmin,
                                                double& tmax)
{
    const double za = fma(tmin, dq[2], g.qs[2]), zb = fma(tmax, dq[2], g.qs[2]);
    // slab s (slices sT .. sT + T - 1) reaches k in [sT - h, sT + T - 1 + h]
    // (one slab more at each end covers the rounding of 1 / T)
    const float zlo = (float)fmin(za, zb) - g.h[2], zhi = (float)fmax(za, zb) + g.h[2];
    const float rT = __builtin_amdgcn_rcpf((float)g.slab_t), lim = (float)g.nslab + 2.0f;
    const int s0 = max(0, (int)floorf(fminf(fmaxf((zlo + 1.0f) * rT - 1.0f, -2.0f), lim)) - 1);
    const int s1 = min(g.nslab - 1, (int)floorf(fminf(fmaxf(fmaf(zhi, rT, 1e-3f), -2.0f), lim)));
    const float o0 = (float)g.qs[0], o1 = (float)g.qs[1], d0 = (float)dq[0], d1 = (float)dq[1];
    const float hd = g.h[0] + g.h[1];
    SlabAxis ax, ay, ap, am, az;
    ax.init(o0, d0, g.h[0]);
    ay.init(o1, d1, g.h[1]);
    ap.init(o0 + o1, d0 + d1, hd);
    am.init(o0 - o1, d0 - d1, hd);
    az.init((float)g.qs[2], (float)dq[2], g.h[2]);
    float tin = INFINITY, tout = -INFINITY;
    // (no branch in the loop, so that the loads of two slabs are in flight)
#pragma unroll 2
    for (int s = s0; s <= s1; ++s) {
        const float* b = g.slabs + 10 * s;
        float ta = -INFINITY, tb = INFINITY;
        az.clip(b[8], b[9], ta, tb);
        ax.clip(b[0], b[1], ta, tb);
        ay.clip(b[2], b[3], ta, tb);
        ap.clip(b[4], b[5], ta, tb);
        am.clip(b[6], b[7], ta, tb);
        const bool in = b[8] <= b[9] && ta <= tb;   // b[8] > b[9]: no nonzero voxel
        tin = in ? fminf(tin, ta) : tin;
        tout = in ? fmaxf(tout, tb) : tout;
    }
    tmin = fmax(tmin, (double)tin);
    tmax = fmin(tmax, (double)tout);
}

// 1 / x and 1 / sqrt(x) in FP64 (x normal and far from the ends of the
// range) from the hardware approximations, good to 2^-24 or better, and two
// Newton steps, each doubling the correct bits: within an ulp or two, at a
// third of the instructions of a division.
__device__ __forceinline__ double rcp64(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma(r, fma(-x, r, 1.0), r);
    return fma(r, fma(-x, r, 1.0), r);
}
__device__ __forceinline__ double rsq64(double x)
{
    double r = __builtin_amdgcn_rsq(x);
    r = fma(0.5 * r, fma(-x * r, r, 1.0), r);
    return fma(0.5 * r, fma(-x * r, r, 1.0), r);
}

// Global sample range [n0, n1] of ray (iu, iv) (n1 < n0: none) on the grid
// t = n dt, clipped to the box (at most the support [-1, n_a] of the
// interpolant) and the slabs, widened by one sample at each end (samples
// outside the support are clamped onto zero cells), and the ray's direction
// (index units per mm).  FP64, once per ray.
struct RayRange {
    int n0, n1;
    double dq[3];
};

// R: the precision in which the ray's positions are formed.
template <typename R>
__device__ __forceinline__ RayRange ray_range(const RayGeom& g, int iu, int iv)
{
    RayRange r;
    r.n0 = 0;
    r.n1 = -1;
    r.dq[0] = r.dq[1] = r.dq[2] = 0.0;
    double u = g.u0 + iu * g.du, v = g.v0 + iv * g.dv;
    double D[3], L2 = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        D[a] = g.qc[a] + u * g.eu[a] + v * g.ev[a] - g.qs[a];
        double w = D[a] * g.sp[a];
        L2 += w * w;
    }
    if (!(L2 > 0.0)) return r;
    const double iL = rsq64(L2);
    // the length and its quotient by dt (and in FP64 the quotients by it)
    // corrected once more: correctly rounded, as by sqrt and /, so that a
    // sample exactly on the detector is kept or dropped as by those, and FP64
    // positions far along a ray are as exact
    double L = L2 * iL;
    L = fma(0.5 * iL, fma(-L, L, L2), L);
    double nl = L * g.inv_dt;
    nl = fma(g.inv_dt, fma(-nl, g.dt, L), nl);
    double tmin = 0.0, tmax = L;
    bool hit = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        double d = D[a] * iL;
        if constexpr (std::is_same<R, double>::value) d = fma(iL, fma(-d, L, D[a]), d);
        r.dq[a] = d;
        if (fabs(d) > 1e-280) {
            const double i = rcp64(d);
            const double t1 = (g.clo[a] - g.qs[a]) * i, t2 = (g.chi[a] - g.qs[a]) * i;
            tmin = fmax(tmin, fmin(t1, t2));
            tmax = fmin(tmax, fmax(t1, t2));
        } else if (!(g.qs[a] > g.clo[a] && g.qs[a] < g.chi[a])) {
            hit = false;
        }
    }
    if (g.slabs && hit && tmin <= tmax) refine_by_slabs(g, r.dq, tmin, tmax);
    if (!hit || !(tmin <= tmax)) return r;
    // (L / dt is below 2^31: checked with the geometry)
    const double n0 = fmax(ceil(tmin * g.inv_dt) - 1.0, 0.0);
    const double n1 = fmin(floor(tmax * g.inv_dt) + 1.0, floor(nl));
    if (n1 >= n0) {
        r.n0 = (int)n0;
        r.n1 = (int)n1;
    }
    return r;
}

// The ray's range split into `seg` equal segments: segment `sid`.  Positions
// are formed from the start of a quarter of the ray at most: more segments
// than four split a quarter's samples, and share its start, so that a sample
// lies at the same point however many threads a ray has (with starts of their
// own, sixteen segments had 3 % more error against 80-bit projections).
template <typename R>
__device__ __forceinline__ RaySeg<R> ray_segment(const RayGeom& g, int iu, int iv, int seg, int sid)
{
    RaySeg<R> r;
    const RayRange rr = ray_range<R>(g, iu, iv);
    const long cnt = rr.n1 >= rr.n0 ? (long)rr.n1 - rr.n0 + 1 : 0;
    // (seg is a power of two: np parts of `per` segments)
    const int np = min(__builtin_ctz(seg), 2), per = __builtin_ctz(seg) - np, p = sid >> per, c = sid & ((1 << per) - 1);
    const long m0 = cnt * p >> np, n = (cnt * (p + 1) >> np) - m0;
    r.first = (int)(n * c >> per);
    r.end = (int)(n * (c + 1) >> per);
    double t0 = (double)(rr.n0 + m0) * g.dt;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        r.q0[a] = (R)(g.qs[a] + t0 * rr.dq[a]);
        r.dq[a] = (R)(g.dt * rr.dq[a]);
    }
    return r;
}

__device__ __forceinline__ void ray_of_thread(const MarchShape& ms, int tiles_u, int& iu, int& iv,
                                              int& sid, int& rloc)
{
    const int rpb = 256 / ms.seg;
    rloc = threadIdx.x % rpb;
    sid = threadIdx.x / rpb;
    const int tv_rows = rpb / ms.tile_u;
    int tu = blockIdx.x % tiles_u, tv = blockIdx.x / tiles_u;
    iu = tu * ms.tile_u + rloc % ms.tile_u;
    iv = tv * tv_rows + rloc / ms.tile_u;
}

// Ray march over the padded image; p and moments per ray.
template <typename R, int C>
__global__ void __launch_bounds__(256) k_march(RayGeom g, MarchShape ms, int tiles_u,
                                               const Chan<R, C>* __restrict__ vol, int px,
                                               int py, float fnx, float fny, float fnz, int kc,
                                               const R* __restrict__ y, R* __restrict__ p_out,
                                               double* __restrict__ partials)
{
    int iu, iv, sid, rloc;
    ray_of_thread(ms, tiles_u, iu, iv, sid, rloc);
    const bool valid = iu < g.nu && iv < g.nv;
    R acc[C];
#pragma unroll
    for (int c = 0; c < C; ++c) acc[c] = (R)0;
    int nsamp = 0;
    if (valid) {
        RaySeg<R> rs = ray_segment<R>(g, iu, iv, ms.seg, sid);
        nsamp = rs.end - rs.first;
        const long pxy = (long)px * py;
        const Chan<R, C>* base = vol + (1 + px + pxy);   // cell of voxel (0,0,0)
        // (two samples' loads in flight, for one channel: FP64 256x256x100 onto
        // 512x384 pixels at 11 / 46 / 86 deg 196 / 234 / 158 -> 174 / 204 / 158
        // us; four take the registers: 205 / 249 / 188)
        constexpr int kUnroll = C == 1 ? 2 : 1;
#pragma unroll kUnroll
        for (int m = rs.first; m < rs.end; ++m) {
            R fm = (R)m;
            R qx = clampv(fma(fm, rs.dq[0], rs.q0[0]), (R)-1, (R)fnx);
            R qy = clampv(fma(fm, rs.dq[1], rs.q0[1]), (R)-1, (R)fny);
            R qz = clampv(fma(fm, rs.dq[2], rs.q0[2]), (R)-1, (R)fnz);
            R flx = floor(qx), fly = floor(qy), flz = floor(qz);
            int ix = (int)flx, iy = (int)fly, iz = (int)flz;
            R ax = qx - flx, ay = qy - fly, az = qz - flz;
            R bx = (R)1 - ax, by = (R)1 - ay, bz = (R)1 - az;
            R w00 = by * bz, w10 = ay * bz, w01 = by * az, w11 = ay * az;
            const Chan<R, C>* c0 = base + ((long)ix + (long)px * iy + pxy * iz);
            Chan<R, C> t000 = c0[0], t100 = c0[1], t010 = c0[px], t110 = c0[px + 1];
            Chan<R, C> t001 = c0[pxy], t101 = c0[pxy + 1], t011 = c0[pxy + px],
                       t111 = c0[pxy + px + 1];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                R x00 = bx * t000.v[c] + ax * t100.v[c];
                R x10 = bx * t010.v[c] + ax * t110.v[c];
                R x01 = bx * t001.v[c] + ax * t101.v[c];
                R x11 = bx * t011.v[c] + ax * t111.v[c];
                acc[c] += w00 * x00 + w10 * x10 + w01 * x01 + w11 * x11;
            }
        }
    }
    if (ms.seg > 1) {
        __shared__ R segbuf[256 * C];
#pragma unroll
        for (int c = 0; c < C; ++c) segbuf[threadIdx.x * C + c] = acc[c];
        __syncthreads();
        if (sid == 0) {
            const int rpb = 256 / ms.seg;
            for (int s = 1; s < ms.seg; ++s)
#pragma unroll
                for (int c = 0; c < C; ++c) acc[c] += segbuf[(threadIdx.x + s * rpb) * C + c];
        }
    }
    const bool owner = valid && sid == 0;
    const R dt = (R)g.dt;
    if (owner && p_out) p_out[iu + (size_t)g.nu * iv] = dt * acc[0];
    if (partials) {
        // record per block: the moments, then the number of samples marched
        constexpr int NM = 5 + 3 * (C - 1);
        double m[NM + 1];
#pragma unroll
        for (int i = 0; i < NM; ++i) m[i] = 0.0;
        m[NM] = (double)nsamp;
        if (owner) {
            double yd = (double)y[iu + (size_t)g.nu * iv];
            double pd = (double)(dt * acc[0]);
            m[0] = yd;
            m[1] = yd * yd;
            m[2] = pd;
            m[3] = yd * pd;
            m[4] = pd * pd;
#pragma unroll
            for (int k = 0; k < C - 1; ++k) {
                if (k + 1 < kc) {
                    double tk = (double)(dt * acc[k + 1]);
                    m[5 + 3 * k] = pd * tk;
                    m[6 + 3 * k] = yd * tk;
                    m[7 + 3 * k] = tk;
                }
            }
        }
        block_sum_store<NM + 1>(m, NM + 1, partials + blockIdx.x, (int)gridDim.x);
    }
}

// ---------------------------------------------------- FP32 ray march ----
// (Blocks go to the XCDs round-robin: xcd_tile, defined with the warps,
// gives each XCD one contiguous band of detector rows, so that the rays
// sharing an XCD's L2 cross the same part of the volume.)

// The march's tile (tu, tv) of dispatch index b: within each XCD's band of
// rows (xcd_tile) the tiles go from the middle column outwards.  The rays
// through the middle of the volume are the longest, and a block takes about
// half the launch's time: with the long blocks first the short ones fill in
// at the end (1833 -> 1805 us a solve at 256x256x100).  With a shifted detector
// or isocentre the middle column need not be the longest; the order then
// gains less, and the sums are the same.
__device__ __forceinline__ void march_tile(int b, int nb, int tiles_u, int& tu, int& tv)
{
    const int q = nb >> 3, rem = nb & 7, x = b & 7;
    const int s = x * q + min(x, rem), n = q + (x < rem ? 1 : 0), i = b >> 3;
    const int k = n / tiles_u;
    int t = s + i;
    if (i < k * tiles_u) {
        const int r = i / k, c = tiles_u >> 1;
        int col = (r & 1) ? c - ((r + 1) >> 1) : c + (r >> 1);
        col -= s % tiles_u;
        if (col < 0) col += tiles_u;
        t = s + col + (i - r * k) * tiles_u;
    }
    tv = t / tiles_u;
    tu = t - tv * tiles_u;
}

// One padded cell pair (x and x+1) of C float channels.
template <int C>
struct CellPair {
    float a[C], b[C];
};
// The pair at byte offset `off` from `base` (plain global loads).
template <int C>
__device__ __forceinline__ CellPair<C> load_pair_g(const char* base, int off)
{
    CellPair<C> p;
    const float* a = (const float*)(base + off);
#pragma unroll
    for (int c = 0; c < C; ++c) {
        p.a[c] = a[c];
        p.b[c] = a[C + c];
    }
    return p;
}

// Same pair from FP16 cells (values as stored: times the channel scale).
typedef _Float16 h4v __attribute__((ext_vector_type(4)));
typedef _Float16 h8v __attribute__((ext_vector_type(8)));
template <int C>
__device__ __forceinline__ CellPair<C> load_pair_h(const char* base, int off)
{
    CellPair<C> p;
    if constexpr (C == 2) {
        h4v v;
        __builtin_memcpy(&v, base + off, sizeof v);
        p.a[0] = (float)v[0];
        p.a[1] = (float)v[1];
        p.b[0] = (float)v[2];
        p.b[1] = (float)v[3];
    } else {
#pragma unroll
        for (int h = 0; h < C / 4; ++h) {
            // cells x and x+1 are adjacent: 2 C halves, read 8 at a time
            h8v v;
            __builtin_memcpy(&v, base + off + 16 * h, sizeof v);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int idx = 8 * h + e;       // half index within the pair
                if (idx < C) p.a[idx] = (float)v[e];
                else p.b[idx - C] = (float)v[e];
            }
        }
    }
    return p;
}

struct MarchArgs {
    RayGeom g;
    MarchShape ms;
    int tiles_u;
    const void* vol;       // padded image, C float channels per cell
    int px, py, pz;        // padded dims in memory order (cells)
    int ys, zs;            // byte strides of the padded y and z axes (offsets are
                           // 32-bit: march_f32_fits bounds the image)
    float fn1[3];          // clamp bound n_a + 1 (padded index space)
    int kc;                // channels used
    const float* y;        // measured projection (moments) or null
    float* p_out;          // projection out or null
    double* partials;      // [NM][blocks] (slot-major) or null
    // the final moments and their publication, where the last block sums them
    double* moments;
    unsigned* arrived;
    unsigned long long* done;
    unsigned long long seq;
    float ihs[8];          // FP16 cells: 1 / channel scale
};

// The march of FP16 cells, gathering its taps through the vector L1 (where the
// VALU binds: FP32 cells, which the L1 bound, go to the LDS-staged k_march_lds
// below).  It got neither the staging nor the tile order of that kernel: at
// 30 deg and K = 3 it takes 149 us, the staged march of FP32 cells 127.
template <int C>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(C <= 4 ? 8 : 1))) k_march_f16(MarchArgs A)
{
    constexpr int CB = 2 * C;   // bytes per cell
    const RayGeom& g = A.g;
    const int rpb = 256 / A.ms.seg;
    const int rloc = threadIdx.x % rpb, sid = threadIdx.x / rpb;
    const int rows = rpb / A.ms.tile_u;
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    const int tu = tile % A.tiles_u, tv = tile / A.tiles_u;
    const int iu = tu * A.ms.tile_u + rloc % A.ms.tile_u;
    const int iv = tv * rows + rloc / A.ms.tile_u;
    const bool valid = iu < g.nu && iv < g.nv;
    float acc[C];
#pragma unroll
    for (int c = 0; c < C; ++c) acc[c] = 0.f;
    int nsamp = 0;
    // The wave marches the union of its rays' sample ranges in step: at each
    // iteration all its lanes sit at the same global sample index n (t = n
    // dt), so neighbouring rays read neighbouring cells and share cache
    // lines; a lane skips the indices outside its own ray's range.  The waves
    // holding the same 64 rays (one per segment) split the union into equal
    // parts, so each sample of a ray is taken exactly once.
    RayRange rr;
    rr.n0 = 0;
    rr.n1 = -1;
    rr.dq[0] = rr.dq[1] = rr.dq[2] = 0.0;
    // LDS: first the block's ray set-ups, then the segments' partial sums
    constexpr int kSeg = 256 * (C + 1) * 4;   // gather_segments
    constexpr int kSmem = kSeg > 128 * (int)sizeof(RayRange) ? kSeg : 128 * (int)sizeof(RayRange);
    __shared__ __align__(16) char smem[kSmem];
    if (A.ms.seg > 1) {
        // the segment-0 waves set up the block's rays, the others read them
        RayRange* rbuf = (RayRange*)smem;
        if (sid == 0) {
            if (valid) rr = ray_range<float>(g, iu, iv);
            rbuf[rloc] = rr;
        }
        __syncthreads();
        rr = rbuf[rloc];
        __syncthreads();   // before the buffer is reused for the partial sums
    } else if (valid) {
        rr = ray_range<float>(g, iu, iv);
    }
    int N0 = rr.n1 >= rr.n0 ? rr.n0 : INT_MAX, N1 = rr.n1 >= rr.n0 ? rr.n1 : INT_MIN;
    N0 = __builtin_amdgcn_readfirstlane(__ockl_wfred_min_i32(N0));
    N1 = __builtin_amdgcn_readfirstlane(__ockl_wfred_max_i32(N1));
    if (N0 <= N1) {
        const long span = (long)N1 - N0 + 1;
        const int na = __builtin_amdgcn_readfirstlane(N0 + (int)(span * sid / A.ms.seg));
        const int nb = __builtin_amdgcn_readfirstlane(N0 + (int)(span * (sid + 1) / A.ms.seg));
        // padded index space: cell i+1 holds voxel i, so q + 1 >= 0 after the
        // clamp and truncation is the floor
        const double ta = (double)na * g.dt;
        const float q0x = (float)(g.qs[0] + ta * rr.dq[0]) + 1.f;
        const float q0y = (float)(g.qs[1] + ta * rr.dq[1]) + 1.f;
        const float q0z = (float)(g.qs[2] + ta * rr.dq[2]) + 1.f;
        const float dqx = (float)(g.dt * rr.dq[0]), dqy = (float)(g.dt * rr.dq[1]),
                    dqz = (float)(g.dt * rr.dq[2]);
        const int YS = A.ys, ZS = A.zs, YZ = A.ys + A.zs, PY = A.py;
        // (a lane loads at every sample, though consecutive ones often fall in
        // the same cell: a branch would cost more than the bandwidth it saves)
        for (int n = na; n < nb; ++n) {
            if (n < rr.n0 || n > rr.n1) continue;
            ++nsamp;
            const float fm = (float)(n - na);
            float qx = __builtin_amdgcn_fmed3f(fmaf(fm, dqx, q0x), 0.f, A.fn1[0]);
            float qy = __builtin_amdgcn_fmed3f(fmaf(fm, dqy, q0y), 0.f, A.fn1[1]);
            float qz = __builtin_amdgcn_fmed3f(fmaf(fm, dqz, q0z), 0.f, A.fn1[2]);
            const int ix = (int)qx, iy = (int)qy, iz = (int)qz;
            const float ax = __builtin_amdgcn_fractf(qx), ay = __builtin_amdgcn_fractf(qy),
                        az = __builtin_amdgcn_fractf(qz);
            // (iz py + iy) < 2^24 and YS < 2^24, and every offset is below
            // the image size < 2^31 (checked at launch), so the 24-bit
            // products are exact
            const int voff = ix * CB + (int)__umul24(__umul24(iz, PY) + iy, YS);
            const char* vb = (const char*)A.vol;
            const CellPair<C> p00 = load_pair_h<C>(vb, voff), p10 = load_pair_h<C>(vb, voff + YS),
                              p01 = load_pair_h<C>(vb, voff + ZS), p11 = load_pair_h<C>(vb, voff + YZ);
            const float bx = 1.f - ax, by = 1.f - ay, bz = 1.f - az;
            const float w00 = by * bz, w10 = ay * bz, w01 = by * az, w11 = ay * az;
            const float w000 = bx * w00, w100 = ax * w00, w010 = bx * w10, w110 = ax * w10;
            const float w001 = bx * w01, w101 = ax * w01, w011 = bx * w11, w111 = ax * w11;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                float t = acc[c];
                t = fmaf(w000, p00.a[c], t);
                t = fmaf(w100, p00.b[c], t);
                t = fmaf(w010, p10.a[c], t);
                t = fmaf(w110, p10.b[c], t);
                t = fmaf(w001, p01.a[c], t);
                t = fmaf(w101, p01.b[c], t);
                t = fmaf(w011, p11.a[c], t);
                t = fmaf(w111, p11.b[c], t);
                acc[c] = t;
            }
        }
    }
    if (A.ms.seg > 1) gather_segments<C, 256>(smem, A.ms.seg, rpb, sid, acc, nsamp);
#pragma unroll
    for (int c = 0; c < C; ++c) acc[c] *= A.ihs[c];   // exact: powers of two
    const bool owner = valid && sid == 0;
    const float dt = (float)g.dt;
    if (owner && A.p_out) A.p_out[iu + (size_t)g.nu * iv] = dt * acc[0];
    if (A.partials) {
        // record per block: the moments, then the number of samples marched
        constexpr int NM = 5 + 3 * (C - 1);
        double mo[NM + 1];
#pragma unroll
        for (int i = 0; i < NM; ++i) mo[i] = 0.0;
        mo[NM] = sid == 0 ? (double)nsamp : 0.0;   // segments were gathered
        if (owner) {
            double yd = (double)A.y[iu + (size_t)g.nu * iv];
            double pd = (double)(dt * acc[0]);
            mo[0] = yd;
            mo[1] = yd * yd;
            mo[2] = pd;
            mo[3] = yd * pd;
            mo[4] = pd * pd;
#pragma unroll
            for (int k = 0; k < C - 1; ++k) {
                if (k + 1 < A.kc) {
                    double tk = (double)(dt * acc[k + 1]);
                    mo[5 + 3 * k] = pd * tk;
                    mo[6 + 3 * k] = yd * tk;
                    mo[7 + 3 * k] = tk;
                }
            }
        }
        block_sum_store<NM + 1>(mo, NM + 1, A.partials + blockIdx.x, (int)gridDim.x, rpb / 64);
    }
}

// ------------------------------------------ FP32 ray march, LDS-staged ----
// The march of FP32 cells: rays per wave, segments and sample positions as in
// k_march_f16, but each wave gathers its taps from a private LDS copy of
// the cells it is about to sample instead of through the vector L1.  The
// wave's sample range is cut into chunks of S sample indices; for each chunk
// the wave finds the index box of the cells its rays can read (from the
// extremes of the rays' coefficients, see below), copies that box from the
// image to LDS with loads that go there directly, whole rows along the
// fastest axis, and marches the chunk out of LDS.  A chunk whose box exceeds
// the wave's buffer is retried at half the length; at the shortest length it
// falls back to gathering through the L1.  A short box grows the next chunk.
// Each staged cell serves ~40 sample taps at paper scale, so the L1 sees a few
// coalesced row loads per chunk instead of 8 scattered cells per sample.
//
// What bounds it: VALU issue first (1.05 wave-instructions per CU and clock at
// 30 deg; independent FMAs alone reach 1.48), then the LDS reads (0.56 of the
// clocks).  Hence the chunk set-up without wave reductions or divisions (the
// box cost six reductions a chunk and the copy 19 instructions per 64 cells),
// no clamps where the box lies inside the image, and no registers or waits in
// the copy.  Measured (march alone, before -> now): K = 3 at 256x256x100,
// 512x384 pixels, 57 deg: 160.5 -> 144 us (136 with the ray set-up and the
// moments of today); one channel there: 163 -> 140 us (126 from the unpadded
// volume); K = 4 at 256x256x128: 205 -> 172 us (168); K = 5 at 512x512x160,
// 1024x768 pixels: 1531 -> 1227 us.  Most of the gain at K = 4 and 5 is the staging of 24-byte
// cells as planes of 16 and 4 bytes: three 8-byte reads a cell pair kept the
// LDS busy 0.77 of the clocks, 16 + 4 byte reads 0.55.
// LDS per wave: six 256-thread blocks per CU at C <= 4 (72 VGPRs), five at
// C = 6 (83-94 VGPRs), four at C = 8 (108 VGPRs), the most that the
// registers allow in each case.
template <int C>
constexpr int stage_bytes() { return C <= 6 ? 6144 : 9216; }
template <int C>
constexpr int march_waves_per_eu() { return C <= 4 ? 6 : (C <= 6 ? 5 : 4); }

// a * b + c with a, b < 2^24 in one v_mad_u32_u24 (b wave-uniform; left to
// itself the compiler spreads a two-term cell offset over more instructions)
__device__ __forceinline__ unsigned mad_u24(int a, unsigned b, unsigned c)
{
    unsigned d;
    asm("v_mad_u32_u24 %0, %1, %2, %3" : "=v"(d) : "v"(a), "s"(b), "v"(c));
    return d;
}

// floor(x / d) for 0 <= x < 2^21 and d >= 1, given rd = rcp(d) from the
// hardware reciprocal (within 1 ulp): (x + 0.5) rd is within 2^-22 relative
// of (x + 0.5) / d, less than 0.5 / d absolute, and (x + 0.5) / d lies at
// least 0.5 / d from every integer, so truncation gives the exact quotient.
__device__ __forceinline__ int small_quot(int x, float rd)
{
    return (int)(((float)x + 0.5f) * rd);
}

// A wave's staging buffer: the KC used channels of C-channel cells in planes
// that a load to LDS can fill, n16 planes of 16-byte quadruples of channels,
// then n4 planes of single channels (the fifth and sixth channel of 24-byte
// cells, which the LDS serves faster as 16 + 4 bytes than as three 8-byte
// pieces; all of a cell of one or two channels).  `buf` cells fit.
template <int C, int KC>
struct Stage {
    static constexpr int n16 = C / 4, n4 = C % 4 ? KC - 4 * n16 : 0;
    static constexpr int bytes = stage_bytes<C>(), buf = bytes / (16 * n16 + 4 * n4) & ~3;
    static constexpr int single = 16 * n16 * buf;   // where the single-channel planes start
    // a cell index is kept in bytes of the planes that are read most simply
    static constexpr int unit = n4 ? 4 : 16;
};

// The cells x and x + 1 at the position `loc` (unit bytes a cell, from the
// start of the first plane of that unit) of the staging buffer at byte `own`
// of the block's LDS.
template <int C, int KC>
__device__ __forceinline__ void lds_pair(const char* st, unsigned own, unsigned loc, CellPair<C>& P)
{
    using G = Stage<C, KC>;
#pragma unroll
    for (int h = 0; h < G::n16; ++h) {
        // (loc holds `own` already, in the unit of the single-channel planes
        // together with their offset)
        const unsigned at = G::unit == 16 ? loc : (loc << 2) + (own - 4u * (own + G::single));
        const float4* q = (const float4*)(st + at + h * 16 * G::buf);
        const float4 u = q[0], v = q[1];
        P.a[4 * h] = u.x; P.a[4 * h + 1] = u.y; P.a[4 * h + 2] = u.z; P.a[4 * h + 3] = u.w;
        P.b[4 * h] = v.x; P.b[4 * h + 1] = v.y; P.b[4 * h + 2] = v.z; P.b[4 * h + 3] = v.w;
    }
#pragma unroll
    for (int j = 0; j < G::n4; ++j) {
        const float* q = (const float*)(st + loc + 4 * G::buf * j);
        P.a[4 * G::n16 + j] = q[0];
        P.b[4 * G::n16 + j] = q[1];
    }
}

// A wave-uniform integer moved to a scalar register (opaque, or the compiler
// moves the conversion behind it and the arithmetic stays on the VALU).
__device__ __forceinline__ int scalar(int v)
{
    asm("" : "+v"(v));
    return __builtin_amdgcn_readfirstlane(v);
}

// Copies `B` bytes (4 or 16) a lane from each lane's `src` to the LDS at the
// wave-uniform dst + B x lane, asynchronously (counted by vmcnt).
template <int B>
__device__ __forceinline__ void load_to_lds(const char* src, float* dst)
{
    typedef const __attribute__((address_space(1))) void* G;
    typedef __attribute__((address_space(3))) void* L;
    static_assert(B == 4 || B == 16, "sizes of a load to LDS");
    if constexpr (B == 4) __builtin_amdgcn_global_load_lds((G)src, (L)dst, 4, 0, 0);
    else __builtin_amdgcn_global_load_lds((G)src, (L)dst, 16, 0, 0);
}

// KC: the channels whose sums are used (A.kc: the moments and the projection
// read only those; the others stay zero); the sample loop accumulates only
// these, so a 5-channel image stored in 6-channel cells (K = 4) does not pay
// for the channel it does not use.
// NW: waves per block, the ray segments times the block's 64-ray tiles.
// RAW (C = 1): the image is the caller's unpadded volume, and cells outside
// it are staged as zeros, so a projection needs no padded copy.
// SUM: the last block forms the final moments (few blocks; a branch in one
// kernel for both cost the large launches 0.7 %).
template <int C, int KC = C, int NW = 4, bool RAW = false, bool SUM = false>
__global__ void __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(march_waves_per_eu<C>()))) k_march_lds(MarchArgs A)
{
    static_assert(KC >= 1 && KC <= C, "used channels");
    static_assert(!RAW || C == 1, "a raw image has one channel");
    constexpr int T = 64 * NW;
    constexpr int CB = 4 * C;                    // bytes per cell
    constexpr int kStageBytes = stage_bytes<C>();
    using G = Stage<C, KC>;
    constexpr int BUF = G::buf;                  // cells per wave
    const RayGeom& g = A.g;
    const int rpb = T / A.ms.seg;
    const int rloc = threadIdx.x % rpb, sid = threadIdx.x / rpb;
    const int rows = rpb / A.ms.tile_u;
    int tu, tv;
    march_tile(blockIdx.x, gridDim.x, A.tiles_u, tu, tv);
    const int iu = tu * A.ms.tile_u + rloc % A.ms.tile_u;
    const int iv = tv * rows + rloc / A.ms.tile_u;
    const bool valid = iu < g.nu && iv < g.nv;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    float acc[C];
#pragma unroll
    for (int c = 0; c < C; ++c) acc[c] = 0.f;
    int nsamp = 0;
    RayRange rr;
    rr.n0 = 0;
    rr.n1 = -1;
    rr.dq[0] = rr.dq[1] = rr.dq[2] = 0.0;
    // LDS: the block's ray set-ups, then the waves' staging buffers, then
    // the segments' partial sums (one after the other, so they share it)
    constexpr int kStage = NW * kStageBytes;
    constexpr int kSeg = T * (C + 1) * 4;   // gather_segments
    constexpr int kRest = kSeg > 128 * (int)sizeof(RayRange) ? kSeg : 128 * (int)sizeof(RayRange);
    constexpr int kSmem = kStage > kRest ? kStage : kRest;
    __shared__ __align__(16) char smem[kSmem];
    if (A.ms.seg > 1) {
        RayRange* rbuf = (RayRange*)smem;
        if (sid == 0) {
            if (valid) rr = ray_range<float>(g, iu, iv);
            rbuf[rloc] = rr;
        }
        __syncthreads();
        rr = rbuf[rloc];
        __syncthreads();   // before the buffer is reused for staging
    } else if (valid) {
        rr = ray_range<float>(g, iu, iv);
    }
    int N0 = rr.n1 >= rr.n0 ? rr.n0 : INT_MAX, N1 = rr.n1 >= rr.n0 ? rr.n1 : INT_MIN;
    N0 = __builtin_amdgcn_readfirstlane(__ockl_wfred_min_i32(N0));
    N1 = __builtin_amdgcn_readfirstlane(__ockl_wfred_max_i32(N1));
    float* st = (float*)(smem + wave * kStageBytes);
    if (N0 <= N1) {
        const long span = (long)N1 - N0 + 1;
        const int na = __builtin_amdgcn_readfirstlane(N0 + (int)(span * sid / A.ms.seg));
        const int nb = __builtin_amdgcn_readfirstlane(N0 + (int)(span * (sid + 1) / A.ms.seg));
        const double ta = (double)na * g.dt;
        const float q0x = (float)(g.qs[0] + ta * rr.dq[0]) + 1.f;
        const float q0y = (float)(g.qs[1] + ta * rr.dq[1]) + 1.f;
        const float q0z = (float)(g.qs[2] + ta * rr.dq[2]) + 1.f;
        const float dqx = (float)(g.dt * rr.dq[0]), dqy = (float)(g.dt * rr.dq[1]),
                    dqz = (float)(g.dt * rr.dq[2]);
        const int YS = A.ys, ZS = A.zs, YZ = A.ys + A.zs, PY = RAW ? A.py - 3 : A.py;
        const char* vb = (const char*)A.vol;
        // The extremes over the wave's rays of a position's two coefficients
        // bound all its positions: every ray starts at the source, so per
        // axis the ray with the smallest step also has the smallest offset at
        // na, and fma is monotone in each operand, rounding included (f >= 0).
        // Lane 0..2 (axis x, y, z) holds the lower bound's (offset, step),
        // lane 3..5 the negated upper bound's, so one minimum serves both.
        const bool any = rr.n1 >= rr.n0;
        float bq, bd, bn;
        {
            const float big = 3.0e38f;
            const float e[6] = {q0x, q0y, q0z, -q0x, -q0y, -q0z}, d[6] = {dqx, dqy, dqz, -dqx, -dqy, -dqz};
            bq = bd = 0.f;
#pragma unroll
            for (int i = 0; i < 6; ++i) {
                const float mq = wave_min(any ? e[i] : big), md = wave_min(any ? d[i] : big);
                bq = lane == i ? mq : bq;
                bd = lane == i ? md : bd;
            }
            const int ax = lane >= 3 ? lane - 3 : lane;
            bn = ax == 0 ? A.fn1[0] : (ax == 1 ? A.fn1[1] : A.fn1[2]);
        }
        // the chunk's samples: positions, weights and order as in
        // k_march_f16; a lane reloads its cells P (the pairs at +0, +y,
        // +z, +y+z) only when they change
        // (fm: the sample's index relative to na, as a float; clamp: positions
        // may lie outside the support and are clamped to it -- wave-uniform)
        auto step = [&](bool clamp, float fm, CellPair<C> (&P)[4], auto&& load) {
            float qx = fmaf(fm, dqx, q0x), qy = fmaf(fm, dqy, q0y), qz = fmaf(fm, dqz, q0z);
            if (clamp) {
                // (opaque, or the branch would become clamps and selects)
                asm volatile("" : "+v"(qx), "+v"(qy), "+v"(qz));
                qx = __builtin_amdgcn_fmed3f(qx, 0.f, A.fn1[0]);
                qy = __builtin_amdgcn_fmed3f(qy, 0.f, A.fn1[1]);
                qz = __builtin_amdgcn_fmed3f(qz, 0.f, A.fn1[2]);
            }
            const int ix = (int)qx, iy = (int)qy, iz = (int)qz;
            const float ax = __builtin_amdgcn_fractf(qx), ay = __builtin_amdgcn_fractf(qy),
                        az = __builtin_amdgcn_fractf(qz);
            load(ix, iy, iz);
            // (one product a weight: forming each pair from a product and a
            // difference saves two of the loop's ~66 instructions, but a
            // solve carries the other rounding through its line searches)
            const float bx = 1.f - ax, by = 1.f - ay, bz = 1.f - az;
            const float w00 = by * bz, w10 = ay * bz, w01 = by * az, w11 = ay * az;
            const float w000 = bx * w00, w100 = ax * w00, w010 = bx * w10, w110 = ax * w10;
            const float w001 = bx * w01, w101 = ax * w01, w011 = bx * w11, w111 = ax * w11;
#pragma unroll
            for (int c = 0; c < KC; ++c) {
                float t = acc[c];
                t = fmaf(w000, P[0].a[c], t);
                t = fmaf(w100, P[0].b[c], t);
                t = fmaf(w010, P[1].a[c], t);
                t = fmaf(w110, P[1].b[c], t);
                t = fmaf(w001, P[2].a[c], t);
                t = fmaf(w101, P[2].b[c], t);
                t = fmaf(w011, P[3].a[c], t);
                t = fmaf(w111, P[3].b[c], t);
                acc[c] = t;
            }
        };
        int S = 16;
        bool gather = false;   // the rest of the range through the L1
        int c0 = na;
        while (c0 < nb) {
            // the chunk [c0, c1) and the box of the cells its samples read;
            // a box beyond the buffer is retried at half the length (in a
            // loop of its own, so the chunk loop has a single way round)
            int c1, lo0, lo1, lo2, dx, dy, dz, dxy, cells;
            bool inside;   // no position of the chunk needs the clamp
            for (;;) {
                c1 = min(nb, c0 + S);
                const float fa = (float)(c0 - na), fb = (float)(c1 - 1 - na);
                float v = fminf(fmaf(fa, bd, bq), fmaf(fb, bd, bq));
                v = lane >= 3 ? -v : v;
                const float vc = __builtin_amdgcn_fmed3f(v, 0.f, bn);
                inside = (__ballot(v == vc) & 63u) == 63u;
                const int iv = (int)vc;
                lo0 = __builtin_amdgcn_readlane(iv, 0);
                lo1 = __builtin_amdgcn_readlane(iv, 1);
                lo2 = __builtin_amdgcn_readlane(iv, 2);
                dx = __builtin_amdgcn_readlane(iv, 3) - lo0 + 2;
                dy = __builtin_amdgcn_readlane(iv, 4) - lo1 + 2;
                dz = __builtin_amdgcn_readlane(iv, 5) - lo2 + 2;
                dxy = dx * dy;
                cells = dxy * dz;
                // (each extent on its own first: the products may overflow)
                const bool fits = dx <= BUF && dy <= BUF && dz <= BUF && dxy <= BUF && cells <= BUF;
                if (fits) break;
                cells = BUF + 1;
                if (S <= 4) break;
                S >>= 1;
            }
            if (cells > BUF) {
                // the rays spread too far for the buffer even over 4 samples
                // (coarse detectors): gather the rest through the L1
                gather = true;
                break;
            }
            // this lane's samples in the chunk
            const int s_lo = max(c0, rr.n0), s_hi = min(c1 - 1, rr.n1);
            const unsigned long long some = __ballot(s_lo <= s_hi);
            if (some == 0) {   // no lane samples this chunk
                c0 = c1;
                continue;
            }
            {
                // every lane is past the previous chunk's reads (the wave runs
                // in order); copy the box, rows along the fastest axis
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                __builtin_amdgcn_wave_barrier();
                // a pass copies rpp whole rows (64 / dx; a longer row takes
                // its passes 64 cells at a time): lane = (row r of the pass,
                // cell lx of the row) and only the row advances, by sz
                // slices and sy rows with at most one carry, so a pass costs
                // half the index arithmetic of 64 consecutive cells
                const float rdx = __builtin_amdgcn_rcpf((float)dx), rdy = __builtin_amdgcn_rcpf((float)dy);
                const bool wide = dx > 64;
                const int rpp = wide ? 1 : scalar(small_quot(64, rdx));
                const int r0 = wide ? 0 : small_quot(lane, rdx);
                const int rows = dy * dz;
                const int sz = scalar(small_quot(rpp, rdy));
                const int sy = rpp - sz * dy;
                const unsigned uYS = (unsigned)YS, uZS = (unsigned)ZS;
                const unsigned a0 = (unsigned)sy * uYS + (unsigned)sz * uZS, a1 = a0 + uZS - (unsigned)dy * uYS;
                const int zr = small_quot(r0, rdy);
                // (raw: padded index 1 is the first voxel; a box inside the
                // volume is copied like any other)
                const unsigned shift = RAW ? (unsigned)CB + uYS + uZS : 0u;
                const bool whole = !RAW || (lo0 >= 1 && lo1 >= 1 && lo2 >= 1 && lo0 + dx <= A.px - 2 &&
                                            lo1 + dy <= A.py - 2 && lo2 + dz <= A.pz - 2);
                for (int x0 = 0; x0 < dx; x0 += 64) {
                    const int lx = lane - (int)__umul24(r0, dx) + x0;
                    // rows left for this lane (none: its cell is beyond the row
                    // or belongs to the next pass)
                    const int left = (r0 < rpp && lx < dx) ? rows - r0 : 0;
                    int ly = r0 - (int)__umul24(zr, dy);
                    unsigned goff = (unsigned)((lo0 + lx) * CB) + __umul24(__umul24(lo2 + zr, PY) + lo1 + ly, YS) - shift;
                    int z = lo2 + zr;
                    auto next = [&] {
                        ly += sy;
                        const bool carry = ly >= dy;
                        ly -= carry ? dy : 0;
                        goff += carry ? a1 : a0;
                        if (RAW) z += sz + (carry ? 1 : 0);
                    };
                    const bool in_x = !RAW || (unsigned)(lo0 + lx - 1) < (unsigned)(A.px - 3);
                    // straight to LDS, without registers and without a wait
                    // before the last pass is issued; the lanes' cells are
                    // consecutive: r0 dx + lx = lane + x0 cells into the pass
                    int cell = x0;
                    for (int p = 0; p < rows; p += rpp) {
                        bool here = left > p;
                        if (RAW && !whole) {
                            const bool vox = in_x && (unsigned)(lo1 + ly - 1) < (unsigned)(A.py - 3) &&
                                             (unsigned)(z - 1) < (unsigned)(A.pz - 3);
                            if (here && !vox) st[cell + lane] = 0.f;
                            here = here && vox;
                        }
                        if (here) {
                            const char* src = vb + goff;
#pragma unroll
                            for (int h = 0; h < G::n16; ++h)
                                load_to_lds<16>(src + 16 * h, st + 4 * (cell + h * BUF));
#pragma unroll
                            for (int j = 0; j < G::n4; ++j)
                                load_to_lds<4>(src + 16 * G::n16 + 4 * j, st + G::single / 4 + cell + j * BUF);
                        }
                        next();
                        cell += rpp * dx;
                    }
                }
                __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0): the loads to LDS are done
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
            }
            // the cells live only within the chunk (no copies of them carried
            // around the chunk loop) and need no initial value: every cell
            // offset in the box is >= 0, so a lane's first sample loads
            // (the box cell of padded cell (ix, iy, iz) at byte offset
            // iz cz + iy cy + ix CB - (lo2 cz + lo1 cy + lo0 CB), in unsigned
            // arithmetic: the wrap of the products cancels in the difference)
            CellPair<C> P[4];
            unsigned last = ~0u;
            const unsigned cy = (unsigned)(dx * G::unit), cz = (unsigned)(dxy * G::unit);
            // (offsets from the start of the block's LDS: the wave's buffer
            // starts kStageBytes x wave into it)
            const unsigned own = (unsigned)__builtin_amdgcn_readfirstlane(wave * kStageBytes);
            unsigned base = own + (G::unit == 16 ? 0u : (unsigned)G::single) -
                            ((unsigned)lo2 * cz + (unsigned)lo1 * cy + (unsigned)(lo0 * G::unit));
            asm("" : "+s"(base));   // one sum, not regrouped by axis in the loop
            const char* stb = smem;
            auto from_lds = [&](int ix, int iy, int iz) {
                const unsigned loc = mad_u24(iz, cz, mad_u24(iy, cy, (unsigned)(ix * G::unit) + base));
                if (loc != last) {
                    last = loc;
                    lds_pair<C, KC>(stb, own, loc, P[0]);
                    lds_pair<C, KC>(stb, own, loc + cy, P[1]);
                    lds_pair<C, KC>(stb, own, loc + cz, P[2]);
                    lds_pair<C, KC>(stb, own, loc + cz + cy, P[3]);
                }
            };
            // the samples, counted once per chunk; the loop runs on the
            // index as a float (0 <= n - na < 2^24: exact)
            const int cnt = s_hi - s_lo + 1;
            if (cnt > 0) nsamp += cnt;
            const float fe = (float)(s_hi - na);
            for (float fm = (float)(s_lo - na); fm <= fe; fm += 1.0f) step(!inside, fm, P, from_lds);
            if (cells * 3 < BUF && S < 64) S <<= 1;
            c0 = c1;
        }
        if (gather) {
            CellPair<C> P[4];   // offsets are >= 0: the first sample loads
            int last = -1;
            const int g0 = max(c0, rr.n0), g1 = min(nb - 1, rr.n1);
            if (g1 >= g0) nsamp += g1 - g0 + 1;
            const float fe = (float)(g1 - na);
            for (float fm = (float)(g0 - na); fm <= fe; fm += 1.0f)
                step(true, fm, P, [&](int ix, int iy, int iz) {
                    if constexpr (RAW) {
                        // taps outside the volume are zero; all eight loads
                        // first, at clamped indices
                        const int nx = A.px - 3, ny = A.py - 3, nz = A.pz - 3;
                        float t[8];
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const int x = min(max(ix - 1 + (e & 1), 0), nx - 1), y = min(max(iy - 1 + ((e >> 1) & 1), 0), ny - 1),
                                      z = min(max(iz - 1 + (e >> 2), 0), nz - 1);
                            t[e] = *(const float*)(vb + (unsigned)(x * CB) + __umul24(__umul24(z, ny) + y, YS));
                        }
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const bool vox = (unsigned)(ix - 1 + (e & 1)) < (unsigned)nx &&
                                             (unsigned)(iy - 1 + ((e >> 1) & 1)) < (unsigned)ny &&
                                             (unsigned)(iz - 1 + (e >> 2)) < (unsigned)nz;
                            (e & 1 ? P[e >> 1].b[0] : P[e >> 1].a[0]) = vox ? t[e] : 0.f;
                        }
                        return;
                    }
                    const int voff = ix * CB + (int)__umul24(__umul24(iz, PY) + iy, YS);
                    if (voff != last) {
                        last = voff;
                        P[0] = load_pair_g<C>(vb, voff);
                        P[1] = load_pair_g<C>(vb, voff + YS);
                        P[2] = load_pair_g<C>(vb, voff + ZS);
                        P[3] = load_pair_g<C>(vb, voff + YZ);
                    }
                });
        }
    }
    if (A.ms.seg > 1) {
        __syncthreads();   // every wave is done with its staging buffer
        gather_segments<C, T>(smem, A.ms.seg, rpb, sid, acc, nsamp);
    }
    const bool owner = valid && sid == 0;
    const float dt = (float)g.dt;
    if (owner && A.p_out) A.p_out[iu + (size_t)g.nu * iv] = dt * acc[0];
    if (A.partials) {
        constexpr int NM = 5 + 3 * (C - 1);
        double mo[NM + 1];
#pragma unroll
        for (int i = 0; i < NM; ++i) mo[i] = 0.0;
        mo[NM] = sid == 0 ? (double)nsamp : 0.0;   // segments were gathered
        if (owner) {
            double yd = (double)A.y[iu + (size_t)g.nu * iv];
            double pd = (double)(dt * acc[0]);
            mo[0] = yd;
            mo[1] = yd * yd;
            mo[2] = pd;
            mo[3] = yd * pd;
            mo[4] = pd * pd;
#pragma unroll
            for (int k = 0; k < C - 1; ++k) {
                if (k + 1 < A.kc) {
                    double tk = (double)(dt * acc[k + 1]);
                    mo[5 + 3 * k] = pd * tk;
                    mo[6 + 3 * k] = yd * tk;
                    mo[7 + 3 * k] = tk;
                }
            }
        }
        block_sum_store<NM + 1>(mo, NM + 1, A.partials + blockIdx.x, (int)gridDim.x, rpb / 64, SUM);
        if constexpr (SUM)
            last_block_sums<NM>(A.partials, 5 + 3 * (A.kc - 1), NM, A.moments, A.arrived, A.done, A.seq);
    }
}

// ------------------------------------------------------------ support --
// Bounds of the nonzero voxels of each slice of an image (see
// launch_support), combined with atomics.  NaN counts as nonzero.
template <typename F>
__global__ void __launch_bounds__(256) k_support(const F* __restrict__ f0, int nx, int ny, int nz,
                                                 int* __restrict__ sl)
{
    __shared__ int sb[8];
    const int nxy = nx * ny;
    for (int z = blockIdx.y; z < nz; z += gridDim.y) {
        if (threadIdx.x < 8) sb[threadIdx.x] = (threadIdx.x & 1) ? INT_MIN : INT_MAX;
        __syncthreads();
        int b[8] = {INT_MAX, INT_MIN, INT_MAX, INT_MIN, INT_MAX, INT_MIN, INT_MAX, INT_MIN};
        for (int e = blockIdx.x * 256 + threadIdx.x; e < nxy; e += gridDim.x * 256) {
            const float v = widen<float>(f0[(size_t)z * nxy + e]);
            if (!(v == 0.0f)) {
                const int x = e % nx, y = e / nx;
                const int q[4] = {x, y, x + y, x - y};
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    b[2 * c] = min(b[2 * c], q[c]);
                    b[2 * c + 1] = max(b[2 * c + 1], q[c]);
                }
            }
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                b[2 * c] = min(b[2 * c], __shfl_xor(b[2 * c], o));
                b[2 * c + 1] = max(b[2 * c + 1], __shfl_xor(b[2 * c + 1], o));
            }
        }
        if ((threadIdx.x & 63) == 0) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                atomicMin(&sb[2 * c], b[2 * c]);
                atomicMax(&sb[2 * c + 1], b[2 * c + 1]);
            }
        }
        __syncthreads();
        if (threadIdx.x < 8) {
            int* t = sl + (size_t)8 * z + threadIdx.x;
            if (threadIdx.x & 1) atomicMax(t, sb[threadIdx.x]);
            else atomicMin(t, sb[threadIdx.x]);
        }
        __syncthreads();
    }
}

// out[row] = max |a[row][i]| over i < n, combined with atomics on the bit
// patterns of the (non-negative) floats; the caller zeroes `out` first.
template <typename S>
__global__ void __launch_bounds__(256) k_absmax_rows(const S* __restrict__ a, size_t n,
                                                     float* __restrict__ out)
{
    __shared__ float wm[4];
    const S* row = a + (size_t)blockIdx.y * n;
    float m = 0.0f;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256)
        m = fmaxf(m, fabsf(widen<float>(row[i])));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    if ((threadIdx.x & 63) == 0) wm[threadIdx.x >> 6] = m;
    __syncthreads();
    // one atomic per block (few blocks per row: little contention)
    if (threadIdx.x == 0)
        atomicMax((int*)&out[blockIdx.y], __float_as_int(fmaxf(fmaxf(wm[0], wm[1]), fmaxf(wm[2], wm[3]))));
}

// ------------------------------------------------- gather backprojection --
// P^T r as a gather: every output voxel sums, over the rays whose samples can
// touch it, r * dt * (its trilinear weight) at each sample -- the weight the
// forward march gives that voxel as a corner of the sample's cell, i.e.
// prod_a max(0, 1 - |q_a - v_a|).  No global atomics, and every voxel's sum
// is formed in a fixed order, so the result is deterministic.
//
// A workgroup owns a brick of 4 x 4 (or, see launch_backproject, 2 x 2)
// columns of 16 voxels along the rays' dominant in-plane axis A.  It walks the
// brick's detector footprint in tiles of 8 (u) x 32 (v) pixels; per tile every
// thread stages one ray in LDS (the sample nearest the brick centre relative
// to the brick origin, the step per sample, slab bounds, r dt, narrowed to the
// valid sample range [0, floor(L / dt)]).  Then the 16 (64) threads of a column
// split the rays of the column's own footprint between them; for each ray a
// slab test gives the samples that pass within one voxel of the column's line,
// and each such sample adds its weight to the two voxels of the column that
// straddle it along A (two neighbouring samples at a time to three voxels,
// where they lie less than a voxel apart), in a per-thread run of accumulators
// in LDS.  Per ray the set-up is paid once per column instead of once per
// voxel, and each sample is visited once.  A fixed-order sum over the threads
// of each column gives the voxel values.
struct BPFoot {
    // for an index-space point X: a = a0 + an.X (depth along the central
    // ray, mm), b = b0 + bn.X and c = c0 + cn.X (offsets along e_u, e_v);
    // it projects to u = sdd b / a + su, v = sdd c / a + sv (mm)
    float a0, an[3], b0, bn[3], c0, cn[3];
    float sdd, su, sv, u0, inv_du, v0, inv_dv;
    int nu, nv;
};

// Pixel box (inclusive, clipped to the detector) that holds every ray
// meeting the index-space box [lo, hi]: the pixels whose centres lie in the
// bounding box of the projected corners (the box projects inside their
// convex hull), widened by `eps` pixels for the FP32 rounding of the
// projection; empty (i0 > i1) if none can.
__device__ __forceinline__ void footprint(const BPFoot& F, const float lo[3], const float hi[3],
                                          float eps, int& iu0, int& iu1, int& iv0, int& iv1)
{
    float umin = 3.0e38f, umax = -3.0e38f, vmin = 3.0e38f, vmax = -3.0e38f;
    bool front = true;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const float X = (c & 1) ? hi[0] : lo[0], Y = (c & 2) ? hi[1] : lo[1], Z = (c & 4) ? hi[2] : lo[2];
        const float a = F.a0 + F.an[0] * X + F.an[1] * Y + F.an[2] * Z;
        const float b = F.b0 + F.bn[0] * X + F.bn[1] * Y + F.bn[2] * Z;
        const float cc = F.c0 + F.cn[0] * X + F.cn[1] * Y + F.cn[2] * Z;
        front = front && a > 1e-3f;
        // the boxes are widened by at least 0.02 pixels, far beyond the
        // error of the hardware reciprocal
        const float t = F.sdd * __builtin_amdgcn_rcpf(a);
        const float u = fmaf(t, b, F.su), v = fmaf(t, cc, F.sv);
        umin = fminf(umin, u);
        umax = fmaxf(umax, u);
        vmin = fminf(vmin, v);
        vmax = fmaxf(vmax, v);
    }
    if (!front) {  // the box reaches behind the source: every pixel
        iu0 = 0; iu1 = F.nu - 1; iv0 = 0; iv1 = F.nv - 1;
        return;
    }
    iu0 = max(0, (int)ceilf(fmaxf((umin - F.u0) * F.inv_du - eps, -2.0f)));
    iu1 = min(F.nu - 1, (int)floorf(fminf((umax - F.u0) * F.inv_du + eps, (float)F.nu + 2.0f)));
    iv0 = max(0, (int)ceilf(fmaxf((vmin - F.v0) * F.inv_dv - eps, -2.0f)));
    iv1 = min(F.nv - 1, (int)floorf(fminf((vmax - F.v0) * F.inv_dv + eps, (float)F.nv + 2.0f)));
}

struct BPArgs {
    RayGeom g;            // unswapped (x-fastest) geometry
    BPFoot F;
    int ax;               // column axis A: 0 (x) or 1 (y)
    int bx, by, bz;       // brick: 16 along A, 4 along the other two axes
    int nbx, nby;         // bricks per axis
    int nx, ny, nz;
    double a, b, scale;   // r = scale (p - a y - b) when no residual is given
};

template <typename R>
struct alignas(4 * sizeof(R)) BPVec4 {
    R x, y, z, w;
};

template <typename R>
__device__ __forceinline__ R fract_of(R x);
template <> __device__ __forceinline__ float fract_of<float>(float x) { return __builtin_amdgcn_fractf(x); }
template <> __device__ __forceinline__ double fract_of<double>(double x) { return __builtin_amdgcn_fract(x); }
// x clamped to [0, 1] (x <= 1 where it is used)
__device__ __forceinline__ float saturate(float x) { return __builtin_amdgcn_fmed3f(x, 0.f, 1.f); }
__device__ __forceinline__ double saturate(double x) { return fmax(x, 0.0); }
// the whole voxel of a position along a column, kept inside the run of slots
__device__ __forceinline__ float run_voxel(float x, float hi) { return __builtin_amdgcn_fmed3f(floorf(x), -10.f, hi); }
__device__ __forceinline__ double run_voxel(double x, double hi) { return fmin(fmax(floor(x), -10.0), hi); }

// What bounds the column gather is the latency of a sample's round trip to
// its LDS run (position, read, add, write: the next sample may touch the same
// voxels), then VALU issue, so blocks in flight count: 11 words a staged ray
// and 20 slots a run make 31 KB a block, five to a CU (four with the 16 words
// and 21 slots of before), and the loop is 16 VALU instructions a sample and
// column (22 before; alone worth 2 %).  256x256x100 voxels, 512x384 pixels,
// at 0 / 30 / 90 deg: 907 / 694 / 887 -> 759 / 580 / 725 us.  Tiles of 4 x 32
// rays (six blocks) 752 / 630 / 710 us; 8 x 4 or 4 x 8 columns with 8 lanes
// each 750-1570 us; LDS float atomics instead of the round trip 5000-5900 us
// (they take the lanes one by one).  Two samples a turn (kPairs) halve the round
// trips: 722 / 569 / 662 us; with the ray's weight applied in the last
// additions, whole sample bounds as floats and positions from the column's
// middle (error against FP64 7.4e-8 - 1.1e-7 relative, 7.9e-8 - 1.5e-7 from
// the brick's corner) 718 / 552 / 653 us, 33 VALU instructions a turn.
// (Loading the next ray's record ahead: 3-4 % slower.)
constexpr int kBpTileU = 8, kBpTileV = 32;   // staged rays: one per thread
// CB x CB columns a brick (along the other in-plane axis and z), the block's
// 256 threads split evenly over them.  MODE: how a lane goes through a ray's
// samples.
//   kPairs: no ray moves more than a voxel a sample along A, so two
//   neighbouring samples touch three voxels of the run
//   kSingles: one sample a turn
//   kMany: one sample a turn with an integer index, where a brick may hold
//   samples further than kBpReach from the one nearest its centre, the end of
//   the other modes' bounds
enum { kPairs, kSingles, kMany };
constexpr float kBpReach = 1.0e6f;
template <typename R, int CB, int MODE>
__global__ void __launch_bounds__(256) k_backproject_columns(BPArgs A, const R* __restrict__ resid,
                                                             const R* __restrict__ p,
                                                             const R* __restrict__ y,
                                                             R* __restrict__ out)
{
    // One staged ray in records of consecutive rays, so the lanes of a
    // column, which take consecutive rays, read without bank conflicts.  Axes
    // in column order (A, B, z):
    //   s_r0: the sample nearest the brick centre minus the brick origin (along
    //   A minus the column's middle, so that positions along it round finest),
    //   r dt
    //   s_r1: the index-space step per sample, slab lower bound along A
    //   s_r2: 1/step in B and z; s_r3: slab upper bound along A
    // Slab bounds are in samples: |q_a + m d_a - l| < 1 for m within |1/d_a|
    // of (l - q_a) / d_a; along A the whole column (-1, 16), narrowed to the
    // ray's valid samples.
    constexpr int TU = kBpTileU, TV = kBpTileV, NR = 256;
    static_assert(TU * TV == NR, "one staged ray per thread");
    __shared__ BPVec4<R> s_r0[NR], s_r1[NR];
    __shared__ float2 s_r2[NR];
    __shared__ float s_r3[NR];
    // thread t's run of 20 accumulators: 16 voxels along A at slots [2, 18)
    // (two pad slots each side take the clipped weights of samples just
    // outside the column, so the accumulation needs no branch); slot-major,
    // slot s of thread t at s * 256 + t, so each slot of the 64 lanes of a
    // wave spans all banks and a lane's bank does not depend on the slot:
    // the read-modify-writes never conflict
    __shared__ R s_acc[20 * 256];
    __shared__ int s_box[4];
    __shared__ int s_odd;   // whether a ray staged so far is infinite or NaN
    // kMany: the rays' valid samples
    __shared__ int2 s_valid[MODE == kMany ? NR : 1];
    const RayGeom& g = A.g;
    const int t = threadIdx.x;
    const int bid = blockIdx.x;
    const int b0[3] = {(bid % A.nbx) * A.bx, ((bid / A.nbx) % A.nby) * A.by, (bid / (A.nbx * A.nby)) * A.bz};
    const int AX = A.ax, BX = 1 - A.ax;           // column axis and the other in-plane axis
    // a wave holds 4 columns x 16 lanes (one of 64): consecutive lanes take
    // consecutive rays of one column, so their record loads hit distinct banks
    constexpr int LPC = 256 / (CB * CB);
    const int col = t / LPC, lane = t % LPC;        // column (lb, lz) and ray lane
    const int lb = col % CB, lz = col / CB;
    for (int e = t; e < 256 * 20; e += 256) s_acc[e] = (R)0;
    R* acc = s_acc + 10 * 256 + t;   // the slot of the voxel at the column's middle
    if (t == 0) {
        s_odd = 0;
        const float lo[3] = {(float)(b0[0] - 1), (float)(b0[1] - 1), (float)(b0[2] - 1)};
        const float hi[3] = {(float)(b0[0] + A.bx), (float)(b0[1] + A.by), (float)(b0[2] + A.bz)};
        footprint(A.F, lo, hi, 1.0f, s_box[0], s_box[1], s_box[2], s_box[3]);
    }
    // the column's footprint: its line (-1, 16) along A, one voxel around it
    int ru0, ru1, rv0, rv1;
    {
        float lo[3], hi[3];
        lo[AX] = (float)(b0[AX] - 1);
        hi[AX] = (float)(b0[AX] + 16);
        lo[BX] = (float)(b0[BX] + lb - 1);
        hi[BX] = (float)(b0[BX] + lb + 1);
        lo[2] = (float)(b0[2] + lz - 1);
        hi[2] = (float)(b0[2] + lz + 1);
        footprint(A.F, lo, hi, 0.02f, ru0, ru1, rv0, rv1);
    }
    __syncthreads();
    const int bu0 = s_box[0], bu1 = s_box[1], bv0 = s_box[2], bv1 = s_box[3];
    const double cb[3] = {b0[0] + 0.5 * (A.bx - 1), b0[1] + 0.5 * (A.by - 1), b0[2] + 0.5 * (A.bz - 1)};
    const R rlb = (R)lb, rlz = (R)lz;
    // Tiles of 8 (u) x 32 (v) rays: a column's footprint is wide along u (the
    // column runs along A) and short along v, so a tall, narrow tile holds
    // the footprints of all columns at once and gives the lanes of a column
    // rays that cross it alike (the lanes of a wave then run their
    // sample loops for similar lengths: with 4 x 4 columns ~0.55 of the lanes
    // busy in the loop against ~0.3 with 16 x 16 tiles, and ~40 % fewer rounds
    // of rays)
    for (int tv0 = bv0; tv0 <= bv1; tv0 += TV) {
        for (int tu0 = bu0; tu0 <= bu1; tu0 += TU) {
            {   // stage one ray per thread (FP64 set-up, once per ray and brick)
                const int iu = tu0 + t % TU, iv = tv0 + t / TU;
                int m0 = 1, m1 = 0;
                R rw = (R)0;
                double qr[3] = {0.0, 0.0, 0.0}, dq[3] = {0.0, 0.0, 0.0};
                if (iu <= bu1 && iv <= bv1) {
                    const size_t pix = iu + (size_t)g.nu * iv;
                    const double r = resid ? (double)resid[pix]
                                           : A.scale * ((double)p[pix] - A.a * (double)y[pix] - A.b);
                    const double uu = g.u0 + iu * g.du, vv = g.v0 + iv * g.dv;
                    double D[3], L2 = 0.0;
#pragma unroll
                    for (int ax = 0; ax < 3; ++ax) {
                        D[ax] = g.qc[ax] + uu * g.eu[ax] + vv * g.ev[ax] - g.qs[ax];
                        const double w = D[ax] * g.sp[ax];
                        L2 += w * w;
                    }
                    if (L2 > 0.0 && r != 0.0) {
                        const double invL = rsq64(L2), L = L2 * invL;
                        double tc = 0.0;
#pragma unroll
                        for (int ax = 0; ax < 3; ++ax) {
                            D[ax] *= invL;   // index units per mm
                            tc += (cb[ax] - g.qs[ax]) * g.sp[ax] * g.sp[ax] * D[ax];
                        }
                        // the last sample lies at the detector, far outside the
                        // volume, and the centre sample only anchors m: neither
                        // needs a correctly rounded quotient
                        const double nlast = floor(L * g.inv_dt);
                        const double nc = fmin(fmax(rint(tc * g.inv_dt), 0.0), nlast);
                        const double tn = nc * g.dt;
#pragma unroll
                        for (int ax = 0; ax < 3; ++ax) {
                            qr[ax] = g.qs[ax] + tn * D[ax] - (double)b0[ax];
                            dq[ax] = g.dt * D[ax];
                        }
                        m0 = -(int)nc;
                        m1 = (int)(nlast - nc);
                        rw = (R)(r * g.dt);
                        if (MODE == kPairs && dq[AX] < 0.0) {   // samples in rising order along A
                            const int n0 = m0;
                            m0 = -m1;
                            m1 = -n0;
#pragma unroll
                            for (int ax = 0; ax < 3; ++ax) dq[ax] = -dq[ax];
                        }
                    }
                }
                // (asked once a wave, and the flag read ahead of its use: 0.4-0.9
                // % of the kernel's time, 689 -> 693 us at 0 deg; a test by each
                // ray of each column took 2-3 %)
                if (__any(!__builtin_isfinite(rw))) s_odd = 1;
                float lo[3], hi[3], inv[3];
#pragma unroll
                for (int ax = 0; ax < 3; ++ax) {
                    const float df = (float)dq[ax];
                    // the slab bounds carry a 1e-3 sample slack, so the
                    // hardware reciprocal (1 ulp) is exact enough
                    inv[ax] = fabsf(df) > 1e-30f ? __builtin_amdgcn_rcpf(df) : 1.0e30f;
                    const float e1 = (-1.0f - (float)qr[ax]) * inv[ax];
                    const float e2 = ((ax == AX ? 16.0f : 1.0f) - (float)qr[ax]) * inv[ax];
                    lo[ax] = fminf(e1, e2);
                    hi[ax] = fmaxf(e1, e2);
                }
                float la, ha;
                if constexpr (MODE == kMany) {
                    // (widened by the rounding of a position in the column)
                    la = lo[AX] - fabsf(1.0e-5f * inv[AX]);
                    ha = hi[AX] + fabsf(1.0e-5f * inv[AX]);
                    s_valid[t] = make_int2(m0, m1);
                } else {
                    // the valid samples [m0, m1] narrow the bounds along A:
                    // with the half-sample margin the rounding below yields
                    // exactly max(m0, .) and min(m1, .); no sample of the brick
                    // is beyond kBpReach, where both are whole numbers and
                    // halves of a float's
                    la = __builtin_amdgcn_fmed3f(fmaxf(lo[AX], (float)m0 - 0.5f), -kBpReach, kBpReach);
                    ha = __builtin_amdgcn_fmed3f(fminf(hi[AX], (float)m1 + 0.5f), -kBpReach, kBpReach);
                }
                s_r0[t] = {(R)(qr[AX] - 8.0), (R)qr[BX], (R)qr[2], rw};
                s_r1[t] = {(R)dq[AX], (R)dq[BX], (R)dq[2], (R)la};
                s_r2[t] = make_float2(inv[BX], inv[2]);
                s_r3[t] = ha;
            }
            __syncthreads();
            const int any_odd = s_odd;
            // rays of this tile inside the column's footprint, split over the
            // column's lanes
            const int ua = max(ru0, tu0), ub = min(ru1, tu0 + TU - 1);
            const int va = max(rv0, tv0), vb = min(rv1, tv0 + TV - 1);
            const int wu = ub - ua + 1, nr = (ub >= ua && vb >= va) ? wu * (vb - va + 1) : 0;
            // ray i of the clipped box (row-major) is (i % wu, i / wu); the
            // lane steps i by LPC, i.e. (LPC % wu, LPC / wu) with one carry
            const int kb = (va - tv0) * TU + (ua - tu0);
            int ou = 0, ov = 0, su = 0, sv = 0;
            if (nr > 0) {
                ou = lane % wu;
                ov = lane / wu;
                su = LPC % wu;
                sv = LPC / wu;
            }
            const bool odd = __builtin_amdgcn_readfirstlane(any_odd);
            for (int i = lane; i < nr; i += LPC) {
                const int k = kb + ov * TU + ou;
                ou += su;
                ov += sv;
                if (ou >= wu) {
                    ou -= wu;
                    ++ov;
                }
                // samples within one voxel of the column line (slab test; the
                // 1e-3 sample slack covers the FP32 rounding of the bounds and
                // the weights clip any sample it admits)
                const BPVec4<R> r0 = s_r0[k], r1 = s_r1[k];
                const float2 r2 = s_r2[k];
                const float ha = s_r3[k];
                // |q + m d - l| < 1 for m within |1/d| of (l - q) / d
                const R qa = r0.x, qb = r0.y - rlb, qz = r0.z - rlz;
                const float cb_ = -(float)qb * r2.x, cz_ = -(float)qz * r2.y;
                float lo = fmaxf(fmaxf((float)r1.w, cb_ - fabsf(r2.x)), cz_ - fabsf(r2.y));
                float hi = fminf(fminf(ha, cb_ + fabsf(r2.x)), cz_ + fabsf(r2.y));
                const R da = r1.x, db = r1.y, dz = r1.z;
                const R rw = r0.w;
                // one sample, to the voxels of nonzero weight alone
                auto single = [&](R fm) {
                    const R xa = fma(fm, da, qa), fl = run_voxel(xa, (R)8);
                    R* a2 = acc + (int)fl * 256;
                    const R w = saturate((R)1 - fabs(fma(fm, db, qb))) * saturate((R)1 - fabs(fma(fm, dz, qz)));
                    const R w1 = w * (xa - fl), w0 = w - w1;
                    if (w0 > (R)0) a2[0] = fma(rw, w0, a2[0]);
                    if (w1 > (R)0) a2[256] = fma(rw, w1, a2[256]);
                };
                if constexpr (MODE == kMany) {
                    // (widened by the rounding of the bounds: the weights
                    // clip any sample admitted)
                    const float eb = 1.0e-5f * (fabsf(cb_) + fabsf(r2.x)), ez = 1.0e-5f * (fabsf(cz_) + fabsf(r2.y));
                    lo = fmaxf(fmaxf((float)r1.w, cb_ - fabsf(r2.x) - eb), cz_ - fabsf(r2.y) - ez) - 1.0f;
                    hi = fminf(fminf(ha, cb_ + fabsf(r2.x) + eb), cz_ + fabsf(r2.y) + ez) + 1.0f;
                    const int2 valid = s_valid[k];
                    const int m0 = max(valid.x, (int)__builtin_amdgcn_fmed3f(lo, -2.1e9f, 2.1e9f));
                    const int m1 = min(valid.y, (int)__builtin_amdgcn_fmed3f(hi, -2.1e9f, 2.1e9f));
                    for (int m = m0; m <= m1; ++m) single((R)m);
                    continue;
                }
                // whole samples, as floats (exact: |m| <= kBpReach between the
                // bounds along A)
                lo = ceilf(lo - 1.0e-3f);
                hi = floorf(hi + 1.0e-3f);
                if (!(lo <= hi)) continue;
                const R fm1 = (R)hi;
                // From the first tile with an infinite or NaN ray on, a brick's
                // rays go sample by sample (below, 0 x inf would reach the
                // run's other voxels and inf - inf stand for a weight).
                if (odd) {
                    for (R fm = (R)lo; fm <= fm1; fm += (R)1) single(fm);
                    continue;
                }
                // the ray's values are in registers before the loop starts,
                // so no wait inside it holds back for the previous sample's
                // LDS write
                __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
                if constexpr (MODE == kPairs) {
                    // two samples a turn, less than a voxel apart along A:
                    // they touch three voxels of the run
                    for (R fm = (R)lo; fm <= fm1; fm += (R)2) {
                        const R xa = fma(fm, da, qa), fl = run_voxel(xa, (R)7);
                        R* a3 = acc + (int)fl * 256;
                        const R s0 = a3[0], s1 = a3[256], s2 = a3[512];
                        // (the reads go out before the weights are formed)
                        __builtin_amdgcn_sched_barrier(0);
                        const R x1 = xa - fl, x2 = x1 + da;
                        const R pb = fma(fm, db, qb), pz = fma(fm, dz, qz);
                        const R w1 = saturate((R)1 - fabs(pb)) * saturate((R)1 - fabs(pz));
                        R w2 = saturate((R)1 - fabs(pb + db)) * saturate((R)1 - fabs(pz + dz));
                        w2 = fm < fm1 ? w2 : (R)0;
                        const R u0 = w1 * saturate((R)1 - x1), v0 = w2 * saturate((R)1 - x2), v2 = w2 * saturate(x2 - (R)1);
                        a3[0] = fma(rw, u0 + v0, s0);
                        a3[256] = fma(rw, (w1 - u0) + (w2 - v0 - v2), s1);
                        a3[512] = fma(rw, v2, s2);
                    }
                } else {
                    for (R fm = (R)lo; fm <= fm1; fm += (R)1) {
                        // (saturated differences: one instruction each in FP32)
                        const R wbz = saturate((R)1 - fabs(fma(fm, db, qb))) *
                                      (saturate((R)1 - fabs(fma(fm, dz, qz))) * rw);
                        // the slab range keeps xa within (-9.01, 8.01): the clamp
                        // only guards the LDS run
                        const R xa = fma(fm, da, qa);
                        const int j = (int)run_voxel(xa, (R)8);
                        const R t1 = fract_of(xa) * wbz, t0 = wbz - t1;
                        // the thread's own LDS run: a plain read-modify-write
                        acc[j * 256] += t0;
                        acc[(j + 1) * 256] += t1;
                    }
                }
            }
            __syncthreads();
        }
    }
    // voxel (column c, position j along A): the sum over the column's lanes,
    // in an order rotated by j so that the lanes of a wave read different
    // banks; with few columns several threads share a voxel's sum
    {
        constexpr int NP = 256 / (CB * CB * 16), per = LPC / NP;
        const int o = t / NP, part = t % NP, c = o >> 4, j = o & 15;
        R v = (R)0;
        for (int l = 0; l < per; ++l) v += s_acc[(2 + j) * 256 + c * LPC + part * per + ((l + j) & (per - 1))];
#pragma unroll
        for (int x = 1; x < NP; x <<= 1) v += __shfl_xor(v, x);
        int vx[3];
        vx[AX] = b0[AX] + j;
        vx[BX] = b0[BX] + c % CB;
        vx[2] = b0[2] + c / CB;
        if (part == 0 && vx[0] < A.nx && vx[1] < A.ny && vx[2] < A.nz)
            out[(size_t)vx[0] + (size_t)A.nx * ((size_t)vx[1] + (size_t)A.ny * vx[2])] = v;
    }
}

// ---------------------------------------------------------- contraction --
// partials[k * blocks + block] = sum_v g[v] * sum_a (1/s_a) dT[f0]/dq_a(q_v) u_k[a][v]
template <typename R, typename S, typename F, int KM>
__global__ void __launch_bounds__(256) k_contract(const F* __restrict__ f0,
                                                  const S* __restrict__ mean,
                                                  const S* __restrict__ U, int K,
                                                  Chan<double, 8> w, VoxGrid g,
                                                  const R* __restrict__ gpad,
                                                  double* __restrict__ partials)
{
    const int i = blockIdx.x * 64 + threadIdx.x, j = blockIdx.y * 4 + threadIdx.y;
    double m[KM];
#pragma unroll
    for (int kk = 0; kk < KM; ++kk) m[kk] = 0.0;
    for (int k = blockIdx.z; k < g.nz; k += gridDim.z) {
        if (i < g.nx && j < g.ny) {
            size_t N = (size_t)g.nx * g.ny * g.nz;
            size_t v = (size_t)i + (size_t)g.nx * ((size_t)j + (size_t)g.ny * k);
            R gv = gpad[v];
            if (gv != (R)0) {
                R x[3], u[KM][3];
                load_fields<R, S, KM, size_t>(mean, U, K, N, v * sizeof(S), w, x, u);
                R qx = (R)i + by_spacing(x[0], g, 0);
                R qy = (R)j + by_spacing(x[1], g, 1);
                R qz = (R)k + by_spacing(x[2], g, 2);
                R dT[3];
                sample_f0<R, F, true>(f0, g.nx, g.ny, g.nz, qx, qy, qz, dT);
                double G0 = (double)dT[0] / g.sp[0], G1 = (double)dT[1] / g.sp[1],
                       G2 = (double)dT[2] / g.sp[2];
                double gd = (double)gv;
    #pragma unroll
                for (int kk = 0; kk < KM; ++kk)
                    if (kk < K)
                        m[kk] += gd * (G0 * (double)u[kk][0] + G1 * (double)u[kk][1] + G2 * (double)u[kk][2]);
            }
        }
    }
    // threadIdx is 2-D (64 x 4): flatten for the block reduction
    __shared__ double red[4][KM];
    const int lane = threadIdx.x, wv = threadIdx.y;
#pragma unroll
    for (int kk = 0; kk < KM; ++kk) {
        double s = wave_sum(m[kk]);
        if (lane == 0) red[wv][kk] = s;
    }
    __syncthreads();
    int t = threadIdx.x + 64 * threadIdx.y;
    if (t < K) {
        size_t blk = blockIdx.x + (size_t)gridDim.x * (blockIdx.y + (size_t)gridDim.y * blockIdx.z);
        size_t nblk = (size_t)gridDim.x * gridDim.y * gridDim.z;
        partials[t * nblk + blk] = red[0][t] + red[1][t] + red[2][t] + red[3][t];
    }
}

// -------------------------------------------------------- warp adjoint ---
// Lane l's value from lane l - 1 (lane 0: its own) of the wave.
template <typename T>
__device__ __forceinline__ T from_left(T v)
{
    static_assert(sizeof(T) % 4 == 0, "whole words");
    int w[sizeof(T) / 4];
    __builtin_memcpy(w, &v, sizeof v);
#pragma unroll
    for (int i = 0; i < (int)(sizeof(T) / 4); ++i)
        w[i] = __builtin_amdgcn_update_dpp(w[i], w[i], 0x138, 0xf, 0xf, false);   // wave_shr:1
    __builtin_memcpy(&v, w, sizeof v);
    return v;
}

// W^T g by atomics, bound by their number: neighbouring voxels along x mostly
// fall in neighbouring cells, so a lane hands its four sums for the cell's
// right side to the next lane where that one's cell follows its own, and
// most lanes issue four atomics instead of eight.  256x256x100: 164 -> 120 us.
template <typename R>
__global__ void __launch_bounds__(256) k_warp_adjoint(const R* __restrict__ dvf,
                                                      const R* __restrict__ gv, VoxGrid g,
                                                      R* __restrict__ out)
{
    const int i = blockIdx.x * 64 + threadIdx.x, j = blockIdx.y * 4 + threadIdx.y, k = blockIdx.z;
    if (j >= g.ny) return;   // whole waves: a wave is one row of voxels
    const bool in = i < g.nx;
    const size_t N = (size_t)g.nx * g.ny * g.nz;
    const size_t v = (size_t)(in ? i : g.nx - 1) + (size_t)g.nx * ((size_t)j + (size_t)g.ny * k);
    const R val = in ? gv[v] : (R)0;
    if (__all(val == (R)0)) return;
    R qx = (R)i + by_spacing(dvf[v], g, 0);
    R qy = (R)j + by_spacing(dvf[N + v], g, 1);
    R qz = (R)k + by_spacing(dvf[2 * N + v], g, 2);
    qx = clampv(qx, (R)-2, (R)(g.nx + 1));
    qy = clampv(qy, (R)-2, (R)(g.ny + 1));
    qz = clampv(qz, (R)-2, (R)(g.nz + 1));
    const R fx = floor(qx), fy = floor(qy), fz = floor(qz);
    const int i0 = (int)fx, j0 = (int)fy, k0 = (int)fz;
    const R ax = qx - fx, ay = qy - fy, az = qz - fz;
    const R bx = (R)1 - ax, by = (R)1 - ay, bz = (R)1 - az;
    // (products in the order x, y, z; a zero value adds nothing anywhere)
    const bool on = val != (R)0;
    const R w[4] = {by * bz, ay * bz, by * az, ay * az};
    R lo[4], hi[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        lo[r] = on ? bx * w[r] * val : (R)0;
        hi[r] = on ? ax * w[r] * val : (R)0;
    }
    const int lane = threadIdx.x;
    // (all lanes take part in each exchange: none inside a condition)
    const int li = from_left(i0), lj = from_left(j0), lk = from_left(k0);
    const bool take = (lane > 0) & (li + 1 == i0) & (lj == j0) & (lk == k0);
    // whether the next lane takes this one's right side (the last has none)
    const bool given = ((__ballot(take) >> 1) >> lane) & 1u;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const R h = from_left(hi[r]);
        lo[r] += take ? h : (R)0;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int jj = j0 + (r & 1), kk = k0 + (r >> 1);
        if ((unsigned)jj < (unsigned)g.ny && (unsigned)kk < (unsigned)g.nz) {
            R* row = out + (size_t)g.nx * ((size_t)jj + (size_t)g.ny * kk);
            if ((unsigned)i0 < (unsigned)g.nx && lo[r] != (R)0) unsafeAtomicAdd(row + i0, lo[r]);
            if (!given && (unsigned)(i0 + 1) < (unsigned)g.nx && hi[r] != (R)0) unsafeAtomicAdd(row + i0 + 1, hi[r]);
        }
    }
}

// ------------------------------------------------------------ localise ---
// One wave: lane t < 8 owns trilinear corner t; FP64 throughout.  KM: most
// fields the instance takes (a step waits for one round of loads; always
// loading eight fields, K = 1 was up to 9 % slower over 30 steps than field by
// field.  18 steps, K = 1 / 3 / 5: 33 -> 25 / 27 / 29 us a call).
template <typename S, int KM>
__global__ void __launch_bounds__(64) k_localize(const S* __restrict__ mean,
                                                 const S* __restrict__ U, int K,
                                                 Chan<double, 8> w, VoxGrid g, double pr0,
                                                 double pr1, double pr2, double org0, double org1,
                                                 double org2, double tol, int max_iter,
                                                 double* out, unsigned long long* done,
                                                 unsigned long long seq)
{
    const int t = threadIdx.x;
    const size_t N = (size_t)g.nx * g.ny * g.nz;
    const int n[3] = {g.nx, g.ny, g.nz};
    const double org[3] = {org0, org1, org2};
    const double pref[3] = {pr0, pr1, pr2};
    double p[3] = {pr0, pr1, pr2};
    int it = 0, conv = 0;
    for (it = 1; it <= max_iter; ++it) {
        int i0[3];
        double ph[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            double q = (p[a] - org[a]) / g.sp[a];
            double hi = (double)(n[a] - 1);
            q = fmin(fmax(q, 0.0), hi);
            double fl = floor(q);
            if (n[a] >= 2 && fl > hi - 1.0) fl = hi - 1.0;
            i0[a] = (int)fl;
            ph[a] = q - fl;
        }
        double X[3] = {0.0, 0.0, 0.0};
        if (t < 8) {
            int dx = t & 1, dy = (t >> 1) & 1, dz = t >> 2;
            double wt = (dx ? ph[0] : 1.0 - ph[0]) * (dy ? ph[1] : 1.0 - ph[1]) *
                        (dz ? ph[2] : 1.0 - ph[2]);
            if (wt != 0.0) {
                size_t v = (size_t)(i0[0] + dx) + (size_t)g.nx * ((size_t)(i0[1] + dy) + (size_t)g.ny * (i0[2] + dz));
                double x[3], u[KM][3];
                load_fields<double, S, KM, size_t>(mean, U, K, N, v * sizeof(S), w, x, u);
#pragma unroll
                for (int a = 0; a < 3; ++a) X[a] = wt * x[a];
            }
        }
        // fixed-order sum over the 8 corners
#pragma unroll
        for (int a = 0; a < 3; ++a) {
#pragma unroll
            for (int off = 4; off > 0; off >>= 1) X[a] += __shfl_down(X[a], off, 8);
            X[a] = __shfl(X[a], 0, 64);
        }
        double d2 = 0.0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            double pn = pref[a] - X[a];
            d2 += (pn - p[a]) * (pn - p[a]);
            p[a] = pn;
        }
        if (sqrt(d2) < tol) {
            conv = 1;
            break;
        }
    }
    if (t == 0) {
        // straight to the host's mapped memory, then the sequence number
        const double r[5] = {p[0], p[1], p[2], (double)(it > max_iter ? max_iter : it), (double)conv};
#pragma unroll
        for (int i = 0; i < 5; ++i) __hip_atomic_store(&out[i], r[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __builtin_amdgcn_s_waitcnt(0);
        __hip_atomic_store(done, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// ============================================================ launchers ===
static VoxGrid vox(const pcr_grid& g)
{
    VoxGrid v;
    v.nx = g.n[0];
    v.ny = g.n[1];
    v.nz = g.n[2];
    for (int a = 0; a < 3; ++a) {
        v.sp[a] = g.spacing_mm[a];
        v.rd[a] = 1.0 / g.spacing_mm[a];
        v.rf[a] = 1.0f / (float)g.spacing_mm[a];
    }
    return v;
}
static dim3 vox_grid(const pcr_grid& g)
{
    return dim3((g.n[0] + 63) / 64, (g.n[1] + 3) / 4, g.n[2]);
}
static Chan<double, 8> wvec(const double* w, int K)
{
    Chan<double, 8> c;
    for (int k = 0; k < 8; ++k) c.v[k] = k < K ? w[k] : 0.0;
    return c;
}

PadLayout make_pad(const pcr_grid& g, int C, bool yfast)
{
    PadLayout L;
    L.nx = g.n[0];
    L.ny = g.n[1];
    L.nz = g.n[2];
    L.px = (yfast ? L.ny : L.nx) + 3;
    L.py = (yfast ? L.nx : L.ny) + 3;
    L.pz = L.nz + 3;
    L.C = C;
    L.yfast = yfast;
    return L;
}

bool prefer_yfast(const pcr_geom& G)
{
    // Measured on the paper-scale volume: the x-fastest layout with compact
    // ray tiles is fastest at every angle except within ~15 degrees of the y
    // axis (rays along x), where the y-fastest layout with one thread per ray
    // gains ~10 %.
    return std::fabs(std::sin(G.angle_rad)) > 0.97;
}

RayGeom make_ray_geom(const pcr_grid& g, const pcr_geom& G, bool swap_xy)
{
    RayGeom r;
    double st = std::sin(G.angle_rad), ct = std::cos(G.angle_rad);
    double s[3] = {G.iso_mm[0] + G.sad_mm * st, G.iso_mm[1] - G.sad_mm * ct, G.iso_mm[2]};
    double dd = G.sdd_mm - G.sad_mm;
    double c[3] = {G.iso_mm[0] - dd * st, G.iso_mm[1] + dd * ct, G.iso_mm[2]};
    double eu[3] = {ct, st, 0.0}, ev[3] = {0.0, 0.0, 1.0};
    for (int a = 0; a < 3; ++a) {
        r.sp[a] = g.spacing_mm[a];
        r.qs[a] = (s[a] - g.origin_mm[a]) / g.spacing_mm[a];
        r.qc[a] = (c[a] - g.origin_mm[a]) / g.spacing_mm[a];
        r.eu[a] = eu[a] / g.spacing_mm[a];
        r.ev[a] = ev[a] / g.spacing_mm[a];
        r.lim[a] = (double)g.n[a];
        r.clo[a] = -1.0;
        r.chi[a] = r.lim[a];
    }
    if (swap_xy) {
        std::swap(r.sp[0], r.sp[1]);
        std::swap(r.qs[0], r.qs[1]);
        std::swap(r.qc[0], r.qc[1]);
        std::swap(r.eu[0], r.eu[1]);
        std::swap(r.ev[0], r.ev[1]);
        std::swap(r.lim[0], r.lim[1]);
        std::swap(r.chi[0], r.chi[1]);
    }
    r.u0 = -0.5 * (G.nu - 1) * G.du_mm + G.off_u_mm;
    r.v0 = -0.5 * (G.nv - 1) * G.dv_mm + G.off_v_mm;
    r.du = G.du_mm;
    r.dv = G.dv_mm;
    r.dt = G.step_mm;
    r.inv_dt = 1.0 / G.step_mm;
    r.nu = G.nu;
    r.nv = G.nv;
    return r;
}

MarchShape choose_march_shape(const RayGeom& rg, pcr_dtype compute, bool projection)
{
    MarchShape ms;
    long rays = (long)rg.nu * rg.nv;
    // aim for >= ~8 waves per SIMD on 1024 SIMDs: split rays into segments
    // when they are few; each wave takes 4 (u) x 16 (v) rays, stepping
    // through the union of their sample ranges together (measured best on
    // both layouts)
    ms.seg = rays >= 8L * 1024 * 64 ? 1 : (rays >= 4L * 1024 * 64 ? 2 : 4);
    // Fewer still, for plain projections: eight segments in blocks of eight
    // waves where an FP32 image is staged.  With under three waves a SIMD a
    // wave's chunks follow each other alone, so halving their number counts:
    // 256x256x100 onto 128x96 pixels 78 -> 56 us, onto 256x192 57 -> 49 us.
    // In FP64 a wave's samples wait for their loads one pair after the other,
    // and sixteen segments pay below 16384 rays: 40^3 onto 64x48 pixels 25 ->
    // 15 us (at 203x151, 0-10 % either way by angle).  (Evaluations keep four:
    // a solve would carry the other grouping of a ray's sum through its line
    // searches.  Eight gained 10 % at 128x96 pixels, and 24-byte cells lost
    // 9 % at 256x192.)
    if (projection && compute == PCR_F32 && rays < 65536) ms.seg = 8;
    if (projection && compute == PCR_F64 && rays < 16384) ms.seg = 16;
    ms.tile_u = 4;
    return ms;
}

static int tiles_u_of(const RayGeom& rg, const MarchShape& ms)
{
    return (rg.nu + ms.tile_u - 1) / ms.tile_u;
}

int march_blocks(const RayGeom& rg, const MarchShape& ms)
{
    int rpb = ms.seg == 8 ? 64 : 256 / ms.seg, rows = rpb / ms.tile_u;
    return tiles_u_of(rg, ms) * ((rg.nv + rows - 1) / rows);
}

// Contraction grid: x-y tiles of 64 x 4 voxels, z split over enough blocks to
// fill the chip (each block then loops over its z slices).
static dim3 contract_grid(const pcr_grid& g)
{
    dim3 d = vox_grid(g);
    unsigned xy = d.x * d.y;
    unsigned zb = std::max(1u, std::min((unsigned)g.n[2], (2048u + xy - 1) / xy));
    return dim3(d.x, d.y, zb);
}

int contract_blocks(const pcr_grid& g)
{
    dim3 d = contract_grid(g);
    return (int)(d.x * d.y * d.z);
}

#define PCR_DISPATCH_S(dt, S, ...)                                   \
    switch (dt) {                                                    \
    case PCR_F32: { using S = float; __VA_ARGS__; } break;           \
    case PCR_F64: { using S = double; __VA_ARGS__; } break;          \
    case PCR_BF16: { using S = bf16; __VA_ARGS__; } break;           \
    case PCR_F16: { using S = _Float16; __VA_ARGS__; } break;        \
    default: return hipErrorInvalidValue;                            \
    }
#define PCR_DISPATCH_R(dt, R, ...)                                   \
    switch (dt) {                                                    \
    case PCR_F32: { using R = float; __VA_ARGS__; } break;           \
    case PCR_F64: { using R = double; __VA_ARGS__; } break;          \
    default: return hipErrorInvalidValue;                            \
    }

hipError_t launch_compose(pcr_dtype compute, pcr_dtype storage, const pcr_grid& g, int K,
                          const void* mean, const void* U, const double* w_eff, void* dvf,
                          hipStream_t s)
{
    const size_t E = 3 * (size_t)g.n[0] * g.n[1] * g.n[2];
    const unsigned blocks = (unsigned)((E + 1023) / 1024);
#define PCR_CO(KK)                                                                                \
    case KK:                                                                                      \
        k_compose<R, S, KK><<<blocks, 256, 0, s>>>((const S*)mean, (const S*)U, E, wvec(w_eff, K), (R*)dvf); \
        break;
    PCR_DISPATCH_R(compute, R, PCR_DISPATCH_S(storage, S,
        switch (K) {
            PCR_CO(1) PCR_CO(2) PCR_CO(3) PCR_CO(4) PCR_CO(5) PCR_CO(6) PCR_CO(7) PCR_CO(8)
        default: return hipErrorInvalidValue;
        }));
#undef PCR_CO
    return hipGetLastError();
}

hipError_t launch_warp_plain(pcr_dtype compute, pcr_dtype f0_dtype, const pcr_grid& g,
                             const void* f0, const void* dvf, void* f, hipStream_t s)
{
    PCR_DISPATCH_R(compute, R, PCR_DISPATCH_S(f0_dtype, S,
        k_warp_plain<R, S><<<vox_grid(g), dim3(64, 4), 0, s>>>((const S*)f0, (const R*)dvf, vox(g),
                                                               (R*)f)));
    return hipGetLastError();
}

template <typename R, typename S, typename F>
static hipError_t warp_fused_c(const pcr_grid& g, const PadLayout& L, int K, bool tangent,
                               const void* f0, const void* mean, const void* U,
                               const double* w_eff, const int* box, void* padded, hipStream_t s)
{
    VoxBox b;
    for (int a = 0; a < 3; ++a) {
        b.lo[a] = box ? std::max(0, box[a]) : 0;
        b.hi[a] = box ? std::min(g.n[a], box[3 + a]) : g.n[a];
        if (b.hi[a] <= b.lo[a]) return hipSuccess;   // nothing to compute
    }
    const int ex = b.hi[0] - b.lo[0], ey = b.hi[1] - b.lo[1], ez = b.hi[2] - b.lo[2];
    dim3 grid((ex + 255) / 256, ey, ez), blk(256, 1);
    auto w = wvec(w_eff, K);
    // one-dimensional grid (the kernel orders its tiles by XCD), tiles of
    // yf_tile_x x 8 voxels
    const int gyy = (ey + 7) / 8;
    auto grid_yf = [&](int tx) { return dim3((unsigned)((long)((ex + tx - 1) / tx) * gyy * ez)); };
    if ((long)((ex + 31) / 32) * gyy * ez > 0x7fffffffL) return hipErrorInvalidValue;
    Chan<float, 8> hs;
    for (int c = 0; c < 8; ++c) hs.v[c] = L.hs[c];
#define PCR_WF2(C, T, H, KM)                                                                      \
    (L.yfast ? k_warp_fused_yf<R, S, F, C, T, H, KM><<<grid_yf(yf_tile_x<R, C, H>()), 256, 0, s>>>( \
                   (const F*)f0, (const S*)mean, (const S*)U, K, w, vox(g), L.px, L.py, hs, b,    \
                   (ex + yf_tile_x<R, C, H>() - 1) / yf_tile_x<R, C, H>(), gyy,                   \
                   (CellOf<R, C, H>*)padded)                                                      \
             : k_warp_fused<R, S, F, C, T, H, KM><<<grid, blk, 0, s>>>(                           \
                   (const F*)f0, (const S*)mean, (const S*)U, K, w, vox(g), L.px, L.py, hs, b,    \
                   (CellOf<R, C, H>*)padded))
#define PCR_WF(C) (L.half ? PCR_WF2(C, true, true, C - 1) : PCR_WF2(C, true, false, C - 1))
#define PCR_WI(KM)                                                                                \
    k_warp_fused<R, S, F, 1, false, false, KM><<<grid, blk, 0, s>>>(                              \
        (const F*)f0, (const S*)mean, (const S*)U, K, w, vox(g), L.px, L.py, hs, b, (CellOf<R, 1, false>*)padded)
    if (L.half && !std::is_same<R, float>::value) return hipErrorInvalidValue;
    if (K < 1 || K > 8 || (tangent && K > L.C - 1)) return hipErrorInvalidValue;
    if (!tangent) {
        // the image alone: one channel, x-fastest
        if (L.C != 1 || L.half || L.yfast) return hipErrorInvalidValue;
        if (K <= 3) PCR_WI(3);
        else if (K <= 5) PCR_WI(5);
        else PCR_WI(8);
    } else {
        switch (L.C) {
        case 2: PCR_WF(2); break;
        case 4: PCR_WF(4); break;
        case 6:
            if (L.half) return hipErrorInvalidValue;
            PCR_WF2(6, true, false, 5);
            break;
        case 8: PCR_WF(8); break;
        default: return hipErrorInvalidValue;
        }
    }
#undef PCR_WI
#undef PCR_WF
#undef PCR_WF2
    return hipGetLastError();
}

hipError_t launch_warp_fused(pcr_dtype compute, pcr_dtype storage, pcr_dtype f0_dtype,
                             const pcr_grid& g, const PadLayout& L, int K, bool tangent,
                             const void* f0, const void* mean, const void* U,
                             const double* w_eff, const int* box, void* padded, hipStream_t s)
{
    PCR_DISPATCH_R(compute, R, PCR_DISPATCH_S(storage, S, PCR_DISPATCH_S(f0_dtype, F,
        return warp_fused_c<R, S, F>(g, L, K, tangent, f0, mean, U, w_eff, box, padded, s))));
    return hipSuccess;
}

hipError_t launch_pad(pcr_dtype compute, const PadLayout& L, const void* vol, void* padded,
                      hipStream_t s)
{
    if (L.C != 1 || L.half || L.yfast) return hipErrorInvalidValue;
    pcr_grid g{};
    g.n[0] = L.nx; g.n[1] = L.ny; g.n[2] = L.nz;
    g.spacing_mm[0] = g.spacing_mm[1] = g.spacing_mm[2] = 1.0;
    const dim3 grid((L.px + 63) / 64, (L.py + 3) / 4, std::min(L.pz, 65535));
    PCR_DISPATCH_R(compute, R,
        k_pad<R><<<grid, dim3(64, 4), 0, s>>>((const R*)vol, vox(g), (R*)padded));
    return hipGetLastError();
}

hipError_t launch_zero(void* p, size_t bytes, hipStream_t s)
{
    // A fill kernel rather than a memset node, so that the call is safe to
    // capture into a graph.  Buffers are whole 4-byte words.
    if (bytes == 0) return hipSuccess;
    if (bytes % 4 != 0 || (uintptr_t)p % 4 != 0) return hipErrorInvalidValue;
    if ((uintptr_t)p % 16 == 0 && bytes % 16 == 0) {
        size_t n16 = bytes / 16;
        unsigned blocks = (unsigned)std::min<size_t>((n16 + 255) / 256, 8192);
        k_zero16<<<blocks, 256, 0, s>>>((uint4*)p, n16);
    } else {
        size_t n4 = bytes / 4;
        unsigned blocks = (unsigned)std::min<size_t>((n4 + 255) / 256, 8192);
        k_zero4<<<blocks, 256, 0, s>>>((uint32_t*)p, n4);
    }
    return hipGetLastError();
}

template <typename R>
static hipError_t march_r(const PadLayout& L, int kc, const RayGeom& rg, const MarchShape& ms,
                          const void* padded, const void* y, void* p_out, double* partials,
                          double* moments, unsigned* arrived, unsigned long long* done,
                          unsigned long long seq, hipStream_t s)
{
    int tiles_u = tiles_u_of(rg, ms);
    int blocks = march_blocks(rg, ms);
#define PCR_MARCH(C)                                                                     \
    k_march<R, C><<<blocks, 256, 0, s>>>(rg, ms, tiles_u, (const Chan<R, C>*)padded, L.px, \
                                         L.py, (float)rg.lim[0], (float)rg.lim[1],         \
                                         (float)rg.lim[2], kc, (const R*)y, (R*)p_out,     \
                                         moments ? partials : nullptr)
    switch (L.C) {
    case 1: PCR_MARCH(1); break;
    case 2: PCR_MARCH(2); break;
    case 4: PCR_MARCH(4); break;
    case 6: PCR_MARCH(6); break;
    case 8: PCR_MARCH(8); break;
    default: return hipErrorInvalidValue;
    }
#undef PCR_MARCH
    if (moments) {
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        return run_reduce(partials, blocks, n_moments(kc), n_moments(L.C), moments, s, arrived, done, seq);
    }
    return hipGetLastError();
}

bool march_f32_fits(const PadLayout& L)
{
    const double cb = (double)L.cell_bytes(4);
    return (double)L.px * L.py * L.pz * cb < 2147483648.0 && (double)L.py * L.pz < 16777216.0 &&
           (double)L.px * cb < 16777216.0;
}

static hipError_t march_f32(const PadLayout& L, int kc, const RayGeom& rg, const MarchShape& ms,
                            const void* padded, bool raw, const void* y, void* p_out, double* partials,
                            double* moments, unsigned* arrived, unsigned long long* done,
                            unsigned long long seq, hipStream_t s)
{
    if (!march_f32_fits(L)) return hipErrorInvalidValue;
    MarchArgs A;
    A.g = rg;
    A.ms = ms;
    A.tiles_u = tiles_u_of(rg, ms);
    A.vol = padded;
    const int cb = (int)L.cell_bytes(4);
    A.px = L.px;
    A.py = L.py;
    A.pz = L.pz;
    // (raw: the caller's volume, without the padding)
    A.ys = (raw ? L.px - 3 : L.px) * cb;
    A.zs = A.ys * (raw ? L.py - 3 : L.py);
    for (int c = 0; c < 8; ++c) A.ihs[c] = 1.0f / L.hs[c];
    for (int a = 0; a < 3; ++a) A.fn1[a] = (float)(rg.lim[a] + 1.0);
    A.kc = kc;
    A.y = (const float*)y;
    A.p_out = (float*)p_out;
    A.partials = moments ? partials : nullptr;
    int blocks = march_blocks(rg, ms);
    const bool fused = moments && done && !L.half && ms.seg <= 4 && blocks <= kFusedSumBlocks;
    A.moments = moments;
    A.arrived = arrived;
    A.done = done;
    A.seq = seq;
    if (L.half && (L.C == 1 || ms.seg > 4)) return hipErrorInvalidValue;
    if (L.half) {
        switch (L.C) {
        case 2: k_march_f16<2><<<blocks, 256, 0, s>>>(A); break;
        case 4: k_march_f16<4><<<blocks, 256, 0, s>>>(A); break;
        case 8: k_march_f16<8><<<blocks, 256, 0, s>>>(A); break;
        default: return hipErrorInvalidValue;
        }
    } else {
        // every FP32 cell size stages through LDS (8-byte cells too: 11-18 %
        // faster than the gather through the L1 at paper scale, K = 1)
        if (ms.seg > 4 && L.C != 1) return hipErrorInvalidValue;
#define PCR_ML(c, kc_) (fused ? k_march_lds<c, kc_, 4, false, true><<<blocks, 256, 0, s>>>(A) \
                               : k_march_lds<c, kc_><<<blocks, 256, 0, s>>>(A))
        switch (L.C) {
        case 1:
            if (raw)
                ms.seg == 8 ? k_march_lds<1, 1, 8, true><<<blocks, 512, 0, s>>>(A)
                            : k_march_lds<1, 1, 4, true><<<blocks, 256, 0, s>>>(A);
            else
                ms.seg == 8 ? k_march_lds<1, 1, 8><<<blocks, 512, 0, s>>>(A) : PCR_ML(1, 1);
            break;
        case 2: PCR_ML(2, 2); break;
        case 4: PCR_ML(4, 4); break;
        case 6:
            // K = 4 sums 5 of the 6 channels.  (Summing only the channels in
            // use pays where the unused ones drop whole loads; 12-byte LDS
            // reads, as for K = 2 in 4-channel cells, were slower than
            // summing the zero channel: 183.6 against 145.6 us at K = 2.)
            if (kc == 5) PCR_ML(6, 5);
            else PCR_ML(6, 6);
            break;
        case 8: PCR_ML(8, 8); break;
        default: return hipErrorInvalidValue;
        }
#undef PCR_ML
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !moments || fused) return e;
    return run_reduce(partials, blocks, n_moments(kc), n_moments(L.C), moments, s, arrived, done, seq);
}

hipError_t launch_march(pcr_dtype compute, const PadLayout& L, int kc, const RayGeom& rg,
                        const MarchShape& ms, const void* padded, const void* y, void* p_out,
                        double* partials, double* moments, unsigned* arrived,
                        unsigned long long* done, unsigned long long seq, hipStream_t s)
{
    if (moments && done && !arrived) return hipErrorInvalidValue;
    if (compute == PCR_F32)
        return march_f32(L, kc, rg, ms, padded, false, y, p_out, partials, moments, arrived, done, seq, s);
    if (compute == PCR_F64)
        return march_r<double>(L, kc, rg, ms, padded, y, p_out, partials, moments, arrived, done, seq, s);
    return hipErrorInvalidValue;
}

bool project_unpadded(pcr_dtype compute, const RayGeom& rg)
{
    // Without the copy a projection saves its pass over the volume (15-25 us
    // at paper scale: 137 -> 126 us there, 64^3 onto 128x96 13.7 -> 10.5 us),
    // but where the rays of a tile spread too far to be staged, the gather
    // through the L1 pays for checking every tap against the volume's edges
    // (256x256x100 onto 40x30: 116 -> 129 us).  The line: whether the cells of
    // four samples of a 4 x 16 tile, at the isocentre's magnification, fit
    // a wave's staging buffer.
    if (compute != PCR_F32) return false;
    double n[3], q = 0.0, d = 0.0;
    for (int a = 0; a < 3; ++a) {
        n[a] = (rg.qc[a] - rg.qs[a]) * rg.sp[a];
        q += n[a] * n[a];
        // depth of the grid's centre along the central ray
        d += (0.5 * (rg.lim[a] - 1.0) - rg.qs[a]) * rg.sp[a] * n[a];
    }
    const double mag = q > 0.0 ? d / q : 1.0, len = std::sqrt(q);
    double cells = 1.0;
    for (int a = 0; a < 3; ++a)
        cells *= mag * (3.0 * rg.du * std::fabs(rg.eu[a]) + 15.0 * rg.dv * std::fabs(rg.ev[a])) +
                 3.0 * rg.dt * std::fabs(n[a]) / (len * rg.sp[a]) + 2.0;
    return cells <= Stage<1, 1>::buf;
}

hipError_t launch_project_f32(const PadLayout& L, const RayGeom& rg, const MarchShape& ms, const void* vol,
                              void* p_out, hipStream_t s)
{
    if (L.C != 1 || L.half || L.yfast) return hipErrorInvalidValue;
    return march_f32(L, 1, rg, ms, vol, true, nullptr, p_out, nullptr, nullptr, nullptr, nullptr, 0, s);
}

hipError_t launch_reduce(const double* partials, int nblocks, int nm, double* out, hipStream_t s)
{
    return run_reduce(partials, nblocks, nm, -1, out, s);
}

hipError_t launch_reduce_publish(const double* partials, int nblocks, int nm, double* out, unsigned* arrived,
                                 unsigned long long* done, unsigned long long seq, hipStream_t s)
{
    if (!arrived || !done) return hipErrorInvalidValue;
    return run_reduce(partials, nblocks, nm, -1, out, s, arrived, done, seq);
}

hipError_t launch_backproject(pcr_dtype compute, const pcr_grid& g, const RayGeom& rg,
                              const void* resid, const void* p, const void* y, double a, double b,
                              double scale, void* out, hipStream_t s)
{
    BPArgs A;
    A.g = rg;
    // footprint geometry (physical, mm): n = unit vector source -> detector
    // centre, e_u / e_v the detector axes; for X in index space the offset
    // from the source is (X - qs) * sp
    double n[3], eu[3], ev[3], nn = 0.0, sdd;
    for (int ax = 0; ax < 3; ++ax) {
        n[ax] = (rg.qc[ax] - rg.qs[ax]) * rg.sp[ax];
        nn += n[ax] * n[ax];
        eu[ax] = rg.eu[ax] * rg.sp[ax];
        ev[ax] = rg.ev[ax] * rg.sp[ax];
    }
    sdd = std::sqrt(nn);
    if (!(sdd > 0.0)) return hipErrorInvalidValue;
    double a0 = 0.0, b0 = 0.0, c0 = 0.0, su = 0.0, sv = 0.0;
    for (int ax = 0; ax < 3; ++ax) {
        n[ax] /= sdd;
        A.F.an[ax] = (float)(rg.sp[ax] * n[ax]);
        A.F.bn[ax] = (float)(rg.sp[ax] * eu[ax]);
        A.F.cn[ax] = (float)(rg.sp[ax] * ev[ax]);
        a0 -= rg.qs[ax] * rg.sp[ax] * n[ax];
        b0 -= rg.qs[ax] * rg.sp[ax] * eu[ax];
        c0 -= rg.qs[ax] * rg.sp[ax] * ev[ax];
        su += (rg.qs[ax] - rg.qc[ax]) * rg.sp[ax] * eu[ax];
        sv += (rg.qs[ax] - rg.qc[ax]) * rg.sp[ax] * ev[ax];
    }
    A.F.a0 = (float)a0;
    A.F.b0 = (float)b0;
    A.F.c0 = (float)c0;
    A.F.sdd = (float)sdd;
    A.F.su = (float)su;
    A.F.sv = (float)sv;
    A.F.u0 = (float)rg.u0;
    A.F.inv_du = (float)(1.0 / rg.du);
    A.F.v0 = (float)rg.v0;
    A.F.inv_dv = (float)(1.0 / rg.dv);
    A.F.nu = rg.nu;
    A.F.nv = rg.nv;
    // bricks of 16 voxels along the rays' dominant in-plane axis by cb x cb
    const double rx = std::fabs(rg.qc[0] - rg.qs[0]) * rg.sp[0], ry = std::fabs(rg.qc[1] - rg.qs[1]) * rg.sp[1];
    A.ax = ry >= rx ? 1 : 0;
    A.nx = g.n[0];
    A.ny = g.n[1];
    A.nz = g.n[2];
    A.a = a;
    A.b = b;
    A.scale = scale;
    auto bricks = [&](int cb) {
        A.bx = A.ax ? cb : 16;
        A.by = A.ax ? 16 : cb;
        A.bz = cb;
        A.nbx = (A.nx + A.bx - 1) / A.bx;
        A.nby = (A.ny + A.by - 1) / A.by;
        return (long)A.nbx * A.nby * ((A.nz + A.bz - 1) / A.bz);
    };
    long blocks = bricks(4);
    if (blocks <= 0 || blocks > 0x7fffffffL) return hipErrorInvalidValue;
    // two samples a turn where no ray moves a voxel or more a sample along A
    // (3-9 % faster at every angle); from there on they touch four voxels or
    // more, one sample's two at a time
    const int mode = rg.dt * 1.001 <= rg.sp[A.ax] ? kPairs : kSingles;
    // steps so small that the half diagonal of a brick and its margin of a
    // voxel holds more samples than the bounds of these modes count
    double diag = 0.0;
    for (int ax = 0; ax < 3; ++ax) {
        const double e = 0.5 * ((ax == A.ax ? 16 : 4) + 1) * rg.sp[ax];
        diag += e * e;
    }
    const bool many = std::sqrt(diag) * rg.inv_dt + 2.0 > (double)kBpReach;
    // 2 x 2 columns make four times the blocks, each column with 64 lanes for
    // its rays (51x57x41 voxels, 623x462 pixels: 4.4 -> 0.54 ms; 48x48x32,
    // 128x96: 38 -> 24 us; 80x80x40, 256x192: 92 -> 80 us).  From 1024 bricks of
    // 4 x 4 on (64^3, equal) the rays staged once per brick count more: 4096
    // bricks 99 against 165 us.  Below, what counts is whether the rays keep
    // the lanes busy for longer than the blocks' own cost (clearing and summing
    // the runs): the samples a column takes, its rays where the volume is
    // nearest the source times the samples of one, against the blocks that each
    // CU goes through (its LDS holds five in FP32, two in FP64).  10x102x110
    // voxels under 13x1 pixels: 12 against 22 us, in FP64 12 against 32.  The
    // line is the best over 450 random calls up to 1.2 M voxels and 0.25 M
    // pixels: in all 2.4 % (FP32) and 2.6 % (FP64) above the better shape of
    // each (2 x 2 wherever there are under 1024 bricks: 7 and 12 %).
    double depth = a0;
    for (int ax = 0; ax < 3; ++ax) {
        const double half = 0.5 * rg.lim[ax] * rg.sp[ax];
        depth += (half - 0.5 * rg.sp[ax]) * n[ax] - half * std::fabs(n[ax]);
    }
    depth = std::max(depth, 0.02 * sdd);
    const int bx = 1 - A.ax;
    const double wide = 2.0 * rg.sp[bx] * std::fabs(eu[bx]) + 17.0 * rg.sp[A.ax] * std::fabs(eu[A.ax]);
    const double rays = std::min((double)rg.nu, wide * sdd / (depth * rg.du)) *
                        std::min((double)rg.nv, 2.0 * rg.sp[2] * sdd / (depth * rg.dv));
    const double samples = std::min(17.0 * rg.sp[A.ax] / std::max(std::fabs(n[A.ax]), 1e-9),
                                    2.0 * rg.sp[bx] / std::max(std::fabs(n[bx]), 1e-9)) * rg.inv_dt;
    const double resident = compute == PCR_F32 ? 1280.0 : 512.0;
    const bool small = !many && blocks < 1024 && rays * samples * resident > 512.0 * (double)bricks(2);
    blocks = bricks(small ? 2 : 4);
#define PCR_BP(CB, MODE) \
    k_backproject_columns<R, CB, MODE><<<(unsigned)blocks, 256, 0, s>>>(A, (const R*)resid, (const R*)p, (const R*)y, (R*)out)
    if (many) {
        PCR_DISPATCH_R(compute, R, PCR_BP(4, kMany));
    } else if (small) {
        PCR_DISPATCH_R(compute, R, if (mode == kPairs) PCR_BP(2, kPairs); else PCR_BP(2, kSingles));
    } else {
        PCR_DISPATCH_R(compute, R, if (mode == kPairs) PCR_BP(4, kPairs); else PCR_BP(4, kSingles));
    }
#undef PCR_BP
    return hipGetLastError();
}

hipError_t launch_contract(pcr_dtype compute, pcr_dtype storage, pcr_dtype f0_dtype,
                           const pcr_grid& g, int K, const void* f0, const void* mean,
                           const void* U, const double* w_eff, const void* gv, double* partials,
                           hipStream_t s)
{
    auto w = wvec(w_eff, K);
#define PCR_CT(KM)                                                                                \
    k_contract<R, S, F, KM><<<contract_grid(g), dim3(64, 4), 0, s>>>(                             \
        (const F*)f0, (const S*)mean, (const S*)U, K, w, vox(g), (const R*)gv, partials)
    PCR_DISPATCH_R(compute, R, PCR_DISPATCH_S(storage, S, PCR_DISPATCH_S(f0_dtype, F,
        if (K <= 3) PCR_CT(3);
        else if (K <= 5) PCR_CT(5);
        else PCR_CT(8))));
#undef PCR_CT
    return hipGetLastError();
}

hipError_t launch_warp_adjoint(pcr_dtype compute, const pcr_grid& g, const void* dvf,
                               const void* gv, void* out, hipStream_t s)
{
    PCR_DISPATCH_R(compute, R,
        k_warp_adjoint<R><<<vox_grid(g), dim3(64, 4), 0, s>>>((const R*)dvf, (const R*)gv, vox(g),
                                                              (R*)out));
    return hipGetLastError();
}

hipError_t launch_support(pcr_dtype f0_dtype, const pcr_grid& g, const void* f0, int* sl,
                          hipStream_t s)
{
    const long nxy = (long)g.n[0] * g.n[1];
    const unsigned bx = (unsigned)std::min<long>((nxy + 2047) / 2048, 32);
    const unsigned bz = (unsigned)std::min(g.n[2], 65535);
    PCR_DISPATCH_S(f0_dtype, F,
        k_support<F><<<dim3(bx, bz), 256, 0, s>>>((const F*)f0, g.n[0], g.n[1], g.n[2], sl));
    return hipGetLastError();
}

hipError_t launch_absmax_rows(pcr_dtype dt, const void* a, size_t n, int rows, float* out,
                              hipStream_t s)
{
    const unsigned bx = (unsigned)std::min<size_t>((n + 1023) / 1024, 256);
    PCR_DISPATCH_S(dt, S,
        k_absmax_rows<S><<<dim3(bx, (unsigned)rows), 256, 0, s>>>((const S*)a, n, out));
    return hipGetLastError();
}

hipError_t launch_localize(pcr_dtype storage, const pcr_grid& g, int K, const void* mean,
                           const void* U, const double* w_eff, const double* p_ref, double tol,
                           int max_iter, double* out, unsigned long long* done, unsigned long long seq,
                           hipStream_t s)
{
    auto w = wvec(w_eff, K);
#define PCR_LO(KM)                                                                              \
    k_localize<S, KM><<<1, 64, 0, s>>>((const S*)mean, (const S*)U, K, w, vox(g), p_ref[0], p_ref[1], \
                                       p_ref[2], g.origin_mm[0], g.origin_mm[1], g.origin_mm[2], tol, \
                                       max_iter, out, done, seq)
    PCR_DISPATCH_S(storage, S,
        if (K == 1) PCR_LO(1);
        else if (K <= 3) PCR_LO(3);
        else if (K <= 5) PCR_LO(5);
        else PCR_LO(8));
#undef PCR_LO
    return hipGetLastError();
}

}  // namespace pcr
