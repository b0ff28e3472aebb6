// Device kernels of the TTN/TDVP library for gfx950 (CDNA4, wave64), apart
// from the contractions: Lanczos reductions with device-resident scalars, the
// tridiagonal exponential of the Krylov projection (scaled Taylor series),
// Cholesky + triangular inverse for CholeskyQR2 gauge moves, precision
// conversions and small helpers.
#include <hip/hip_runtime.h>

#include <initializer_list>

#include <cmath>
#include <cstdint>
#include <cstdio>

#include "lanes.h"
#include "ttn_internal.h"

namespace ttn {

// ---------------------------------------------------------------------------
// reductions for Lanczos
// ---------------------------------------------------------------------------
namespace {

constexpr int RED_THREADS = 256;

__device__ inline double block_sum(double v, double* sh) {
    // wave64 shuffle reduction, then across the four waves of the block
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    const int lane = threadIdx.x % 64, wv = threadIdx.x / 64;
    __syncthreads();
    if (lane == 0) sh[wv] = v;
    __syncthreads();
    double r = 0;
    if (threadIdx.x == 0)
        for (int i = 0; i < (int)(blockDim.x / 64); ++i) r += sh[i];
    return r;   // valid in thread 0
}

// block_sum with the total returned in every thread (sh: blockDim / 64 + 1
// doubles).
__device__ inline double block_sum_all(double v, double* sh) {
    const double r = block_sum(v, sh);
    if (threadIdx.x == 0) sh[blockDim.x / 64] = r;
    __syncthreads();
    const double t = sh[blockDim.x / 64];
    __syncthreads();
    return t;
}

// Sums P values (P a power of two, 2 <= P <= 32) over the block with one
// barrier: a butterfly inside each wave leaves value (l >> 1) & (P - 1),
// summed over the wave, in lane l; the waves' results meet in sh (P per wave).
// Returns the block total of value threadIdx.x in threads 0 .. P-1.
template <int H, int P>
__device__ inline void butterfly_step(double (&a)[P], int lane) {
    // lanes that differ in bit 2H exchange one half of their first 2H values
    const bool hi = (lane & (2 * H)) != 0;
#pragma unroll
    for (int i = 0; i < H; ++i) {
        const double send = hi ? a[i] : a[i + H];
        const double keep = hi ? a[i + H] : a[i];
        a[i] = keep + __shfl_xor(send, 2 * H, 64);
    }
}

template <int P>
__device__ inline double block_sum_p(double (&a)[P], double* sh) {
    static_assert(P >= 2 && P <= 32 && (P & (P - 1)) == 0, "P must be a power of two in [2, 32]");
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if constexpr (P >= 32) butterfly_step<16>(a, lane);
    if constexpr (P >= 16) butterfly_step<8>(a, lane);
    if constexpr (P >= 8) butterfly_step<4>(a, lane);
    if constexpr (P >= 4) butterfly_step<2>(a, lane);
    butterfly_step<1>(a, lane);
    a[0] += __shfl_xor(a[0], 1, 64);
#pragma unroll
    for (int b = 2 * P; b < 64; b <<= 1) a[0] += __shfl_xor(a[0], b, 64);
    const int idx = (lane >> 1) & (P - 1);
    __syncthreads();
    if ((lane & 1) == 0 && lane < 2 * P) sh[P * wv + idx] = a[0];
    __syncthreads();
    double r = 0;
    if (threadIdx.x < P)
        for (int w2 = 0; w2 < (int)(blockDim.x >> 6); ++w2) r += sh[P * w2 + threadIdx.x];
    return r;
}

// smallest power of two >= 2 kc
constexpr int pow2_pairs(int kc) {
    int p = 2;
    while (p < 2 * kc) p *= 2;
    return p;
}

__global__ void k_norm2_partial(const double* x, int64_t n, double* partial, const int* skip) {
    if (skip && *skip) return;
    __shared__ double sh[16];
    double acc = 0;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const double a = x[i], b = x[i + n];
        acc += a * a + b * b;
    }
    const double r = block_sum(acc, sh);
    if (threadIdx.x == 0) partial[blockIdx.x] = r;
}

// Sum of p[start], p[start + step], ... below count, with eight loads in
// flight per thread (independent accumulators) instead of one.
__device__ inline double strided_sum(const double* p, int count, int start, int step) {
    double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    int i = start;
    for (; i + 7 * step < count; i += 8 * step) {
#pragma unroll
        for (int u = 0; u < 8; ++u) acc[u] += p[i + u * step];
    }
    for (; i < count; i += step) acc[0] += p[i];
    return ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
}

__device__ inline double wave_sum_partials(const double* partial, int nb) {
    double s = strided_sum(partial, nb, threadIdx.x, 64);
    for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
    return s;   // valid in lane 0
}

__global__ void k_lz_begin(const double* partial, int nb, LanczosDev* lz, int nonherm) {
    const double s = wave_sum_partials(partial, nb);
    if (threadIdx.x == 0) {
        lz->beta0 = sqrt(s);
        lz->zero = (s == 0.0) ? 1 : 0;
        lz->done = lz->zero;
        lz->m_eff = 0;
        lz->nonherm = nonherm;
    }
}

// y = x / beta (FP64), and its FP32 or planar FP64 copy yf, yp when not null
// (the input of the next matvec); y planar (S == 0) or a slot of a chunked
// Krylov basis with chunk stride S
__global__ void k_scale_by(const double* x, int64_t n, double* y, int64_t S, const LanczosDev* lz, int use_beta0,
                           int j, float* yf, double* yp) {
    if (lz->done) return;
    const double s = 1.0 / (use_beta0 ? lz->beta0 : lz->beta[j]);
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < 2 * n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const double v = x[i] * s;
        y[S ? kch_elem(i, n, S) : i] = v;
        if (yf) yf[i] = (float)v;
        if (yp) yp[i] = v;
    }
}

// v_{j+1} = w / beta_j (y planar, S == 0, or a chunked basis slot) with
// beta_j totalled by every block from the nb
// norm partials of k_sub_fused<2> and the breakdown test of k_lz_beta taken
// alike in every block (block 0 records beta_j, or the breakdown); also the
// FP32 copy yf when yf != nullptr.
__global__ __launch_bounds__(256) void k_scale_next(const double* x, int64_t n, double* y, int64_t S,
                                                  LanczosDev* lz, const double* pnorm, int nb, int j, double tol,
                                                  float* yf, double* yp) {
    if (lz->done) return;
    __shared__ double sh[16];
    __shared__ double s_b;
    const double t = block_sum(strided_sum(pnorm, nb, threadIdx.x, blockDim.x), sh);
    if (threadIdx.x == 0) s_b = sqrt(t);
    __syncthreads();
    const double b = s_b;
    const double bprev = j > 0 ? lz->beta[j - 1] : 0.0;
    const bool stop = !(b > tol * (fabs(lz->alpha[j]) + bprev));
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (stop)
            lz->done = 1;
        else
            lz->beta[j] = b;
    }
    if (stop) return;
    const double inv = 1.0 / b;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < 2 * n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const double v = x[i] * inv;
        y[S ? kch_elem(i, n, S) : i] = v;
        if (yf) yf[i] = (float)v;
        if (yp) yp[i] = v;
    }
}

// The matvec outputs that a Lanczos vector w is the sum of (y[1], y[2] may be
// null); y[0] null: w is there already.
template <typename R>
struct LzOut {
    const R* y[3];
};

// w[i .. i + W) (re, im) from the matvec outputs
template <int W, typename R, typename DV>
__device__ inline void lz_out_load(const LzOut<R>& in, int64_t i, int64_t n, DV& wr, DV& wi) {
    typedef R rv __attribute__((ext_vector_type(W)));
    const rv a = *(const rv*)(in.y[0] + i), b = *(const rv*)(in.y[0] + i + n);
#pragma unroll
    for (int e = 0; e < W; ++e) {
        wr[e] = (double)a[e];
        wi[e] = (double)b[e];
    }
#pragma unroll
    for (int q = 1; q < 3; ++q)
        if (in.y[q]) {
            const rv c = *(const rv*)(in.y[q] + i), d = *(const rv*)(in.y[q] + i + n);
#pragma unroll
            for (int e = 0; e < W; ++e) {
                wr[e] += (double)c[e];
                wi[e] += (double)d[e];
            }
        }
}

// re, im [k] += conj(V_k[i]) w[i] over the thread's elements, W consecutive ones
// per step (16-byte loads for W = 2); w is first formed from `in` (and stored).
template <int KC, int W, typename R>
__device__ inline void multidot_body(const double* V, int64_t S, double* w, int64_t n, const LzOut<R>& in,
                                     double (&re)[KC], double (&im)[KC]) {
    typedef double dv __attribute__((ext_vector_type(W)));
    const int64_t nw = n / W;
    // slot and plane strides: chunked basis (S > 0) or planar vectors (S == 0)
    const int64_t ks = S ? 2 * KCH : 2 * n, ps = S ? KCH : n;
    for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < nw; q += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = q * W;
        const double* Vi = V + (S ? kch_ofs(i, S) : i);
        dv vr[KC], vi[KC];
#pragma unroll
        for (int k = 0; k < KC; ++k) {
            vr[k] = *(const dv*)(Vi + ks * k);
            vi[k] = *(const dv*)(Vi + ks * k + ps);
        }
        dv wr, wi;
        if (in.y[0]) {
            lz_out_load<W>(in, i, n, wr, wi);
            *(dv*)(w + i) = wr;
            *(dv*)(w + i + n) = wi;
        } else {
            wr = *(const dv*)(w + i);
            wi = *(const dv*)(w + i + n);
        }
#pragma unroll
        for (int e = 0; e < W; ++e)
#pragma unroll
            for (int k = 0; k < KC; ++k) {
                re[k] += vr[k][e] * wr[e] + vi[k][e] * wi[e];
                im[k] += vr[k][e] * wi[e] - vi[k][e] * wr[e];
            }
    }
}

// partial[blk][k] = sum_i conj(V_k[i]) w[i] for k < KC (2 KC reals per
// block).  KC is a template argument so that the per-thread arrays hold exactly
// the vectors in use; vectors of even length are read two elements at a time.
template <int KC, typename R>
__global__ __launch_bounds__(256) void k_multidot_partial(const double* V, int64_t S, double* w, int64_t n,
                                                         double* partial, const LanczosDev* lz, LzOut<R> in) {
    if (lz->done) return;
    constexpr int P = pow2_pairs(KC);
    __shared__ double shp[4 * P];
    double re[KC], im[KC];
#pragma unroll
    for (int k = 0; k < KC; ++k) re[k] = im[k] = 0;
    const uintptr_t al = (uintptr_t)V | (uintptr_t)w | (uintptr_t)in.y[0] | (uintptr_t)in.y[1] | (uintptr_t)in.y[2];
    if (n % 2 == 0 && (al & 15) == 0)
        multidot_body<KC, 2, R>(V, S, w, n, in, re, im);
    else
        multidot_body<KC, 1, R>(V, S, w, n, in, re, im);
    double a[P];
#pragma unroll
    for (int k = 0; k < P / 2; ++k) {
        a[2 * k] = k < KC ? re[k] : 0.0;
        a[2 * k + 1] = k < KC ? im[k] : 0.0;
    }
    const double t = block_sum_p<P>(a, shp);
    if (threadIdx.x < 2 * KC) partial[blockIdx.x * 2 * KC + threadIdx.x] = t;
}

// Records the projections tot[2k], tot[2k + 1] (k < kcount) of one
// Gram-Schmidt pass in the Lanczos state; called by thread k of one block.
// alpha_index >= 0 marks the first pass of iteration alpha_index (alpha_j,
// and for an Arnoldi basis the Hessenberg column), -1 the second pass (its
// projections are added to the Hessenberg column).
__device__ inline void lz_record_projection(LanczosDev* lz, const double* tot, int kcount, int alpha_index,
                                            int k) {
    const double re = tot[2 * k], im = tot[2 * k + 1];
    lz->c[2 * k] = re;
    lz->c[2 * k + 1] = im;
    if (k == alpha_index) {
        lz->alpha[k] = re;
        lz->m_eff = k + 1;
    }
    if (lz->nonherm) {
        double* hp = lz->hs + 2 * ((kcount - 1) * KRYLOV_MAX + k);
        if (alpha_index >= 0) {
            hp[0] = re;
            hp[1] = im;
        } else {
            hp[0] += re;
            hp[1] += im;
        }
    }
}

// Totals of the nv <= 32 reals per block of nb block partials (layout
// [block][nv]) into out[0..nv), in an order that does not depend on the
// calling block; 256 threads, sh holds 256 doubles.
__device__ inline void block_partials_total(const double* p, int nb, int nv, double* sh, double* out) {
    const int v = threadIdx.x & 31, g = threadIdx.x >> 5, ng = blockDim.x >> 5;
    double u[4] = {0, 0, 0, 0};
    if (v < nv) {
        int b = g;
        for (; b + 3 * ng < nb; b += 4 * ng) {
#pragma unroll
            for (int q = 0; q < 4; ++q) u[q] += p[(int64_t)(b + q * ng) * nv + v];
        }
        for (; b < nb; b += ng) u[0] += p[(int64_t)b * nv + v];
    }
    sh[32 * g + v] = (u[0] + u[1]) + (u[2] + u[3]);
    __syncthreads();
    if (threadIdx.x < nv) {
        double r = 0;
        for (int q = 0; q < ng; ++q) r += sh[32 * q + threadIdx.x];
        out[threadIdx.x] = r;
    }
    __syncthreads();
}

// Totals of the 2 kcount reals per block (layout of k_multidot_partial) into
// the Lanczos state.  1024 threads: thread (g, v) = (t / 32, t % 32) sums value
// v of blocks g, g + 32, ..., so that each step of the 32 groups reads one
// contiguous stretch of the partials.
__global__ __launch_bounds__(1024) void k_multidot_final(const double* partial, int nb, int kcount,
                                                         LanczosDev* lz, int alpha_index) {
    if (lz->done) return;
    __shared__ double sh[32][33];
    __shared__ double tot[32];
    const int v = threadIdx.x & 31, g = threadIdx.x >> 5;
    const int nv = 2 * kcount;
    double acc = 0;
    if (v < nv) {
        double u[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        int b = g;
        for (; b + 7 * 32 < nb; b += 8 * 32) {
#pragma unroll
            for (int q = 0; q < 8; ++q) u[q] += partial[(int64_t)(b + 32 * q) * nv + v];
        }
        for (; b < nb; b += 32) u[0] += partial[(int64_t)b * nv + v];
        acc = ((u[0] + u[1]) + (u[2] + u[3])) + ((u[4] + u[5]) + (u[6] + u[7]));
    }
    sh[g][v] = acc;
    __syncthreads();
    if (threadIdx.x < 32) {
        double r = 0;
        for (int q = 0; q < 32; ++q) r += sh[q][threadIdx.x];
        tot[threadIdx.x] = r;
    }
    __syncthreads();
    const int k = threadIdx.x;
    if (k >= kcount) return;
    lz_record_projection(lz, tot, kcount, alpha_index, k);
}

// w -= sum_k c_k V_k; then, per block, partial sums of either the new
// projections conj(V_k) w (mode 1, 2 KC reals per block) or |w|^2 (mode 2,
// one real per block).  The coefficients c come from
// the Lanczos state, or, with pin != nullptr, every block totals them from
// the previous pass's nbin block partials itself (the same sums in every
// block) and block 0 records them in the state (alpha_index as in
// lz_record_projection); pin must not alias partial.
template <int MODE, int KC, int W>
__device__ inline void sub_fused_body(const double* V, int64_t S, double* w, int64_t n, const double* c,
                                      double (&pr)[KC], double (&pi)[KC], double& nrm) {
    // W consecutive elements per thread and step (16-byte loads for W = 2)
    typedef double dv __attribute__((ext_vector_type(W)));
    const int64_t nw = n / W;
    // slot and plane strides: chunked basis (S > 0) or planar vectors (S == 0)
    const int64_t ks = S ? 2 * KCH : 2 * n, ps = S ? KCH : n;
    for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < nw; q += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = q * W;
        const double* Vi = V + (S ? kch_ofs(i, S) : i);
        dv vr[KC], vi[KC];
#pragma unroll
        for (int k = 0; k < KC; ++k) {
            vr[k] = *(const dv*)(Vi + ks * k);
            vi[k] = *(const dv*)(Vi + ks * k + ps);
        }
        dv wr = *(const dv*)(w + i), wi = *(const dv*)(w + i + n);
#pragma unroll
        for (int k = 0; k < KC; ++k) {
            const double cr = c[2 * k], ci = c[2 * k + 1];
#pragma unroll
            for (int e = 0; e < W; ++e) {
                wr[e] -= cr * vr[k][e] - ci * vi[k][e];
                wi[e] -= cr * vi[k][e] + ci * vr[k][e];
            }
        }
        *(dv*)(w + i) = wr;
        *(dv*)(w + i + n) = wi;
#pragma unroll
        for (int e = 0; e < W; ++e) {
            if (MODE == 1) {
#pragma unroll
                for (int k = 0; k < KC; ++k) {
                    pr[k] += vr[k][e] * wr[e] + vi[k][e] * wi[e];
                    pi[k] += vr[k][e] * wi[e] - vi[k][e] * wr[e];
                }
            } else if (MODE == 2) {
                nrm += wr[e] * wr[e] + wi[e] * wi[e];
            }
        }
    }
}

template <int MODE, int KC>
__global__ __launch_bounds__(256) void k_sub_fused(const double* V, int64_t S, double* w, int64_t n, double* partial,
                                                   LanczosDev* lz, const double* pin, int nbin, int alpha_index) {
    if (lz->done) return;
    constexpr int P = pow2_pairs(KC);
    __shared__ double c[32];
    __shared__ double sh[16];
    __shared__ double shp[4 * P];
    __shared__ double shq[256];
    if (pin) {
        block_partials_total(pin, nbin, 2 * KC, shq, c);
        if (blockIdx.x == 0 && threadIdx.x < KC) lz_record_projection(lz, c, KC, alpha_index, threadIdx.x);
    } else {
        if (threadIdx.x < 2 * KC) c[threadIdx.x] = lz->c[threadIdx.x];
        __syncthreads();
    }
    double pr[KC], pi[KC], nrm = 0;
#pragma unroll
    for (int k = 0; k < KC; ++k) pr[k] = pi[k] = 0;
    if (n % 2 == 0 && (((uintptr_t)V | (uintptr_t)w) & 15) == 0)
        sub_fused_body<MODE, KC, 2>(V, S, w, n, c, pr, pi, nrm);
    else
        sub_fused_body<MODE, KC, 1>(V, S, w, n, c, pr, pi, nrm);
    if (MODE == 1) {
        double a[P];
#pragma unroll
        for (int k = 0; k < P / 2; ++k) {
            a[2 * k] = k < KC ? pr[k] : 0.0;
            a[2 * k + 1] = k < KC ? pi[k] : 0.0;
        }
        const double t = block_sum_p<P>(a, shp);
        if (threadIdx.x < 2 * KC) partial[blockIdx.x * 2 * KC + threadIdx.x] = t;
    } else if (MODE == 2) {
        const double a = block_sum(nrm, sh);
        if (threadIdx.x == 0) partial[blockIdx.x] = a;
    }
}

// One block does everything between two matvecs of an operator of n <=
// LZ_BLOCK_N entries (the basis V planar, slot stride 2 n): w is the sum of up
// to three matvec outputs (widened from FP32 in the mixed path), c = V^H w
// (alpha_j = Re c_j); unless j is the last index: w -= V c, c' = V^H w, w -= V
// c', beta_j = |w| with the breakdown test, v_{j+1} = w / beta_j, also written to
// x, the next matvec's input.  At these sizes an iteration is bound by its
// launches (four of 4-8 us over many blocks).  A thread owns E elements of w and
// of every basis vector and keeps them in registers, so V is read once: reading
// it again for every pass took 16 us at n = 1296 and eleven vectors, and at n =
// 4096, where it does not fit, 33 us against 25 for the four launches.
constexpr int LZB_THREADS = 512;
static_assert(LZ_BLOCK_N <= 3 * LZB_THREADS, "at most three elements a thread");

// totals of the KC complex partial sums of a block into c (LDS)
template <int KC>
__device__ inline void lzb_totals(const double (&re)[KC], const double (&im)[KC], double* sh, double* c) {
    constexpr int P = pow2_pairs(KC);
    double a[P];
#pragma unroll
    for (int k = 0; k < P / 2; ++k) {
        a[2 * k] = k < KC ? re[k] : 0.0;
        a[2 * k + 1] = k < KC ? im[k] : 0.0;
    }
    const double t = block_sum_p<P>(a, sh);
    if (threadIdx.x < 2 * KC) c[threadIdx.x] = t;
    __syncthreads();
}

template <int KC, int E, typename R>
__global__ __launch_bounds__(LZB_THREADS) void k_lz_iter(double* V, int m, LzOut<R> in, int n, LanczosDev* lz,
                                                        double tol, double* x, float* xf) {
    if (lz->done) return;
    constexpr int j = KC - 1;
    __shared__ double sh[(LZB_THREADS / 64) * pow2_pairs(KC)];
    __shared__ double sh1[LZB_THREADS / 64 + 1];
    __shared__ double c[2 * KRYLOV_MAX];
    // element e of the thread: tid + LZB_THREADS e (zero past the end)
    double vr[KC][E], vi[KC][E], wr[E], wi[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int i = threadIdx.x + LZB_THREADS * e;
        const bool ok = i < n;
        wr[e] = wi[e] = 0.0;
#pragma unroll
        for (int k = 0; k < KC; ++k) {
            vr[k][e] = ok ? V[2 * n * k + i] : 0.0;
            vi[k][e] = ok ? V[2 * n * k + n + i] : 0.0;
        }
        if (ok) {
            wr[e] = (double)in.y[0][i];
            wi[e] = (double)in.y[0][n + i];
#pragma unroll
            for (int q = 1; q < 3; ++q)
                if (in.y[q]) {
                    wr[e] += (double)in.y[q][i];
                    wi[e] += (double)in.y[q][n + i];
                }
        }
    }
    auto project = [&]() {
        double re[KC], im[KC];
#pragma unroll
        for (int k = 0; k < KC; ++k) {
            re[k] = im[k] = 0.0;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                re[k] += vr[k][e] * wr[e] + vi[k][e] * wi[e];
                im[k] += vr[k][e] * wi[e] - vi[k][e] * wr[e];
            }
        }
        lzb_totals<KC>(re, im, sh, c);
    };
    auto subtract = [&]() {
#pragma unroll
        for (int k = 0; k < KC; ++k) {
            const double cr = c[2 * k], ci = c[2 * k + 1];
#pragma unroll
            for (int e = 0; e < E; ++e) {
                wr[e] -= cr * vr[k][e] - ci * vi[k][e];
                wi[e] -= cr * vi[k][e] + ci * vr[k][e];
            }
        }
    };
    project();
    if (threadIdx.x < KC) lz_record_projection(lz, c, KC, j, threadIdx.x);
    if (j == m - 1) return;
    subtract();
    __syncthreads();   // c is read before the second totals replace it
    project();
    if (threadIdx.x < KC && lz->nonherm) lz_record_projection(lz, c, KC, -1, threadIdx.x);
    subtract();
    double nrm = 0.0;
#pragma unroll
    for (int e = 0; e < E; ++e) nrm += wr[e] * wr[e] + wi[e] * wi[e];
    const double b = sqrt(block_sum_all(nrm, sh1));
    const double bprev = j > 0 ? lz->beta[j > 0 ? j - 1 : 0] : 0.0;
    const bool stop = !(b > tol * (fabs(lz->alpha[j]) + bprev));
    if (threadIdx.x == 0) {
        if (stop)
            lz->done = 1;
        else
            lz->beta[j] = b;
    }
    if (stop) return;
    const double inv = 1.0 / b;
    double* vn = V + 2 * n * KC;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int i = threadIdx.x + LZB_THREADS * e;
        if (i >= n) continue;
        const double r = wr[e] * inv, q = wi[e] * inv;
        vn[i] = r;
        vn[n + i] = q;
        if (x) {
            x[i] = r;
            x[n + i] = q;
        }
        if (xf) {
            xf[i] = (float)r;
            xf[n + i] = (float)q;
        }
    }
}

// v_0 = x / |x| for the same operators, with its copies for the first matvec
__global__ __launch_bounds__(LZB_THREADS) void k_lz_begin_block(const double* x, int n, double* v0, LanczosDev* lz,
                                                               int nonherm, double* x0, float* xf) {
    __shared__ double sh[LZB_THREADS / 64 + 1];
    double acc = 0.0;
    for (int i = threadIdx.x; i < 2 * n; i += LZB_THREADS) acc += x[i] * x[i];
    const double t = block_sum_all(acc, sh);
    if (threadIdx.x == 0) {
        lz->beta0 = sqrt(t);
        lz->zero = lz->done = t == 0.0 ? 1 : 0;
        lz->m_eff = 0;
        lz->nonherm = nonherm;
    }
    if (t == 0.0) return;
    const double s = 1.0 / sqrt(t);
    for (int i = threadIdx.x; i < 2 * n; i += LZB_THREADS) {
        const double v = x[i] * s;
        v0[i] = v;
        if (x0) x0[i] = v;
        if (xf) xf[i] = (float)v;
    }
}

__global__ __launch_bounds__(256) void k_lz_beta(const double* partial, int nb, LanczosDev* lz, int j,
                                                 double tol) {
    if (lz->done) return;
    __shared__ double sh[16];
    const double s = block_sum(strided_sum(partial, nb, threadIdx.x, blockDim.x), sh);
    if (threadIdx.x == 0) {
        const double b = sqrt(s);
        const double bprev = j > 0 ? lz->beta[j - 1] : 0.0;
        if (!(b > tol * (fabs(lz->alpha[j]) + bprev)))
            lz->done = 1;
        else
            lz->beta[j] = b;
    }
}

// y = exp(-i tau H) e_1 for the m_eff x m_eff projection H of the Krylov
// basis: the Taylor series of exp(B/s), B = -i tau H, applied s times to the
// vector, with s chosen so that theta = ||B/s||_1 <= 1 and as many terms as
// make the remainder bound of the series, theta^(K+1) / (K+1)! e^theta, fall
// below 1e-18 for every such theta (K = 20: 5e-20).  theta near 1 is where the
// rounding bound of the whole product, s e^theta, and the number of terms per
// unit of tau are both small (theta <= 1/4 takes 2.2 times the terms).  H is
// the real symmetric tridiagonal (alpha, beta) of a Lanczos basis, or the
// complex upper Hessenberg matrix of an Arnoldi basis (columns in hs,
// subdiagonal beta) when lz->nonherm.  The first wave does all of it, lane t
// holding row t of H and element t of the vectors (neighbours by DPP, the norm
// by one wave reduction); a serial chain, so what counts is its latency.  The
// other waves of the block only meet it at the closing barrier.

// entry (row, col) of the projection (re, im), zero outside m x m
__device__ inline double2 lz_h_entry(const LanczosDev* lz, bool herm, int m, int row, int col) {
    double a = 0.0, b = 0.0;
    if (row < 0 || col < 0 || row >= m || col >= m) return make_double2(a, b);
    if (herm) {
        if (row == col)
            a = lz->alpha[col];
        else if (row == col + 1)
            a = lz->beta[col];
        else if (col == row + 1)
            a = lz->beta[row];
    } else if (row <= col) {
        a = lz->hs[2 * (col * KRYLOV_MAX + row)];
        b = lz->hs[2 * (col * KRYLOV_MAX + row) + 1];
    } else if (row == col + 1) {
        a = lz->beta[col];
    }
    return make_double2(a, b);
}

// maximum over the first row of 16 lanes, the same value in every lane
__device__ inline double row0_max(double v) {
    auto step = [](double a, double u) { return u > a ? u : a; };
    v = step(v, dpp_move<DPP_QUAD_XOR1>(v));
    v = step(v, dpp_move<DPP_QUAD_XOR2>(v));
    v = step(v, dpp_move<DPP_ROW_HALF_MIRROR>(v));
    v = step(v, dpp_move<DPP_ROW_MIRROR>(v));
    return lane_value(v, 0);
}

// y: 2 KRYLOV_MAX doubles in LDS
__device__ __forceinline__ void lz_expm_hessenberg(const LanczosDev* lz, double tau, double* y, StepDev* st) {
    constexpr int KM = KRYLOV_MAX;
    const int t = threadIdx.x;
    if (t < 64) {
        const int m = lz->m_eff;
        const bool herm = !lz->nonherm;
        // row t of H (Hessenberg case; the tridiagonal case reads its three
        // entries below)
        double hr[KM], hi[KM];
#pragma unroll
        for (int c = 0; c < KM; ++c) {
            const double2 e = herm ? make_double2(0.0, 0.0) : lz_h_entry(lz, false, m, t, c);
            hr[c] = e.x;
            hi[c] = e.y;
        }
        // H[t][t-1], H[t][t], H[t][t+1] (tridiagonal)
        const double dl = herm ? lz_h_entry(lz, true, m, t, t - 1).x : 0.0;
        const double dd = herm ? lz_h_entry(lz, true, m, t, t).x : 0.0;
        const double du = herm ? lz_h_entry(lz, true, m, t, t + 1).x : 0.0;
        // 1-norm bound of tau H: the largest column sum (the tridiagonal H is
        // symmetric; else lane t sums column t in row order)
        double cs = fabs(dl) + fabs(dd) + fabs(du);
        if (!herm)
            for (int row = 0; row < m; ++row) {
                const double2 e = lz_h_entry(lz, false, m, row, t);
                cs += fabs(e.x) + fabs(e.y);
            }
        double nrm = row0_max(t < m ? cs : 0.0) * fabs(tau);
        int ns = (int)ceil(nrm);
        if (ns < 1) ns = 1;
        constexpr int TERMS = 20;
        const double fk = tau / ns / (t + 1);   // lane k - 1: h / k
        double vr = t == 0 ? 1.0 : 0.0, vi = 0.0;
        for (int rep = 0; rep < ns; ++rep) {
            double tr = vr, ti = vi, wr = vr, wi = vi;
#pragma unroll 4
            for (int k = 1; k <= TERMS; ++k) {
                // term <- (-i h H term) / k
                double sr = 0, si = 0;
                if (herm) {   // rows 0 .. 15 of H lie in one row of lanes
                    sr = dl * dpp_move<DPP_ROW_SHR1>(tr) + dd * tr + du * dpp_move<DPP_ROW_SHL1>(tr);
                    si = dl * dpp_move<DPP_ROW_SHR1>(ti) + dd * ti + du * dpp_move<DPP_ROW_SHL1>(ti);
                } else {
#pragma unroll
                    for (int c = 0; c < KM; ++c) {
                        const double trc = lane_value(tr, c), tic = lane_value(ti, c);
                        sr += hr[c] * trc - hi[c] * tic;
                        si += hr[c] * tic + hi[c] * trc;
                    }
                }
                const double f = lane_value(fk, k - 1);
                if (t < m) {
                    tr = f * si;
                    ti = -f * sr;
                    wr += tr;
                    wi += ti;
                }
            }
            vr = wr;
            vi = wi;
        }
        if (t < KM) {
            y[2 * t] = t < m ? vr : 0.0;
            y[2 * t + 1] = t < m ? vi : 0.0;
        }
        if (t == 0 && st) atomicMin(&st->min_krylov, m);
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------
// Fused evolution of a small operator: x <- exp(-i tau Op) x for an
// effective Hamiltonian with n = DL DR DP <= SMALL_EVOLVE_N entries in one
// workgroup, every vector and operator stack in LDS, FP64 throughout: the
// matvec (the same four stages as the GEMM path), the Krylov recursion with
// two Gram-Schmidt passes, the small exponential and the recombination.
// Replaces about a hundred launches per evolution of the bottom nodes and
// their bonds.
// ---------------------------------------------------------------------------
constexpr int SMALL_THREADS = 1024;

// What bounds it: a serial chain of m Krylov steps in one workgroup (waits for
// LDS, lane reductions and barriers; the arithmetic is small).  So: complex
// numbers interleaved (one 16-byte LDS access each); wave k keeps basis vector
// k in registers and forms the k-th projection alone; subtractions deal the
// basis over the four lanes of a quad; every wave forms the norm for itself,
// and the next product takes the unscaled vector and scales its result: five
// barriers a step.  Operators of n <= SMALL_DENSE_N are formed once as an
// n x n matrix in registers (16 lanes two rows), which leaves one pass per
// product instead of images and sums.
// Measured, m = 12 (us; planar LDS vectors, two passes a product, projections
// through LDS reductions / this): 3 x 3 x 9 node (n = 81) 95 / 48, 16 x 16
// bond over five operators (n = 256) 163 / 86.
constexpr int SMALL_DENSE_N = 96;
constexpr int SMALL_DENSE_COLS = SMALL_DENSE_N / 16;   // of each of a thread's two rows

// The structured product deals the elements i < n <= SMALL_EVOLVE_N so: four
// lanes share each element and split its terms (images and operator stacks
// dealt round-robin), summed by two lane exchanges: lane e + 16 q of wave w
// (e < 16, q < 4) takes part q of the elements i = e + 16 w + SMALL_GROUPS t.
// Each 16-lane row of a wave then reads 16 consecutive entries of one vector
// and one operator entry (no LDS bank conflicts).  The (l, r, p) split of every
// element is tabulated in LDS once per launch (10 bits each).
constexpr int SMALL_SPLIT = 4;
constexpr int SMALL_GROUPS = SMALL_THREADS / SMALL_SPLIT;
static_assert(SMALL_SPLIT * 16 == 64 && SMALL_GROUPS == 16 * (SMALL_THREADS / 64), "four 16-lane parts per wave");
static_assert(SMALL_EVOLVE_N <= 1024, "leg dimensions must fit the 10-bit fields of the index table");
static_assert(KRYLOV_MAX <= SMALL_THREADS / 64, "one wave per Krylov vector");
static_assert(SMALL_DENSE_N * 8 <= SMALL_THREADS && SMALL_DENSE_N % 16 == 0, "16 threads per two rows");

// Row stride of the basis in LDS: 4 (mod 16) entries, so that the four rows a
// quad reads at one element lie on different banks; n where only that fits the
// pool.
inline int small_stride(int n, int m, int64_t doubles, int64_t pool) {
    const int ns = (n + 11) / 16 * 16 + 4;
    return doubles + 2 * (int64_t)(ns - n) * m <= pool ? ns : n;
}

__device__ inline void cmul_add(double2 a, double2 b, double& re, double& im) {
    re += a.x * b.x - a.y * b.y;
    im += a.x * b.y + a.y * b.x;
}

// acc += sum_q op[o + D q] src[base + sq q], q < D
__device__ inline void small_term(const double2* op, int D, int o, const double2* src, int base, int sq, double& ar,
                                  double& ai) {
#pragma unroll 4
    for (int q = 0; q < D; ++q) cmul_add(op[o + D * q], src[base + sq * q], ar, ai);
}

struct SmallOp {
    const double2 *L, *R, *B, *W;   // stacks in LDS (R, B, W may be null)
    int DL, DR, DP, sL, nz;
};

// y = inv Op x; S holds the left (U_k = L_k x, k = 1..sL) and right (Z_j = R_j x)
// images, n entries each.  Ends with a barrier (y is complete).
__device__ void small_matvec(const SmallOp& o, const int* sidx, const double2* x, double inv, double2* S, double2* y) {
    const int DL = o.DL, DR = o.DR, DP = o.DP, sL = o.sL, nz = o.nz;
    const int n = DL * DR * DP;
    const int q = (threadIdx.x >> 4) & (SMALL_SPLIT - 1), g = (threadIdx.x & 15) + 16 * (threadIdx.x >> 6);
    // images: lane q of a quad forms images k = q, q + 4, ... of its elements
    for (int k = q; k < sL + nz; k += SMALL_SPLIT) {
        const bool left = k < sL;
        for (int i = g; i < n; i += SMALL_GROUPS) {
            const int lx = sidx[i] & 1023, rx = (sidx[i] >> 10) & 1023;
            double ar = 0, ai = 0;
            if (left)
                small_term(o.L + DL * DL * (k + 1), DL, lx, x, i - lx, 1, ar, ai);
            else
                small_term(o.R + DR * DR * (k - sL + 1), DR, rx, x, i - DL * rx, DL, ar, ai);
            S[n * k + i] = make_double2(ar, ai);
        }
    }
    __syncthreads();
    // sums: unit 0 is the left block Hamiltonian, units 1..sL+1 the right-leg
    // stack (H_R x, B_i U_i), the next sL+nz+1 the parent-leg stack (H_P x,
    // W U, W Z); lane q takes the units u = q mod 4
    const int uW = 1 + (o.B ? sL + 1 : 0);
    for (int i0 = 0; i0 < n; i0 += SMALL_GROUPS) {
        const int i = i0 + g;
        double ar = 0, ai = 0;
        if (i < n) {
            const int e = sidx[i];
            const int l = e & 1023, r = (e >> 10) & 1023, p = e >> 20;
            if (q == 0) small_term(o.L, DL, l, x, i - l, 1, ar, ai);
            if (o.B)
                for (int k = (q - 1) & (SMALL_SPLIT - 1); k <= sL; k += SMALL_SPLIT)
                    small_term(o.B + DR * DR * k, DR, r, k == 0 ? x : S + n * (k - 1), i - DL * r, DL, ar, ai);
            if (o.W)
                for (int k = (q - uW) & (SMALL_SPLIT - 1); k <= sL + nz; k += SMALL_SPLIT)
                    small_term(o.W + DP * DP * k, DP, p, k == 0 ? x : S + n * (k - 1), i - DL * DR * p, DL * DR, ar,
                               ai);
        }
        // the four lanes of element i (16 apart) all take part
        ar += __shfl_xor(ar, 16, 64);
        ai += __shfl_xor(ai, 16, 64);
        ar += __shfl_xor(ar, 32, 64);
        ai += __shfl_xor(ai, 32, 64);
        if (q == 0 && i < n) y[i] = make_double2(ar * inv, ai * inv);
    }
    __syncthreads();
}

// entry (row, col) of the operator as a matrix; ir, ic are their table entries
__device__ double2 small_entry(const SmallOp& o, int ir, int ic) {
    const int l = ir & 1023, r = (ir >> 10) & 1023, p = ir >> 20;
    const int l2 = ic & 1023, r2 = (ic >> 10) & 1023, p2 = ic >> 20;
    const int el = l + o.DL * l2, er = r + o.DR * r2, ep = p + o.DP * p2;
    const int L2 = o.DL * o.DL, R2 = o.DR * o.DR, P2 = o.DP * o.DP;
    double re = 0, im = 0;
    const double2 one = make_double2(1.0, 0.0);
    if (r == r2 && p == p2) cmul_add(o.L[el], one, re, im);
    if (o.B && p == p2) {
        if (l == l2) cmul_add(o.B[er], one, re, im);
        for (int k = 1; k <= o.sL; ++k) cmul_add(o.L[L2 * k + el], o.B[R2 * k + er], re, im);
    }
    if (o.W && r == r2) {
        if (l == l2) cmul_add(o.W[ep], one, re, im);
        for (int k = 1; k <= o.sL; ++k) cmul_add(o.L[L2 * k + el], o.W[P2 * k + ep], re, im);
    }
    if (o.W && l == l2)
        for (int k = 1; k <= o.nz; ++k) cmul_add(o.R[R2 * k + er], o.W[P2 * (o.sL + k) + ep], re, im);
    return make_double2(re, im);
}

typedef double cb_d4 __attribute__((ext_vector_type(4)));

__device__ inline cb_d4 cb_mfma(double a, double b, cb_d4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// The structured product on the FP64 matrix cores: every operator of the two
// stages is a task per 16 x 16 output tile (rows the operator's leg, columns the
// other two; D padded to 16 in the rows and to 4 in the sum), dealt to the
// waves; the sums' tasks write a slot of their operator, and one pass adds the
// slots.  jt: for every leg, the first element of each of its n / D columns.
struct SmallTasks {
    int tl, tr, tp;                    // tiles of a product on each leg
    const int *jl, *jr, *jp;           // column tables
};
inline __host__ __device__ int small_tiles(int D, int n) { return (D + 15) / 16 * ((n / D + 15) / 16); }
inline __host__ __device__ int small_units(int sL, int nz, bool hasB, bool hasW) {
    return 1 + (hasB ? sL + 1 : 0) + (hasW ? sL + nz + 1 : 0);
}
__device__ inline void small_tile(const double2* op, int D, int sq, const int* jt, int cols, int tile,
                                  const double2* src, double2* dst) {
    const int lane = threadIdx.x & 63, c16 = lane & 15, q4 = lane >> 4;
    const int ot = (D + 15) / 16, o = 16 * (tile % ot) + c16, j0 = 16 * (tile / ot);
    const bool ook = o < D, jok = j0 + c16 < cols;
    const int jb = jok ? jt[j0 + c16] : 0, oo = ook ? o : 0;
    cb_d4 re = {0, 0, 0, 0}, im = {0, 0, 0, 0};
    const double2 none = make_double2(0.0, 0.0);
#pragma unroll 4
    for (int k = 0; k < D; k += 4) {
        const int q = k + q4;
        const double2 a = ook && q < D ? op[oo + D * q] : none;
        const double2 b = jok && q < D ? src[jb + sq * q] : none;
        re = cb_mfma(b.x, a.x, re);
        im = cb_mfma(b.x, a.y, im);
        re = cb_mfma(-b.y, a.y, re);
        im = cb_mfma(b.y, a.x, im);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int j = j0 + q4 + 4 * r;
        if (ook && j < cols) dst[jt[j] + sq * o] = make_double2(re[r], im[r]);
    }
}
__device__ void small_matvec_mfma(const SmallOp& o, const SmallTasks& t, const double2* x, double inv, double2* S,
                                  double2* slots, double2* y) {
    constexpr int WAVES = SMALL_THREADS / 64;
    const int DL = o.DL, DR = o.DR, DP = o.DP, sL = o.sL, nz = o.nz, n = DL * DR * DP;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int e = wave; e < sL * t.tl + nz * t.tr; e += WAVES) {
        if (e < sL * t.tl) {
            const int k = e / t.tl;
            small_tile(o.L + DL * DL * (k + 1), DL, 1, t.jl, n / DL, e - k * t.tl, x, S + n * k);
        } else {
            const int f = e - sL * t.tl, k = f / t.tr;
            small_tile(o.R + DR * DR * (k + 1), DR, DL, t.jr, n / DR, f - k * t.tr, x, S + n * (sL + k));
        }
    }
    __syncthreads();
    const int nB = o.B ? sL + 1 : 0, nW = o.W ? sL + nz + 1 : 0;
    for (int e = wave; e < t.tl + nB * t.tr + nW * t.tp; e += WAVES) {
        if (e < t.tl) {
            small_tile(o.L, DL, 1, t.jl, n / DL, e, x, slots);
        } else if (e < t.tl + nB * t.tr) {
            const int f = e - t.tl, k = f / t.tr;
            small_tile(o.B + DR * DR * k, DR, DL, t.jr, n / DR, f - k * t.tr, k == 0 ? x : S + n * (k - 1),
                       slots + n * (1 + k));
        } else {
            const int f = e - t.tl - nB * t.tr, k = f / t.tp;
            small_tile(o.W + DP * DP * k, DP, DL * DR, t.jp, n / DP, f - k * t.tp, k == 0 ? x : S + n * (k - 1),
                       slots + n * (1 + nB + k));
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += SMALL_THREADS) {
        double re = 0, im = 0;
#pragma unroll 4
        for (int u = 0; u < 1 + nB + nW; ++u) {
            re += slots[n * u + i].x;
            im += slots[n * u + i].y;
        }
        y[i] = make_double2(re * inv, im * inv);
    }
    __syncthreads();
}

// E: entries of a vector per lane (n <= 64 E); up to 4 of them, a wave keeps its
// basis vector in registers, else it reads it from LDS.  FORM: the product as
// loops over the stacks, as a dense matrix, or on the matrix cores.
constexpr int SMALL_LOOPS = 0, SMALL_DENSE = 1, SMALL_MFMA = 2;
// LDS of the matrix-core form, doubles: the stacks and vectors and the slots
constexpr int SMALL_MFMA_POOL = 18432;
template <int E, int FORM>
__global__ __launch_bounds__(SMALL_THREADS) void k_small_evolve(const double* gL, const double* gR, const double* gB,
                                                             const double* gW, int DL, int DR, int DP, int sL,
                                                             int sR, int m, int NS, double tau, double tol,
                                                             int nonherm, double* x, StepDev* st) {
    __shared__ double2 pool[(FORM == SMALL_MFMA ? SMALL_MFMA_POOL : SMALL_EVOLVE_POOL) / 2];
    __shared__ LanczosDev lz;
    __shared__ int sidx[SMALL_EVOLVE_N];
    __shared__ double2 c[KRYLOV_MAX];
    constexpr bool KEEP = E <= 4, DENSE = FORM == SMALL_DENSE;
    constexpr int UNROLL = KEEP ? E : 4;
    const int n = DL * DR * DP;
    const int L2 = DL * DL, R2 = DR * DR, P2 = DP * DP;
    const int nz = (gW && sR > 0) ? sR : 0;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // carve: V[m] (stride NS), the current and the next vector, S[sL + nz], L, R, B, W
    double2* V = pool;
    double2* cur = V + NS * m;
    double2* nxt = cur + n;
    double2* S = nxt + n;
    double2* L = S + n * (sL + nz);
    double2* Rr = L + L2 * (1 + sL);
    double2* B = Rr + (nz ? R2 * (1 + sR) : 0);
    double2* W = B + (gB ? R2 * (1 + sL) : 0);
    // stacks: slots of D^2 entries, planes inside a slot
    auto stage = [&](const double* src, double2* dst, int D2, int slots) {
        for (int e = tid; e < D2 * slots; e += SMALL_THREADS) {
            const int k = e / D2;
            dst[e] = make_double2(src[e + D2 * k], src[e + D2 * (k + 1)]);
        }
    };
    stage(gL, L, L2, 1 + sL);
    if (nz) stage(gR, Rr, R2, 1 + sR);
    if (gB) stage(gB, B, R2, 1 + sL);
    if (gW) stage(gW, W, P2, 1 + sL + sR);
    const SmallOp op{L, nz ? Rr : nullptr, gB ? B : nullptr, gW ? W : nullptr, DL, DR, DP, sL, nz};
    double2* slots = W + (gW ? P2 * (1 + sL + sR) : 0);
    SmallTasks tasks{};
    if constexpr (FORM == SMALL_MFMA) {
        int* jl = sidx;
        int* jr = jl + n / DL;
        int* jp = jr + n / DR;
        for (int j = tid; j < n / DL; j += SMALL_THREADS) jl[j] = DL * j;
        for (int j = tid; j < n / DR; j += SMALL_THREADS) jr[j] = j % DL + DL * DR * (j / DL);
        for (int j = tid; j < n / DP; j += SMALL_THREADS) jp[j] = j;
        tasks = SmallTasks{small_tiles(DL, n), small_tiles(DR, n), small_tiles(DP, n), jl, jr, jp};
    }
    for (int i = tid; i < n; i += SMALL_THREADS) {
        if constexpr (FORM != SMALL_MFMA) sidx[i] = (i % DL) | ((i / DL) % DR) << 10 | (i / (DL * DR)) << 20;
        cur[i] = make_double2(x[i], x[n + i]);
    }
    __syncthreads();
    // sum of |u|^2, the same in every wave
    auto norm2 = [&](const double2* u) {
        double a = 0;
#pragma unroll(UNROLL)
        for (int e = 0; e < E; ++e) {
            const int i = lane + 64 * e;
            const double2 z = i < n ? u[i] : make_double2(0.0, 0.0);
            a += z.x * z.x + z.y * z.y;
        }
        return wave_total(a);
    };
    // basis vector of this wave
    double2 own[KEEP ? E : 1];
#pragma unroll
    for (int e = 0; e < (KEEP ? E : 1); ++e) own[e] = make_double2(0.0, 0.0);
    auto take = [&](int k, const double2* u, double s) {   // v_k = s u, by wave k
        if (wave != k) return;
#pragma unroll(UNROLL)
        for (int e = 0; e < E; ++e) {
            const int i = lane + 64 * e;
            if (i < n) {
                const double2 z = u[i], v = make_double2(z.x * s, z.y * s);
                if constexpr (KEEP) own[e] = v;
                V[NS * k + i] = v;
            }
        }
    };
    auto project = [&](int kc, const double2* u) {   // c_k = <v_k, u>, k < kc
        if (wave < kc) {
            double re = 0, im = 0;
#pragma unroll(UNROLL)
            for (int e = 0; e < E; ++e) {
                const int i = lane + 64 * e;
                const double2 z = i < n ? u[i] : make_double2(0.0, 0.0);
                double2 v;
                if constexpr (KEEP)
                    v = own[e];
                else
                    v = i < n ? V[NS * wave + i] : make_double2(0.0, 0.0);
                re += v.x * z.x + v.y * z.y;
                im += v.x * z.y - v.y * z.x;
            }
            re = wave_total(re);
            im = wave_total(im);
            if (lane == 0) c[wave] = make_double2(re, im);
        }
        __syncthreads();
    };
    // sum_k c_k v_k[i] for i = tid / 4 + 256 t, in all four lanes of a quad
    auto expand = [&](int kc, int i, double& re, double& im) {
        re = im = 0;
        if (i < n)
#pragma unroll 2
            for (int k = tid & 3; k < kc; k += 4) cmul_add(c[k], V[NS * k + i], re, im);
        re += dpp_move<DPP_QUAD_XOR1>(re);
        im += dpp_move<DPP_QUAD_XOR1>(im);
        re += dpp_move<DPP_QUAD_XOR2>(re);
        im += dpp_move<DPP_QUAD_XOR2>(im);
    };
    auto subtract = [&](int kc, double2* u) {
        for (int i0 = 0; i0 < n; i0 += SMALL_GROUPS) {
            const int i = i0 + (tid >> 2);
            double re, im;
            expand(kc, i, re, im);
            if ((tid & 3) == 0 && i < n) {
                const double2 z = u[i];
                u[i] = make_double2(z.x - re, z.y - im);
            }
        }
        __syncthreads();
    };
    const double beta0 = sqrt(norm2(cur));
    if (tid == 0) {
        lz.beta0 = beta0;
        lz.zero = beta0 == 0.0 ? 1 : 0;
        lz.done = lz.zero;
        lz.m_eff = 0;
        lz.nonherm = nonherm;
    }
    if (beta0 == 0.0) return;   // x = 0 stays 0
    double inv = 1.0 / beta0;
    take(0, cur, inv);
    // the operator as a matrix: rows row0 and row0 + 1, columns tid % 16 + 16 t
    const int row0 = 2 * (tid >> 4);
    double2 mat[2][DENSE ? SMALL_DENSE_COLS : 1];
    if constexpr (DENSE) {
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int t = 0; t < SMALL_DENSE_COLS; ++t) {
                const int row = row0 + r, col = (tid & 15) + 16 * t;
                mat[r][t] = row < n && col < n ? small_entry(op, sidx[row], sidx[col]) : make_double2(0.0, 0.0);
            }
    }
    double bprev = 0.0;
    for (int j = 0; j < m; ++j) {
        const int kc = j + 1;
        if constexpr (DENSE) {
            if (8 * wave < n) {   // eight rows a wave
                double re[2] = {0, 0}, im[2] = {0, 0};
#pragma unroll
                for (int t = 0; t < SMALL_DENSE_COLS; ++t) {
                    const int col = (tid & 15) + 16 * t;
                    const double2 z = col < n ? cur[col] : make_double2(0.0, 0.0);
                    cmul_add(mat[0][t], z, re[0], im[0]);
                    cmul_add(mat[1][t], z, re[1], im[1]);
                }
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const double a = row_total(re[r]), b = row_total(im[r]);
                    if ((tid & 15) == 0 && row0 + r < n) nxt[row0 + r] = make_double2(a * inv, b * inv);
                }
            }
            __syncthreads();
        } else if constexpr (FORM == SMALL_MFMA)
            small_matvec_mfma(op, tasks, cur, inv, S, slots, nxt);
        else
            small_matvec(op, sidx, cur, inv, S, nxt);
        project(kc, nxt);
        if (tid == 0) {
            lz.alpha[j] = c[j].x;
            lz.m_eff = kc;
        }
        if (nonherm && tid < kc) {
            lz.hs[2 * (j * KRYLOV_MAX + tid)] = c[tid].x;
            lz.hs[2 * (j * KRYLOV_MAX + tid) + 1] = c[tid].y;
        }
        const double alpha = c[j].x;
        if (j == m - 1) break;
        subtract(kc, nxt);
        project(kc, nxt);
        if (nonherm && tid < kc) {
            lz.hs[2 * (j * KRYLOV_MAX + tid)] += c[tid].x;
            lz.hs[2 * (j * KRYLOV_MAX + tid) + 1] += c[tid].y;
        }
        subtract(kc, nxt);
        const double b = sqrt(norm2(nxt));
        if (!(b > tol * (fabs(alpha) + bprev))) {   // the same in every wave
            if (tid == 0) lz.done = 1;
            break;
        }
        if (tid == 0) lz.beta[j] = b;
        bprev = b;
        inv = 1.0 / b;
        take(kc, nxt, inv);
        double2* const t = cur;
        cur = nxt;
        nxt = t;
    }
    __syncthreads();   // lz and c as the last step left them
    // y = exp(-i tau H_m) e_1, then x = beta0 sum_k y_k v_k
    lz_expm_hessenberg(&lz, tau, (double*)c, st);
    for (int i0 = 0; i0 < n; i0 += SMALL_GROUPS) {
        const int i = i0 + (tid >> 2);
        double re, im;
        expand(lz.m_eff, i, re, im);
        if ((tid & 3) == 0 && i < n) {
            x[i] = re * beta0;
            x[n + i] = im * beta0;
        }
    }
}

// out[k][plane][n] = slot k of the chunked basis V, k < slots (planar copy)
__global__ void k_unchunk(const double* V, int64_t S, int64_t n, int slots, double* out, const int* skip) {
    if (skip && *skip) return;
    const int64_t total = 2 * n * slots;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t k = e / (2 * n), r = e - k * 2 * n;
        out[e] = V[2 * KCH * k + kch_elem(r, n, S)];
    }
}

// out_q = beta0 sum_k y_k v_k, y = exp(-i tau_q H_m) e_1, for q = blockIdx.y (outputs
// 2 n apart); V planar (S == 0, slot stride 2 n) or chunked.  Every block forms
// the small exponential itself (one wave, the same numbers in every block),
// which takes as long as a launch of its own would.  A zero vector stays as it
// is in out, or (fill) its image is written.
struct LzTaus {
    double t[LZ_TAUS];
};
__global__ __launch_bounds__(256) void k_lz_combine(const double* V, int64_t S, int64_t n, double* out0,
                                                   const LanczosDev* lz, LzTaus taus, int fill, StepDev* st) {
    double* out = out0 + 2 * n * blockIdx.y;
    if (lz->zero) {
        if (fill)
            for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < 2 * n;
                 i += (int64_t)gridDim.x * blockDim.x)
                out[i] = 0.0;
        return;
    }
    __shared__ double y[2 * KRYLOV_MAX];
    const int m = lz->m_eff;
    lz_expm_hessenberg(lz, taus.t[blockIdx.y], y, blockIdx.x == 0 ? st : nullptr);
    if (threadIdx.x < 2 * KRYLOV_MAX) y[threadIdx.x] *= lz->beta0;
    __syncthreads();
    if (n % 2 == 0 && (((uintptr_t)V | (uintptr_t)out) & 15) == 0) {   // two elements per step, 16-byte loads
        typedef double d2 __attribute__((ext_vector_type(2)));
        for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < n / 2;
             q += (int64_t)gridDim.x * blockDim.x) {
            const int64_t i = 2 * q;
            d2 re = {0, 0}, im = {0, 0};
            const double* Vi = V + (S ? kch_ofs(i, S) : i);
            const int64_t ks = S ? 2 * KCH : 2 * n, ps = S ? KCH : n;
            for (int k = 0; k < m; ++k) {
                const double* v = Vi + ks * k;
                const d2 vr = *(const d2*)v, vi = *(const d2*)(v + ps);
                re += y[2 * k] * vr - y[2 * k + 1] * vi;
                im += y[2 * k] * vi + y[2 * k + 1] * vr;
            }
            *(d2*)(out + i) = re;
            *(d2*)(out + i + n) = im;
        }
        return;
    }
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        double re = 0, im = 0;
        const double* Vi = V + (S ? kch_ofs(i, S) : i);
        const int64_t ks = S ? 2 * KCH : 2 * n, ps = S ? KCH : n;
        for (int k = 0; k < m; ++k) {
            const double* v = Vi + ks * k;
            const double vr = v[0], vi = v[ps];
            re += y[2 * k] * vr - y[2 * k + 1] * vi;
            im += y[2 * k] * vi + y[2 * k + 1] * vr;
        }
        out[i] = re;
        out[i + n] = im;
    }
}

inline int grid_for(int64_t n) {
    const int64_t b = (n + 255) / 256;
    return (int)std::max<int64_t>(1, std::min<int64_t>(b, 2048));
}

}  // namespace

void lz_start(const double* x, int64_t n, double* v0, int64_t S, LanczosDev* lz, double* partial, int nb,
              hipStream_t s, int nonherm, float* v0f, double* v0p) {
    if (g_dry_run) return;
    hipLaunchKernelGGL(k_norm2_partial, dim3(nb), dim3(RED_THREADS), 0, s, x, n, partial,
                       (const int*)nullptr);
    hipLaunchKernelGGL(k_lz_begin, dim3(1), dim3(64), 0, s, partial, nb, lz, nonherm);
    hipLaunchKernelGGL(k_scale_by, dim3(grid_for(2 * n)), dim3(256), 0, s, x, n, v0, S, lz, 1, 0, v0f, v0p);
}

// Instantiates a launch for every basis size 1 .. KRYLOV_MAX.
#define TTN_KC_DISPATCH(kc, LAUNCH)                    \
    do {                                               \
        switch (kc) {                                  \
            case 1: LAUNCH(1); break;                  \
            case 2: LAUNCH(2); break;                  \
            case 3: LAUNCH(3); break;                  \
            case 4: LAUNCH(4); break;                  \
            case 5: LAUNCH(5); break;                  \
            case 6: LAUNCH(6); break;                  \
            case 7: LAUNCH(7); break;                  \
            case 8: LAUNCH(8); break;                  \
            case 9: LAUNCH(9); break;                  \
            case 10: LAUNCH(10); break;                \
            case 11: LAUNCH(11); break;                \
            case 12: LAUNCH(12); break;                \
            case 13: LAUNCH(13); break;                \
            case 14: LAUNCH(14); break;                \
            case 15: LAUNCH(15); break;                \
            case 16: LAUNCH(16); break;                \
            default: break;                            \
        }                                              \
    } while (0)
static_assert(KRYLOV_MAX == 16, "TTN_KC_DISPATCH covers basis sizes up to 16");

template <typename R>
void lz_project(const double* V, int64_t S, int kcount, double* w, int64_t n, double* partial, int nb, LanczosDev* lz,
                int alpha_index, hipStream_t s, const R* y0, const R* y1, const R* y2, bool total) {
    if (g_dry_run) return;
    const LzOut<R> in{{y0, y1, y2}};
#define TTN_L(KC) \
    hipLaunchKernelGGL((k_multidot_partial<KC, R>), dim3(nb), dim3(RED_THREADS), 0, s, V, S, w, n, partial, lz, in)
    TTN_KC_DISPATCH(kcount, TTN_L);
#undef TTN_L
    if (total)
        hipLaunchKernelGGL(k_multidot_final, dim3(1), dim3(1024), 0, s, partial, nb, kcount, lz, alpha_index);
}
template void lz_project<double>(const double*, int64_t, int, double*, int64_t, double*, int, LanczosDev*, int,
                                 hipStream_t, const double*, const double*, const double*, bool);
template void lz_project<float>(const double*, int64_t, int, double*, int64_t, double*, int, LanczosDev*, int,
                                hipStream_t, const float*, const float*, const float*, bool);

// With fuse (nb <= LZ_FUSE_NB) the totals of the first pass are taken inside
// k_sub_fused<1> from the partials lz_project left at `partial`, and its own
// partials go to partial + LZ_PARTIAL_HALF.
void lz_subtract_project(const double* V, int64_t S, int kcount, double* w, int64_t n, double* partial, int nb,
                         LanczosDev* lz, hipStream_t s, bool fuse) {
    if (g_dry_run) return;
    if (fuse) {
#define TTN_L(KC)                                                                                             \
    hipLaunchKernelGGL((k_sub_fused<1, KC>), dim3(nb), dim3(256), 0, s, V, S, w, n, partial + LZ_PARTIAL_HALF, lz, \
                       (const double*)partial, nb, kcount - 1)
        TTN_KC_DISPATCH(kcount, TTN_L);
#undef TTN_L
        return;
    }
#define TTN_L(KC)                                                                                         \
    hipLaunchKernelGGL((k_sub_fused<1, KC>), dim3(nb), dim3(256), 0, s, V, S, w, n, partial, lz, \
                       (const double*)nullptr, 0, 0)
    TTN_KC_DISPATCH(kcount, TTN_L);
#undef TTN_L
    hipLaunchKernelGGL(k_multidot_final, dim3(1), dim3(1024), 0, s, partial, nb, kcount, lz, -1);
}

// With fuse the second pass's totals are taken inside k_sub_fused<2> from
// partial + LZ_PARTIAL_HALF, and beta_j inside the scaling kernel.
void lz_subtract_next(const double* V, int64_t S, int kcount, double* w, int64_t n, double* vnext, LanczosDev* lz,
                      int j, double* partial, int nb, double tol, hipStream_t s, float* vnextf, bool fuse,
                      double* vnextp) {
    if (g_dry_run) return;
    if (fuse) {
#define TTN_L(KC)                                                                                              \
    hipLaunchKernelGGL((k_sub_fused<2, KC>), dim3(nb), dim3(256), 0, s, V, S, w, n, partial, lz,               \
                       (const double*)(partial + LZ_PARTIAL_HALF), nb, -1)
        TTN_KC_DISPATCH(kcount, TTN_L);
#undef TTN_L
        hipLaunchKernelGGL(k_scale_next, dim3(grid_for(2 * n)), dim3(256), 0, s, w, n, vnext, S, lz,
                           (const double*)partial, nb, j, tol, vnextf, vnextp);
        return;
    }
#define TTN_L(KC)                                                                                         \
    hipLaunchKernelGGL((k_sub_fused<2, KC>), dim3(nb), dim3(256), 0, s, V, S, w, n, partial, lz, \
                       (const double*)nullptr, 0, 0)
    TTN_KC_DISPATCH(kcount, TTN_L);
#undef TTN_L
    hipLaunchKernelGGL(k_lz_beta, dim3(1), dim3(256), 0, s, partial, nb, lz, j, tol);
    hipLaunchKernelGGL(k_scale_by, dim3(grid_for(2 * n)), dim3(256), 0, s, w, n, vnext, S, lz, 0, j, vnextf, vnextp);
}

void lz_start_block(const double* x, int64_t n, double* v0, LanczosDev* lz, hipStream_t s, int nonherm, double* x0,
                    float* xf) {
    if (g_dry_run) return;
    hipLaunchKernelGGL(k_lz_begin_block, dim3(1), dim3(LZB_THREADS), 0, s, x, (int)n, v0, lz, nonherm, x0, xf);
}

template <typename R>
void lz_iter(double* V, int j, int m, const R* y0, const R* y1, const R* y2, int64_t n, LanczosDev* lz, double tol,
             double* x, float* xf, hipStream_t s) {
    if (g_dry_run) return;
    const LzOut<R> in{{y0, y1, y2}};
#define TTN_LE(KC, E)                                                                                               \
    hipLaunchKernelGGL((k_lz_iter<KC, E, R>), dim3(1), dim3(LZB_THREADS), 0, s, V, m, in, (int)n, lz, tol, x, xf)
#define TTN_L(KC)                      \
    if (n <= LZB_THREADS)              \
        TTN_LE(KC, 1);                 \
    else if (n <= 2 * LZB_THREADS)     \
        TTN_LE(KC, 2);                 \
    else                               \
        TTN_LE(KC, 3)
    TTN_KC_DISPATCH(j + 1, TTN_L);
#undef TTN_L
#undef TTN_LE
}
template void lz_iter<double>(double*, int, int, const double*, const double*, const double*, int64_t, LanczosDev*,
                              double, double*, float*, hipStream_t);
template void lz_iter<float>(double*, int, int, const float*, const float*, const float*, int64_t, LanczosDev*,
                             double, double*, float*, hipStream_t);

int64_t small_evolve_doubles(int DL, int DR, int DP, int sL, int sR, int m, bool hasB, bool hasW) {
    const int64_t n = (int64_t)DL * DR * DP;
    const int64_t nz = (hasW && sR > 0) ? sR : 0;
    return 2 * n * (m + 2) + 2 * n * (sL + nz) + 2 * (int64_t)DL * DL * (1 + sL) +
           (nz ? 2 * (int64_t)DR * DR * (1 + sR) : 0) + (hasB ? 2 * (int64_t)DR * DR * (1 + sL) : 0) +
           (hasW ? 2 * (int64_t)DP * DP * (1 + sL + sR) : 0);
}

void small_evolve(const double* L, const double* R, const double* B, const double* W, int DL, int DR, int DP,
                  int sL, int sR, int m, double tau, double tol, bool nonherm, double* x, StepDev* st,
                  hipStream_t s) {
    if (g_dry_run) return;
#define TTN_L(E, D)                                                                                                \
    hipLaunchKernelGGL((k_small_evolve<E, D>), dim3(1), dim3(SMALL_THREADS), 0, s, L, R, B, W, DL, DR, DP, sL, sR, \
                       m, NS, tau, tol, nonherm ? 1 : 0, x, st)
    const int n = DL * DR * DP, nz = W && sR > 0 ? sR : 0;
    // the matrix-core form where its slots fit beside the rest (16 x 16 bond over
    // five operators: 86 us, 109 with the loops)
    const int64_t doubles = small_evolve_doubles(DL, DR, DP, sL, sR, m, B != nullptr, W != nullptr);
    const int64_t slots = 2 * (int64_t)n * small_units(sL, nz, B != nullptr, W != nullptr);
    const bool mfma = n > SMALL_DENSE_N && n <= 256 && doubles + slots <= SMALL_MFMA_POOL;
    const int NS = mfma ? small_stride(n, m, doubles + slots, SMALL_MFMA_POOL)
                        : small_stride(n, m, doubles, SMALL_EVOLVE_POOL);
    if (n <= SMALL_DENSE_N)
        TTN_L(2, SMALL_DENSE);
    else if (mfma)
        TTN_L(4, SMALL_MFMA);
    else if (n <= 256)
        TTN_L(4, SMALL_LOOPS);
    else
        TTN_L(16, SMALL_LOOPS);
#undef TTN_L
}

void lz_expm_combine(const double* V, int64_t S, int64_t n, double* out, const LanczosDev* lz,
                     std::initializer_list<double> taus, bool fill, StepDev* st, hipStream_t s) {
    if (g_dry_run || taus.size() == 0) return;
    LzTaus t{};
    int k = 0;
    for (double x : taus) t.t[k++] = x;
    hipLaunchKernelGGL(k_lz_combine, dim3(grid_for(n), k), dim3(256), 0, s, V, S, n, out, lz, t, fill ? 1 : 0, st);
}

void krylov_unchunk(const double* V, int64_t S, int64_t n, int slots, double* out, const int* skip, hipStream_t s) {
    if (g_dry_run) return;
    hipLaunchKernelGGL(k_unchunk, dim3(grid_for(2 * n * slots)), dim3(256), 0, s, V, S, n, slots, out, skip);
}

// ---------------------------------------------------------------------------
// conversions / copies
// ---------------------------------------------------------------------------
namespace {
// several conversions in one launch: the concatenated index space of the
// arrays
__global__ void k_d2f_batch(D2FBatch b, int64_t total, const int* skip) {
    if (skip && *skip) return;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        int k = 0;
        int64_t off = i;
        while (k < b.n - 1 && off >= b.c[k]) {
            off -= b.c[k];
            ++k;
        }
        const int D = b.eye[k];
        b.y[k][off] = D ? ((off < (int64_t)D * D && off % (D + 1) == 0) ? 1.0f : 0.0f) : (float)b.x[k][off];
    }
}
__global__ void k_copy(const double* x, double* y, int64_t c, const int* skip) {
    if (skip && *skip) return;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < c;
         i += (int64_t)gridDim.x * blockDim.x)
        y[i] = x[i];
}
__global__ void k_zero(double* y, int64_t c) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < c;
         i += (int64_t)gridDim.x * blockDim.x)
        y[i] = 0.0;
}
// y[c + cols*r] = x[r + rows*c] (planar complex, column-major)
__global__ void k_transpose(const double* x, double* y, int rows, int cols) {
    const int64_t n = (int64_t)rows * cols;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int r = (int)(e % rows), c = (int)(e / rows);
        y[c + (int64_t)cols * r] = x[e];
        y[n + c + (int64_t)cols * r] = x[n + e];
    }
}
__global__ void k_herm_f2d(const float* in, double* out, int D, int count, int raw_first) {
    const int64_t D2 = (int64_t)D * D, total = D2 * count;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t k = e / D2, ab = e % D2;
        const int a = (int)(ab % D), b = (int)(ab / D);
        const float* m = in + 2 * D2 * k;
        if (k == 0 && raw_first) {
            out[ab] = (double)m[ab];
            out[D2 + ab] = (double)m[D2 + ab];
            continue;
        }
        const int64_t t = b + (int64_t)D * a;
        out[2 * D2 * k + ab] = 0.5 * ((double)m[ab] + (double)m[t]);
        out[2 * D2 * k + D2 + ab] = 0.5 * ((double)m[D2 + ab] - (double)m[D2 + t]);
    }
}
__global__ void k_sum_mats(const double* src, int64_t D2, int count, double* dst) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < 2 * D2;
         e += (int64_t)gridDim.x * blockDim.x) {
        double a = 0.0;
        for (int k = 0; k < count; ++k) a += src[2 * D2 * k + e];
        dst[e] = a;
    }
}
}  // namespace

void herm_f2d(const float* in, double* out, int D, int count, hipStream_t s, bool raw_first) {
    if (g_dry_run) return;
    const int64_t total = (int64_t)D * D * count;
    hipLaunchKernelGGL(k_herm_f2d, dim3(grid_for(total)), dim3(256), 0, s, in, out, D, count, raw_first ? 1 : 0);
}

void sum_mats(const double* src, int D, int count, double* dst, hipStream_t s) {
    if (g_dry_run) return;
    const int64_t D2 = (int64_t)D * D;
    hipLaunchKernelGGL(k_sum_mats, dim3(grid_for(2 * D2)), dim3(256), 0, s, src, D2, count, dst);
}

void convert_d2f_many(std::initializer_list<D2FItem> items, const int* skip, hipStream_t s) {
    if (g_dry_run) return;
    D2FBatch b{};
    int64_t total = 0;
    for (const D2FItem& it : items) {
        if ((!it.x && it.eye <= 0) || it.count <= 0) continue;
        if (b.n == D2F_MAX) {   // full: flush
            hipLaunchKernelGGL(k_d2f_batch, dim3(grid_for(total)), dim3(256), 0, s, b, total, skip);
            b = D2FBatch{};
            total = 0;
        }
        b.x[b.n] = it.x;
        b.y[b.n] = it.y;
        b.c[b.n] = it.count;
        b.eye[b.n] = it.eye > 0 ? it.eye : 0;
        ++b.n;
        total += it.count;
    }
    if (b.n > 0) hipLaunchKernelGGL(k_d2f_batch, dim3(grid_for(total)), dim3(256), 0, s, b, total, skip);
}
void copy_d(const double* x, double* y, int64_t count, const int* skip, hipStream_t s) {
    if (g_dry_run) return;
    hipLaunchKernelGGL(k_copy, dim3(grid_for(count)), dim3(256), 0, s, x, y, count, skip);
}
void fill_zero_d(double* y, int64_t count, hipStream_t s) {
    if (g_dry_run) return;
    hipLaunchKernelGGL(k_zero, dim3(grid_for(count)), dim3(256), 0, s, y, count);
}
void transpose_c(const double* x, double* y, int rows, int cols, hipStream_t s) {
    if (g_dry_run) return;
    hipLaunchKernelGGL(k_transpose, dim3(grid_for((int64_t)rows * cols)), dim3(256), 0, s, x, y,
                       rows, cols);
}

// ---------------------------------------------------------------------------
// Cholesky + inverse for CholeskyQR2
// ---------------------------------------------------------------------------
namespace {

constexpr int CHOL_THREADS = 512;
constexpr int CHOL_PANEL = 16;
constexpr int CHOL_LDS_MAX = 128;   // packed lower triangle of 128 x 128 fits LDS

__device__ inline int64_t pidx(int i, int j, int D) {   // packed lower, column-major, i >= j
    return (int64_t)j * D - (int64_t)j * (j - 1) / 2 + (i - j);
}

// The second factorization of a gauge move meets G = I + E with E the loss of
// orthogonality of the first: its factor is then R = I + Phi(E) up to second
// order, Phi(E) the strict upper triangle and half the diagonal, and R^{-1} = I -
// Phi(E).  What is left out is at most |E|_F^2 / (2 sqrt 2) in either, so with
// |E|_F^2 <= CHOL_NEAR (|E|_F <= 5e-9) it is below 1e-17, under a tenth of the
// rounding of the entries themselves, and the factorization's serial chain is
// skipped.  Anything else (and NaN) is factored in full.
// Measured, gauge moves of an 8 x 8 lattice, us per second factorization:
// D = 16 11.6 / 4.3, D = 64 43 / 10, D = 128 90 / 20 (full / this).
constexpr double CHOL_NEAR = 2.5e-17;

// min_k of Rprev[k, k] rdiag(k), folded into the step's minimum (positive
// doubles order like their bit patterns), by one wave: the diagonal of the
// product of two upper triangular factors.
template <typename F>
__device__ inline void rdiag_fold(const double* Rprev, int D, F rdiag, StepDev* st, int lane) {
    double mn = 1e308;
    for (int k = lane; k < D; k += 64) {
        const double v = rdiag(k) * Rprev[k + (int64_t)D * k];
        mn = v < mn ? v : mn;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const double t = __shfl_xor(mn, o, 64);
        mn = t < mn ? t : mn;
    }
    if (lane == 0 && mn > 0) atomicMin(&st->min_rdiag_bits, (unsigned long long)__double_as_longlong(mn));
}

// Panel-blocked Cholesky G = L L^H and in-place inverse X = L^{-1} (lower,
// packed, column-major).  Each panel of P columns (Cholesky) or P rows
// (inverse) is processed by the first wave with the panel held in registers
// (RPL rows or columns per lane) and pivots / column entries broadcast by
// cross-lane shuffles; the rank-P updates of the rest of the matrix use the
// whole workgroup between barriers.
template <bool LDS, int RPL, int P>
__global__ __launch_bounds__(CHOL_THREADS) void k_chol_inv(const double* G, int D, double* Linv,
                                                           double* R, const double* Rfirst,
                                                           double* work, StepDev* st) {
    __shared__ double sLre[LDS ? CHOL_LDS_MAX * (CHOL_LDS_MAX + 1) / 2 : 1];
    __shared__ double sLim[LDS ? CHOL_LDS_MAX * (CHOL_LDS_MAX + 1) / 2 : 1];
    __shared__ int s_bad;
    const int64_t np = (int64_t)D * (D + 1) / 2;
    double* Lre = LDS ? sLre : work;
    double* Lim = LDS ? sLim : work + np;
    double* Tre = work + 2 * np;                 // rows x P copy of L for the inverse
    double* Tim = Tre + (int64_t)D * P;
    const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
    const int64_t DD = (int64_t)D * D;
    if (tid == 0) s_bad = 0;
    if (Rfirst) {   // second factorization: near the identity?
        double acc = 0.0;
        for (int64_t e = tid; e < DD; e += CHOL_THREADS) {
            const int i = (int)(e % D), j = (int)(e / D);
            if (i > j)
                acc += 2.0 * (G[e] * G[e] + G[DD + e] * G[DD + e]);
            else if (i == j)
                acc += (G[e] - 1.0) * (G[e] - 1.0);
        }
        __shared__ double s_near[CHOL_THREADS / 64 + 1];
        if (block_sum_all(acc, s_near) <= CHOL_NEAR) {
            for (int64_t e = tid; e < DD; e += CHOL_THREADS) {
                const int i = (int)(e % D), j = (int)(e / D);
                const int64_t t = j + (int64_t)D * i;   // (j, i), of the lower triangle when i <= j
                const double dh = 0.5 * (G[e] - 1.0);
                Linv[e] = i > j ? -G[e] : i == j ? 1.0 - dh : 0.0;
                Linv[DD + e] = i > j ? -G[DD + e] : 0.0;
                R[e] = i < j ? G[t] : i == j ? 1.0 + dh : 0.0;
                R[DD + e] = i < j ? -G[DD + t] : 0.0;
            }
            if (wave == 0)
                rdiag_fold(Rfirst, D, [&](int k) { return 1.0 + 0.5 * (G[k + (int64_t)D * k] - 1.0); }, st, lane);
            return;
        }
    }
    for (int64_t e = tid; e < DD; e += CHOL_THREADS) {
        const int i = (int)(e % D), j = (int)(e / D);
        if (i >= j) {
            Lre[pidx(i, j, D)] = G[e];
            Lim[pidx(i, j, D)] = G[DD + e];
        }
    }
    __syncthreads();
    // ---------------- Cholesky ----------------
    for (int p0 = 0; p0 < D; p0 += P) {
        const int pe = min(p0 + P, D);
        if (wave == 0) {
            double xr[RPL][P], xi[RPL][P];   // rows p0 + lane + 64 r, columns p0 + c
#pragma unroll
            for (int r = 0; r < RPL; ++r) {
                const int i = p0 + lane + 64 * r;
#pragma unroll
                for (int c = 0; c < P; ++c) {
                    const bool ok = i < D && p0 + c < pe && p0 + c <= i;
                    const int64_t q = ok ? pidx(i, p0 + c, D) : 0;
                    xr[r][c] = ok ? Lre[q] : 0.0;
                    xi[r][c] = ok ? Lim[q] : 0.0;
                }
            }
            bool bad = false;
#pragma unroll
            for (int j = 0; j < P; ++j) {
                if (p0 + j < pe) {
                    const double piv = __shfl(xr[0][j], j, 64);   // diagonal: row p0 + j is lane j
                    bad = bad || !(piv > 1e-290);
                    const double d = sqrt(piv > 1e-290 ? piv : 1e-290), dinv = 1.0 / d;
#pragma unroll
                    for (int r = 0; r < RPL; ++r) {
                        const int i = p0 + lane + 64 * r;
                        if (i == p0 + j) {
                            xr[r][j] = d;
                            xi[r][j] = 0.0;
                        } else if (i > p0 + j) {
                            xr[r][j] *= dinv;
                            xi[r][j] *= dinv;
                        }
                    }
#pragma unroll
                    for (int k = j + 1; k < P; ++k) {
                        if (p0 + k < pe) {
                            const double lr = __shfl(xr[0][j], k, 64), li = __shfl(xi[0][j], k, 64);
#pragma unroll
                            for (int r = 0; r < RPL; ++r) {
                                const int i = p0 + lane + 64 * r;
                                if (i >= p0 + k) {   // L[i][k] -= L[i][j] conj(L[k][j])
                                    xr[r][k] -= xr[r][j] * lr + xi[r][j] * li;
                                    xi[r][k] -= xi[r][j] * lr - xr[r][j] * li;
                                }
                            }
                        }
                    }
                }
            }
            if (bad && lane == 0) s_bad = 1;
#pragma unroll
            for (int r = 0; r < RPL; ++r) {
                const int i = p0 + lane + 64 * r;
#pragma unroll
                for (int c = 0; c < P; ++c)
                    if (i < D && p0 + c < pe && p0 + c <= i) {
                        const int64_t q = pidx(i, p0 + c, D);
                        Lre[q] = xr[r][c];
                        Lim[q] = xi[r][c];
                    }
            }
        }
        __syncthreads();
        // trailing update: L[i][k] -= sum_{j in panel} L[i][j] conj(L[k][j]), pe <= k <= i
        const int rn = D - pe;
        for (int64_t e = tid; e < (int64_t)rn * rn; e += CHOL_THREADS) {
            const int ii = (int)(e % rn), kk = (int)(e / rn);
            if (ii < kk) continue;
            const int i = pe + ii, k = pe + kk;
            double sr = 0, si = 0;
            for (int j = p0; j < pe; ++j) {
                const int64_t cj = pidx(j, j, D) - j;
                const double ar = Lre[cj + i], ai = Lim[cj + i];
                const double br = Lre[cj + k], bi = Lim[cj + k];
                sr += ar * br + ai * bi;
                si += ai * br - ar * bi;
            }
            const int64_t q = pidx(i, k, D);
            Lre[q] -= sr;
            Lim[q] -= si;
        }
        __syncthreads();
    }
    // R = L^H
    for (int64_t e = tid; e < DD; e += CHOL_THREADS) {
        const int k = (int)(e % D), a = (int)(e / D);
        double rr = 0, ri = 0;
        if (a >= k) {
            const int64_t ck = pidx(k, k, D) - k;
            rr = Lre[ck + a];
            ri = -Lim[ck + a];
        }
        R[e] = rr;
        R[DD + e] = ri;
    }
    __syncthreads();
    if (tid == 0) {
        double mn = 1e308;
        for (int k = 0; k < D; ++k) {
            const double v = R[k + (int64_t)D * k];
            mn = v < mn ? v : mn;
        }
        if (s_bad || !(mn == mn)) atomicExch(&st->bad, 1);
    }
    if (Rfirst && wave == 1) rdiag_fold(Rfirst, D, [&](int k) { return R[k + (int64_t)D * k]; }, st, lane);
    // ---------------- inverse by elimination on the identity ----------------
    // Position (i, j), i > j, holds L[i][j] until step j and the partial
    // X[i][j] afterwards; the diagonal becomes 1 / L[i][i].
    for (int p0 = 0; p0 < D; p0 += P) {
        const int pe = min(p0 + P, D);
        if (wave == 0) {
            double yr[P][RPL], yi[P][RPL];   // panel rows p0 + t, columns lane + 64 s
#pragma unroll
            for (int t = 0; t < P; ++t)
#pragma unroll
                for (int sl = 0; sl < RPL; ++sl) {
                    const int c = lane + 64 * sl, k = p0 + t;
                    const bool ok = k < pe && c <= k;
                    const int64_t q = ok ? pidx(k, c, D) : 0;
                    yr[t][sl] = ok ? Lre[q] : 0.0;
                    yi[t][sl] = ok ? Lim[q] : 0.0;
                }
#pragma unroll
            for (int t = 0; t < P; ++t) {
                const int k = p0 + t;
                if (k < pe) {
                    const int kl = k & 63, ks = k >> 6;
                    double sel = 0.0;
#pragma unroll
                    for (int sl = 0; sl < RPL; ++sl)
                        if (sl == ks) sel = yr[t][sl];
                    const double d = 1.0 / __shfl(sel, kl, 64);
                    // column k of the later panel rows (still L values)
                    double cr[P], ci[P];
#pragma unroll
                    for (int u = t + 1; u < P; ++u) {
                        double a = 0.0, b2 = 0.0;
#pragma unroll
                        for (int sl = 0; sl < RPL; ++sl)
                            if (sl == ks) {
                                a = yr[u][sl];
                                b2 = yi[u][sl];
                            }
                        cr[u] = __shfl(a, kl, 64);
                        ci[u] = __shfl(b2, kl, 64);
                    }
#pragma unroll
                    for (int sl = 0; sl < RPL; ++sl) {
                        const int c = lane + 64 * sl;
                        if (c < k) {
                            yr[t][sl] *= d;
                            yi[t][sl] *= d;
                        } else if (c == k) {
                            yr[t][sl] = d;
                            yi[t][sl] = 0.0;
                        }
                    }
#pragma unroll
                    for (int u = t + 1; u < P; ++u) {
                        if (p0 + u < pe) {
#pragma unroll
                            for (int sl = 0; sl < RPL; ++sl) {
                                const int c = lane + 64 * sl;
                                if (c <= k) {
                                    const double orr = (c == k) ? 0.0 : yr[u][sl];
                                    const double oii = (c == k) ? 0.0 : yi[u][sl];
                                    yr[u][sl] = orr - (cr[u] * yr[t][sl] - ci[u] * yi[t][sl]);
                                    yi[u][sl] = oii - (cr[u] * yi[t][sl] + ci[u] * yr[t][sl]);
                                }
                            }
                        }
                    }
                }
            }
#pragma unroll
            for (int t = 0; t < P; ++t)
#pragma unroll
                for (int sl = 0; sl < RPL; ++sl) {
                    const int c = lane + 64 * sl, k = p0 + t;
                    if (k < pe && c <= k) {
                        const int64_t q = pidx(k, c, D);
                        Lre[q] = yr[t][sl];
                        Lim[q] = yi[t][sl];
                    }
                }
        }
        const int rn = D - pe;
        // copy L[i][panel] for the rows below the panel (not touched by wave 0)
        for (int e = tid; e < rn * (pe - p0); e += CHOL_THREADS) {
            const int r = e % rn, c = e / rn;
            const int64_t q = pidx(pe + r, p0 + c, D);
            Tre[r + (int64_t)D * c] = Lre[q];
            Tim[r + (int64_t)D * c] = Lim[q];
        }
        __syncthreads();
        // rows i >= pe: X[i][j] = (j in panel ? 0 : X[i][j]) - sum_{k in panel, k >= j} L[i][k] X[k][j]
        for (int64_t e = tid; e < (int64_t)rn * pe; e += CHOL_THREADS) {
            const int r = (int)(e % rn), j = (int)(e / rn);
            const int i = pe + r;
            double sr = 0, si = 0;
            for (int k = max(j, p0); k < pe; ++k) {
                const double lr = Tre[r + (int64_t)D * (k - p0)], li = Tim[r + (int64_t)D * (k - p0)];
                const int64_t qk = pidx(k, j, D);
                const double xr = Lre[qk], xi = Lim[qk];
                sr += lr * xr - li * xi;
                si += lr * xi + li * xr;
            }
            const int64_t qi = pidx(i, j, D);
            const double or_ = (j >= p0) ? 0.0 : Lre[qi];
            const double oi = (j >= p0) ? 0.0 : Lim[qi];
            Lre[qi] = or_ - sr;
            Lim[qi] = oi - si;
        }
        __syncthreads();
    }
    for (int64_t e = tid; e < DD; e += CHOL_THREADS) {
        const int i = (int)(e % D), j = (int)(e / D);
        double xr = 0, xi = 0;
        if (i >= j) {
            xr = Lre[pidx(i, j, D)];
            xi = Lim[pidx(i, j, D)];
        }
        Linv[e] = xr;
        Linv[DD + e] = xi;
    }
}

}  // namespace

namespace {

// Blocked Cholesky + inverse for D <= 128 in one workgroup: the lower
// triangle in 16 x 16 blocks in LDS (36 blocks, 144 KB).  Right-looking by
// block columns: one wave factors the diagonal block (pivots broadcast with
// readlane, columns through LDS), the panel rows are solved by substitution
// (one lane per row), the trailing blocks are updated with the FP64 matrix
// cores while one wave already updates and factors the next diagonal block.
// The inverse: every diagonal block inverted by its own wave, then the block
// diagonals X_IJ = -X_II sum_{K=J}^{I-1} L_IK X_KJ, one level at a time, on
// the matrix cores (the output fragments of one product are the B operand
// fragments of the next).  Sizes that are not a multiple of 16 are padded
// with an identity block.
constexpr int CB = 16;
constexpr int CB_MAXNB = 8;
constexpr int CB_NBLK = CB_MAXNB * (CB_MAXNB + 1) / 2;
constexpr int CB_THREADS = 512;
constexpr int CB_WAVES = CB_THREADS / 64;

__device__ inline int cb_bidx(int I, int J) { return I * (I + 1) / 2 + J; }

__device__ inline double cb_readlane(double v, int src) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), src);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), src);
    return __hiloint2double(hi, lo);
}

__device__ inline void cb_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// O -= A B^H on a 16 x 16 block by one wave with the FP64 matrix cores.
// Fragments: A lane l -> A[l%16][k], B lane l -> B[k][l%16], k = kk + l/16;
// the output register r of lane l is row l/16 + 4 r, column l%16.  The
// products are formed transposed (B as the first operand, A^T as the
// second), so that lane l holds O[l%16][l/16 + 4 r]: the 16 lanes of a row
// group then touch 16 consecutive entries of a column of O in LDS, where
// the untransposed layout strode 16 entries and put them on one bank.
__device__ inline void cb_sub_abh_mfma(const double* Ar, const double* Ai, const double* Br, const double* Bi,
                                       double* Or, double* Oi, int lane) {
    const int m = lane & 15, q = lane >> 4;
    // three real products per complex product (Gauss): with C = conj(B),
    // P1 = Ar Cr^T, P2 = Ai Ci^T, P3 = (Ar + Ai)(Cr + Ci)^T, Re = P1 - P2 and
    // Im = P3 - P1 - P2; independent accumulator chains
    cb_d4 d1 = {0, 0, 0, 0}, d2 = {0, 0, 0, 0}, d3 = {0, 0, 0, 0};
    double ar[4], ai[4], br[4], bi[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int ia = m + CB * (4 * t + q);   // A[m][kk+q]; B^H[kk+q][m] = conj(B[m][kk+q])
        ar[t] = Ar[ia];
        ai[t] = Ai[ia];
        br[t] = Br[ia];
        bi[t] = Bi[ia];
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        d1 = cb_mfma(br[t], ar[t], d1);                    // P1^T
        d2 = cb_mfma(-bi[t], ai[t], d2);                   // P2^T
        d3 = cb_mfma(br[t] - bi[t], ar[t] + ai[t], d3);    // P3^T
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int o = m + CB * (q + 4 * r);
        Or[o] -= d1[r] - d2[r];
        Oi[o] -= d3[r] - d1[r] - d2[r];
    }
}

// Cholesky of the 16 x 16 Hermitian block (br, bi) in place by one wave:
// L lower (upper zeroed); dinv[j] = 1 / L_jj to ds[0..15]; cs: 128 doubles.
// Lane (r, g) holds row r of columns 4 g .. 4 g + 3.  The columns go in four
// groups of four: the 16 lanes of group g factor its columns in registers
// (each pivot and each entry L[c][j] the group's later columns need comes by
// a lane read, no memory round trip), publish the four columns through LDS
// once, and the lanes of the later groups take the rank-4 update.  Every
// entry sees its subtractions in the order j = 0, 1, .., as in the
// column-by-column form.
__device__ inline void cb_chol_diag(double* br, double* bi, double* ds, double* cs, int lane, int& bad) {
    const int r = lane & 15, cg = lane >> 4;
    double a_r[4], a_i[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        a_r[s] = br[r + CB * (4 * cg + s)];
        a_i[s] = bi[r + CB * (4 * cg + s)];
    }
    double* cre = cs;            // [4 columns][16 rows]
    double* cim = cs + 4 * CB;
#pragma unroll
    for (int G = 0; G < 4; ++G) {
        const bool mine = cg == G;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int j = 4 * G + s;
            const double piv = cb_readlane(a_r[s], j + CB * G);
            bad |= !(piv > 1e-290);
            const double pv = piv > 1e-290 ? piv : 1e-290;
            double y = __builtin_amdgcn_rsq(pv);   // 1/sqrt refined by two Newton steps
            y = y * (1.5 - 0.5 * pv * y * y);
            y = y * (1.5 - 0.5 * pv * y * y);
            if (lane == 0) ds[j] = y;
            {
                const double vr = r > j ? a_r[s] * y : (r == j ? pv * y : 0.0);
                const double vi = r > j ? a_i[s] * y : 0.0;
                a_r[s] = mine ? vr : a_r[s];
                a_i[s] = mine ? vi : a_i[s];
            }
            // the group's later columns c: a[r][c] -= L[r][j] conj(L[c][j])
#pragma unroll
            for (int t = s + 1; t < 4; ++t) {
                const int c = 4 * G + t;
                const double cr_ = cb_readlane(a_r[s], c + CB * G), ci_ = cb_readlane(a_i[s], c + CB * G);
                const double lr = a_r[s], li = a_i[s];
                const double ur = a_r[t] - (lr * cr_ + li * ci_);
                const double ui = a_i[t] - (li * cr_ - lr * ci_);
                a_r[t] = mine ? ur : a_r[t];
                a_i[t] = mine ? ui : a_i[t];
            }
        }
        if (G == 3) break;
        if (mine)
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                cre[r + CB * s] = a_r[s];
                cim[r + CB * s] = a_i[s];
            }
        cb_wave_sync();
        if (cg > G) {
            // rank-4 update of the later groups' columns c = 4 cg + t
            double lr[4], li[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                lr[s] = cre[r + CB * s];
                li[s] = cim[r + CB * s];
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int c = 4 * cg + t;
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const double cr_ = cre[c + CB * s], ci_ = cim[c + CB * s];
                    a_r[t] -= lr[s] * cr_ + li[s] * ci_;
                    a_i[t] -= li[s] * cr_ - lr[s] * ci_;
                }
            }
        }
        cb_wave_sync();
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        br[r + CB * (4 * cg + s)] = a_r[s];
        bi[r + CB * (4 * cg + s)] = a_i[s];
    }
}

// X = L^{-1} of the lower block (lr_, li_) (LDS) by one wave, into global
// (xr, xi) with leading dimension ld; ds: dinv; cs: 32 doubles scratch.
__device__ inline void cb_inv_diag(const double* lr_, const double* li_, const double* ds, double* xr, double* xi,
                                   int64_t ld, double* cs, int lane) {
    const int r = lane & 15, cg = lane >> 4;
    double x_r[4], x_i[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        x_r[s] = (r == 4 * cg + s) ? 1.0 : 0.0;
        x_i[s] = 0.0;
    }
    double* rowr = cs;
    double* rowi = cs + CB;
#pragma unroll
    for (int k = 0; k < CB; ++k) {
        if (r == k) {
            const double dk = ds[k];
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                x_r[s] *= dk;
                x_i[s] *= dk;
                rowr[4 * cg + s] = x_r[s];
                rowi[4 * cg + s] = x_i[s];
            }
        }
        cb_wave_sync();
        if (r > k) {
            const double l_r = lr_[r + CB * k], l_i = li_[r + CB * k];
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const double xr_ = rowr[4 * cg + s], xi_ = rowi[4 * cg + s];
                x_r[s] -= l_r * xr_ - l_i * xi_;
                x_i[s] -= l_r * xi_ + l_i * xr_;
            }
        }
        cb_wave_sync();
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        xr[r + ld * (4 * cg + s)] = x_r[s];
        xi[r + ld * (4 * cg + s)] = x_i[s];
    }
}

// G (D x D Hermitian, planar, column-major) = L L^H; Linv = L^{-1} (lower),
// R = L^H (upper).  Rfirst: the R of the first factorization, if this is the
// second (CHOL_NEAR, rdiag_fold).  work: 2 Dp^2 doubles (Dp = 16 ceil(D / 16)), untouched
// when D is a multiple of 16.
__global__ __launch_bounds__(CB_THREADS) void k_chol_blk(const double* G, int D, double* Linv, double* R,
                                                         const double* Rfirst, double* work, StepDev* st) {
    __shared__ double s_re[CB_NBLK * 256], s_im[CB_NBLK * 256];
    __shared__ double s_cs[CB_WAVES * 64];
    __shared__ double s_col[8 * CB];   // the diagonal factorization's four published columns
    __shared__ double s_dinv[CB_MAXNB * CB];
    __shared__ int s_bad;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int NB = (D + CB - 1) / CB, Dp = NB * CB;
    const int64_t DD = (int64_t)D * D, P2 = (int64_t)Dp * Dp;
    // the inverse is built in place in Linv when D is a whole number of
    // blocks (no padding), else in the padded work array and copied out
    const bool direct = Dp == D;
    double* Xr = direct ? Linv : work;   // Dp x Dp column-major
    double* Xi = direct ? Linv + DD : work + P2;
    double* dall = s_dinv;            // 1 / L_jj of every diagonal block, 16 per block
    double* csw = s_cs + 64 * wave;   // per-wave scratch (32 used)
    if (tid == 0) s_bad = 0;
    const int nbl = NB * (NB + 1) / 2;
    {
        // lower blocks of G into LDS (packed by cb_bidx): every load of a
        // thread is issued before its first LDS store
        constexpr int LQ = CB_NBLK * 256 / CB_THREADS;
        static_assert(LQ * CB_THREADS == CB_NBLK * 256, "blocks must split evenly over the threads");
        if (nbl == 1) {   // D <= 16: one block, one entry per thread
            if (tid < 256) {
                const int gi = tid & 15, gj = tid >> 4;
                const bool in = gi < D && gj < D;
                s_re[tid] = in ? G[gi + (int64_t)D * gj] : (gi == gj ? 1.0 : 0.0);
                s_im[tid] = in ? G[DD + gi + (int64_t)D * gj] : 0.0;
            }
        } else {
            double gr[LQ], gim[LQ];
#pragma unroll
            for (int q = 0; q < LQ; ++q) {
                const int e = tid + CB_THREADS * q, b = e >> 8, rc = e & 255;
                // block row of packed block b: the largest I with I (I + 1) / 2 <= b,
                // floor((sqrt(8 b + 1) - 1) / 2); for b < 36 the value stays at
                // least 0.11 below the next integer, so the 0.05 guard absorbs any
                // rounding of the root at the perfect squares
                const int I = (int)((sqrtf((float)(8 * b + 1)) - 1.0f) * 0.5f + 0.05f);
                const int J = b - I * (I + 1) / 2;
                const int gi = CB * I + (rc & 15), gj = CB * J + (rc >> 4);
                const bool in = b < nbl && gi < D && gj < D;
                gr[q] = in ? G[gi + (int64_t)D * gj] : (gi == gj ? 1.0 : 0.0);
                gim[q] = in ? G[DD + gi + (int64_t)D * gj] : 0.0;
            }
#pragma unroll
            for (int q = 0; q < LQ; ++q) {
                const int e = tid + CB_THREADS * q;
                if ((e >> 8) < nbl) {
                    s_re[e] = gr[q];
                    s_im[e] = gim[q];
                }
            }
        }
    }
    __syncthreads();
    auto diag_at = [&](int k) { return 256 * cb_bidx(k >> 4, k >> 4) + (CB + 1) * (k & 15); };
    if (Rfirst) {
        // |G - I|_F^2 from the lower triangle (padded rows are those of I)
        double acc = 0.0;
        for (int I = 0, b = 0; I < NB; ++I)
            for (int J = 0; J <= I; ++J, ++b)
                if (tid < 256) {
                    const int r = tid & 15, c = tid >> 4;
                    const double er = s_re[256 * b + tid] - (I == J && r == c ? 1.0 : 0.0), ei = s_im[256 * b + tid];
                    acc += I > J || r > c ? 2.0 * (er * er + ei * ei) : r == c ? er * er : 0.0;
                }
        if (block_sum_all(acc, s_cs) <= CHOL_NEAR) {
            for (int j = wave; j < D; j += CB_WAVES)
                for (int i = lane; i < D; i += 64) {
                    double xr = 0.0, xi = 0.0, rr = 0.0, ri = 0.0;
                    if (i == j) {
                        const double dh = 0.5 * (s_re[diag_at(j)] - 1.0);
                        xr = 1.0 - dh;
                        rr = 1.0 + dh;
                    } else {
                        const int a = i > j ? i : j, k = i > j ? j : i;   // entry (a, k) of the lower triangle
                        const int q = 256 * cb_bidx(a >> 4, k >> 4) + (a & 15) + CB * (k & 15);
                        (i > j ? xr : rr) = i > j ? -s_re[q] : s_re[q];
                        (i > j ? xi : ri) = -s_im[q];
                    }
                    Linv[i + (int64_t)D * j] = xr;
                    Linv[DD + i + (int64_t)D * j] = xi;
                    R[i + (int64_t)D * j] = rr;
                    R[DD + i + (int64_t)D * j] = ri;
                }
            if (wave == 0)
                rdiag_fold(Rfirst, D, [&](int k) { return 1.0 + 0.5 * (s_re[diag_at(k)] - 1.0); }, st, lane);
            return;
        }
    }
    int bad = 0;
    if (wave == 0) cb_chol_diag(s_re, s_im, dall, s_col, lane, bad);
    __syncthreads();
    for (int K = 0; K < NB; ++K) {
        const double* Lkr = s_re + 256 * cb_bidx(K, K);
        const double* Lki = s_im + 256 * cb_bidx(K, K);
        const double* dsum = dall + CB * K;
        // panel: rows of A_IK (I > K) solve L_IK L_KK^H = A_IK by substitution,
        // column-oriented: once x_k is known it is taken out of every later
        // column at once, so the dependent chain is one product per column
        // (the subtractions of each column still run in the order k = 0, 1, ..)
        const int nrows = CB * (NB - K - 1);
        if (tid < nrows) {
            const int I = K + 1 + tid / CB, r = tid % CB;
            double* ar = s_re + 256 * cb_bidx(I, K);
            double* ai = s_im + 256 * cb_bidx(I, K);
            double xr[CB], xi[CB];
#pragma unroll
            for (int c = 0; c < CB; ++c) {
                xr[c] = ar[r + CB * c];
                xi[c] = ai[r + CB * c];
            }
#pragma unroll
            for (int k = 0; k < CB; ++k) {
                const double dk = dsum[k];
                xr[k] *= dk;
                xi[k] *= dk;
#pragma unroll
                for (int c = k + 1; c < CB; ++c) {   // - x_k conj(L[c][k])
                    const double l_r = Lkr[c + CB * k], l_i = -Lki[c + CB * k];
                    xr[c] -= xr[k] * l_r - xi[k] * l_i;
                    xi[c] -= xr[k] * l_i + xi[k] * l_r;
                }
            }
#pragma unroll
            for (int c = 0; c < CB; ++c) {
                ar[r + CB * c] = xr[c];
                ai[r + CB * c] = xi[c];
            }
        }
        __syncthreads();
        // trailing update A_IJ -= L_IK L_JK^H (K < J <= I); wave 0 first updates
        // the next diagonal block and factors it (look-ahead).  Wave 4, which
        // shares wave 0's SIMD, takes no update blocks, so the factorization's
        // serial chain has that SIMD to itself (it clears the upper blocks of
        // the output once, global stores only); waves 1-3 and 5-7 share the rest
        const int m = NB - K - 1, nt = m * (m + 1) / 2;
        constexpr int UPD = CB_WAVES - 2;
        const int uw = wave < 4 ? wave - 1 : wave - 2;
        if (wave == 0) {
            if (m > 0) {
                const int b1 = cb_bidx(K + 1, K + 1), bk = cb_bidx(K + 1, K);
                cb_sub_abh_mfma(s_re + 256 * bk, s_im + 256 * bk, s_re + 256 * bk, s_im + 256 * bk,
                                s_re + 256 * b1, s_im + 256 * b1, lane);
                cb_wave_sync();
                cb_chol_diag(s_re + 256 * b1, s_im + 256 * b1, dall + CB * (K + 1), s_col, lane, bad);
            }
        } else if (wave == 4) {
            // meanwhile: the blocks (I, J), I < J, of an in-place inverse are
            // zero; the NB (NB - 1) / 2 of them, in order J, then I, are spread
            // over the iterations, ceil(that / NB) per iteration (lane l: row
            // l % 16 of columns 4 s + l / 16, four 128-byte segments a store)
            if (direct) {
                const int nup = NB * (NB - 1) / 2, per = (nup + NB - 1) / NB;
                for (int u = K * per; u < nup && u < (K + 1) * per; ++u) {
                    int J = 1;
                    while (J * (J + 1) / 2 <= u) ++J;
                    const int I = u - J * (J - 1) / 2;
                    const int i = CB * I + (lane & 15);
#pragma unroll
                    for (int s4 = 0; s4 < 4; ++s4) {
                        const int j = CB * J + 4 * s4 + (lane >> 4);
                        Linv[i + (int64_t)D * j] = 0.0;
                        Linv[DD + i + (int64_t)D * j] = 0.0;
                    }
                }
            }
        } else {
            for (int t = uw; t < nt; t += UPD) {
                int ii = 0;
                while ((ii + 1) * (ii + 2) / 2 <= t) ++ii;
                const int jj = t - ii * (ii + 1) / 2;
                if (ii == 0 && jj == 0) continue;   // the next diagonal block (wave 0)
                const int I = K + 1 + ii, J = K + 1 + jj;
                const int bi_ = cb_bidx(I, K), bj = cb_bidx(J, K), bo = cb_bidx(I, J);
                cb_sub_abh_mfma(s_re + 256 * bi_, s_im + 256 * bi_, s_re + 256 * bj, s_im + 256 * bj,
                                s_re + 256 * bo, s_im + 256 * bo, lane);
            }
        }
        __syncthreads();
    }
    if (bad && lane == 0) atomicOr(&s_bad, 1);
    if (Rfirst && wave == CB_WAVES - 1) rdiag_fold(Rfirst, D, [&](int k) { return s_re[diag_at(k)]; }, st, lane);
    // inverses of the diagonal blocks, one wave each
    if (wave < NB)
        cb_inv_diag(s_re + 256 * cb_bidx(wave, wave), s_im + 256 * cb_bidx(wave, wave), dall + CB * wave,
                    Xr + CB * wave + (int64_t)Dp * CB * wave, Xi + CB * wave + (int64_t)Dp * CB * wave, Dp, csw, lane);
    // R = L^H (upper): R[k, a] = conj(L[a, k]); lanes over k, so that a
    // store writes 512 contiguous bytes of a column of R (reading by 16 x 16
    // blocks instead, conflict-free in LDS but with 32-byte store segments,
    // measured slower)
    for (int a = wave; a < D; a += CB_WAVES)
        for (int k = lane; k < D; k += 64) {
            double vr = 0.0, vi = 0.0;
            if (a >= k) {
                const int q = 256 * cb_bidx(a >> 4, k >> 4) + (a & 15) + CB * (k & 15);
                vr = s_re[q];
                vi = -s_im[q];
            }
            R[k + (int64_t)D * a] = vr;
            R[DD + k + (int64_t)D * a] = vi;
        }
    __threadfence_block();
    __syncthreads();
    // inverse by block columns: X_IJ = -X_II sum_{K=J}^{I-1} L_IK X_KJ for
    // I = J + 1 ..; each wave owns one column J (columns 0-3 on waves 0-3 and
    // 7-4 on waves 4-7, so that the two waves sharing a SIMD share the work
    // evenly) and keeps the column's blocks X_KJ as B fragments in registers
    // (the output layout of one product is the B fragment layout of the
    // next), so the waves need no barrier between blocks; only the diagonal
    // inverses X_II, written before the last barrier, come from memory
    static_assert(CB_WAVES == 8 && CB_MAXNB == 8, "one wave per block column");
    {
        const int J = wave < 4 ? wave : 11 - wave;
        const int m = lane & 15, q = lane >> 4;
        double xb_r[4 * CB_MAXNB], xb_i[4 * CB_MAXNB];   // X_{J+t, J}, fragment j of block t
#pragma unroll
        for (int j = 0; j < 4 * CB_MAXNB; ++j) {
            xb_r[j] = 0.0;
            xb_i[j] = 0.0;
        }
        if (J < NB) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int64_t g = (CB * J + 4 * j + q) + (int64_t)Dp * (CB * J + m);
                xb_r[j] = Xr[g];
                xb_i[j] = Xi[g];
            }
        }
#pragma unroll
        for (int dl = 1; dl < CB_MAXNB; ++dl) {
            const int I = J + dl;
            if (I < NB) {
                double xa_r[4], xa_i[4];   // A fragments of X_II[m][kk + q]
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int64_t g = (CB * I + m) + (int64_t)Dp * (CB * I + 4 * j + q);
                    xa_r[j] = Xr[g];
                    xa_i[j] = Xi[g];
                }
                // T = sum_t L_{I,J+t} X_{J+t,J}, three real products per complex
                // product (Gauss): P1 = Lr Xr, P2 = Li Xi, P3 = (Lr + Li)(Xr + Xi),
                // Re T = P1 - P2, Im T = P3 - P1 - P2
                cb_d4 p1 = {0, 0, 0, 0}, p2 = {0, 0, 0, 0}, p3 = {0, 0, 0, 0};
#pragma unroll
                for (int t = 0; t < dl; ++t) {
                    const double* Lr = s_re + 256 * cb_bidx(I, J + t);
                    const double* Li = s_im + 256 * cb_bidx(I, J + t);
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int ia = m + CB * (4 * j + q);
                        const double lr = Lr[ia], li = Li[ia], br = xb_r[4 * t + j], bi = xb_i[4 * t + j];
                        p1 = cb_mfma(lr, br, p1);
                        p2 = cb_mfma(li, bi, p2);
                        p3 = cb_mfma(lr + li, br + bi, p3);
                    }
                }
                const cb_d4 tr = p1 - p2, ti = p3 - p1 - p2;
                // X_IJ = - X_II T, the same three-product form
                cb_d4 q1 = {0, 0, 0, 0}, q2 = {0, 0, 0, 0}, q3 = {0, 0, 0, 0};
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    q1 = cb_mfma(xa_r[j], tr[j], q1);
                    q2 = cb_mfma(xa_i[j], ti[j], q2);
                    q3 = cb_mfma(xa_r[j] + xa_i[j], tr[j] + ti[j], q3);
                }
                const cb_d4 orr = q2 - q1, oi = q1 + q2 - q3;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int64_t g = (CB * I + q + 4 * r) + (int64_t)Dp * (CB * J + m);
                    Xr[g] = orr[r];
                    Xi[g] = oi[r];
                    xb_r[4 * dl + r] = orr[r];
                    xb_i[4 * dl + r] = oi[r];
                }
            }
        }
    }
    __threadfence_block();
    __syncthreads();
    if (!direct)
        for (int j = wave; j < D; j += CB_WAVES)
            for (int i = lane; i < D; i += 64) {
                const bool lo = i >= j;
                const int64_t g = i + (int64_t)Dp * j;
                Linv[i + (int64_t)D * j] = lo ? Xr[g] : 0.0;
                Linv[DD + i + (int64_t)D * j] = lo ? Xi[g] : 0.0;
            }
    __syncthreads();
    if (tid == 0 && s_bad) atomicExch(&st->bad, 1);
}

// A whole gauge move of a small tensor in one workgroup: Gram matrix, Cholesky
// factor and inverse, product, twice (CholeskyQR2), and R = R2 R1.  The tensor is
// D columns of M rows (row index rest = e % s + s (e / (s D)) of element e, column
// (e / s) % D), D <= 16, M <= QRS_ROWS, held in LDS as X[rest][a]; Gram matrices and
// products run on the FP64 matrix cores (16 x 16 tiles, D padded), the waves'
// partial Gram matrices meet in LDS in wave order.
// Bound by the chain of its passes; as seven launches (two of them the
// factorizations) it was bound by those.  Measured, us per move (summed launch
// times / this): 9 x 9 x 16 node 38 / 20, 16 x 16 x 16 node 43 / 25.
constexpr int QRS_ROWS = 256, QRS_THREADS = 512, QRS_WAVES = QRS_THREADS / 64, QRS_LD = CB + 1;
__global__ __launch_bounds__(QRS_THREADS) void k_qr_small(double* T, int n, int D, int s, double* Rout, double* rinvh,
                                                         StepDev* st) {
    __shared__ double2 X[QRS_ROWS * QRS_LD];
    __shared__ double2 part[QRS_WAVES * 256];
    __shared__ double g_re[256], g_im[256];    // Gram matrix, then its factor L
    __shared__ double l_re[2][256], l_im[2][256];   // L^{-1} of both passes
    __shared__ double2 fac[2][256];            // R of both passes, [k + 16 a]
    __shared__ double dinv[CB], cs[8 * CB], sum[QRS_WAVES + 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c16 = lane & 15, q4 = lane >> 4;
    const int M = n / D, Mp = (M + 15) / 16 * 16;
    // the tensor, with zero rows and columns up to whole tiles
    if (Mp * D != n || D < CB)
        for (int e = tid; e < Mp * QRS_LD; e += QRS_THREADS) X[e] = make_double2(0.0, 0.0);
    __syncthreads();
    auto place = [&](int e) {
        const int h = e / s, lo = e - h * s, hi = h / D;
        return (lo + s * hi) * QRS_LD + (h - hi * D);
    };
    for (int e = tid; e < n; e += QRS_THREADS) X[place(e)] = make_double2(T[e], T[n + e]);
    __syncthreads();
    int bad = 0;
    for (int pass = 0; pass < 2; ++pass) {
        // G = X^H X: wave w takes rows 4 (w + 8 i) ..
        cb_d4 re = {0, 0, 0, 0}, im = {0, 0, 0, 0};
        for (int k = 4 * wave; k < Mp; k += 4 * QRS_WAVES) {
            const double2 x = X[(k + q4) * QRS_LD + c16];
            re = cb_mfma(x.x, x.x, re);
            im = cb_mfma(x.y, x.x, im);
            re = cb_mfma(x.y, x.y, re);
            im = cb_mfma(x.x, -x.y, im);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) part[256 * wave + 64 * r + lane] = make_double2(re[r], im[r]);
        __syncthreads();
        double acc = 0.0;   // |G - 1|_F^2
        if (tid < 256) {
            double2 t = part[tid];
#pragma unroll
            for (int w = 1; w < QRS_WAVES; ++w) {
                t.x += part[256 * w + tid].x;
                t.y += part[256 * w + tid].y;
            }
            const int a = tid & 15, b = ((tid & 63) >> 4) + 4 * (tid >> 6);
            if (a == b && a >= D) t.x = 1.0;
            g_re[a + CB * b] = t.x;
            g_im[a + CB * b] = t.y;
            acc = a > b ? 2.0 * (t.x * t.x + t.y * t.y) : a == b ? (t.x - 1.0) * (t.x - 1.0) : 0.0;
        }
        acc = block_sum_all(acc, sum);
        const int a = tid & 15, b = (tid >> 4) & 15, ab = a + CB * b, ba = b + CB * a;
        if (pass == 1 && acc <= CHOL_NEAR) {
            if (tid < 256) {   // L = 1 + E below the diagonal, half of it on it
                const double dh = 0.5 * (g_re[ab] - 1.0);
                l_re[1][ab] = a > b ? -g_re[ab] : a == b ? 1.0 - dh : 0.0;
                l_im[1][ab] = a > b ? -g_im[ab] : 0.0;
                fac[1][ab] = a < b ? make_double2(g_re[ba], -g_im[ba]) : make_double2(a == b ? 1.0 + dh : 0.0, 0.0);
            }
        } else {
            if (wave == 0) {
                cb_chol_diag(g_re, g_im, dinv, cs, lane, bad);
                cb_wave_sync();
                cb_inv_diag(g_re, g_im, dinv, l_re[pass], l_im[pass], CB, cs, lane);
            }
            __syncthreads();
            if (tid < 256) fac[pass][ab] = a <= b ? make_double2(g_re[ba], -g_im[ba]) : make_double2(0.0, 0.0);
        }
        __syncthreads();
        // X <- X L^{-H}, a 16-row tile a wave
        const double* lr = l_re[pass];
        const double* li = l_im[pass];
        for (int t = wave; t < Mp / 16; t += QRS_WAVES) {
            double2* row = X + (16 * t + c16) * QRS_LD;
            cb_d4 yr = {0, 0, 0, 0}, yi = {0, 0, 0, 0};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int k = 4 * j + q4;
                const double2 x = row[k];
                const double br = lr[c16 + CB * k], bi = -li[c16 + CB * k];
                yr = cb_mfma(br, x.x, yr);
                yi = cb_mfma(bi, x.x, yi);
                yr = cb_mfma(-bi, x.y, yr);
                yi = cb_mfma(br, x.y, yi);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) row[q4 + 4 * r] = make_double2(yr[r], yi[r]);
        }
        __syncthreads();
    }
    for (int e = tid; e < n; e += QRS_THREADS) {
        const double2 x = X[place(e)];
        T[e] = x.x;
        T[n + e] = x.y;
    }
    const int a = tid & 15, b = (tid >> 4) & 15, D2 = D * D;
    if (a < D && b < D) {
        if (tid < 256) {   // R[a, b]
            double re = 0, im = 0;
            for (int j = a; j <= b; ++j) {
                const double2 x = fac[1][a + CB * j], y = fac[0][j + CB * b];
                re += x.x * y.x - x.y * y.y;
                im += x.x * y.y + x.y * y.x;
            }
            Rout[a + D * b] = re;
            Rout[D2 + a + D * b] = im;
        } else if (rinvh) {   // R^{-H} = L2^{-1} L1^{-1}
            double re = 0, im = 0;
            for (int j = b; j <= a; ++j) {
                const double xr = l_re[1][a + CB * j], xi = l_im[1][a + CB * j];
                const double yr = l_re[0][j + CB * b], yi = l_im[0][j + CB * b];
                re += xr * yr - xi * yi;
                im += xr * yi + xi * yr;
            }
            rinvh[a + D * b] = re;
            rinvh[D2 + a + D * b] = im;
        }
    }
    if (wave == 0) {
        if (bad && lane == 0) atomicExch(&st->bad, 1);
        double mn = lane < D ? fac[1][17 * lane].x * fac[0][17 * lane].x : 1e308;
        mn = mn < 1e308 ? mn : 1e308;
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) {
            const double t = __shfl_xor(mn, o, 64);
            mn = t < mn ? t : mn;
        }
        if (lane == 0 && mn > 0) atomicMin(&st->min_rdiag_bits, (unsigned long long)__double_as_longlong(mn));
    }
}

}  // namespace

bool qr_small_fits(int DL, int DR, int DP, int leg) {
    const int64_t D = leg == 0 ? DL : leg == 1 ? DR : DP, n = (int64_t)DL * DR * DP;
    return D <= CB && n / D <= QRS_ROWS;
}
void qr_small(double* T, int DL, int DR, int DP, int leg, double* Rout, double* rinvh, StepDev* st, hipStream_t s) {
    if (g_dry_run) return;
    const int D = leg == 0 ? DL : leg == 1 ? DR : DP, stride = leg == 0 ? 1 : leg == 1 ? DL : DL * DR;
    hipLaunchKernelGGL(k_qr_small, dim3(1), dim3(QRS_THREADS), 0, s, T, DL * DR * DP, D, stride, Rout, rinvh, st);
}

void chol_inv(const double* G, int D, double* Linv, double* R, const double* Rfirst, double* work,
              StepDev* st, hipStream_t s) {
    if (g_dry_run) return;
    if (D <= CB * CB_MAXNB)
        hipLaunchKernelGGL(k_chol_blk, dim3(1), dim3(CB_THREADS), 0, s, G, D, Linv, R, Rfirst, work, st);
    else
        hipLaunchKernelGGL((k_chol_inv<false, 4, 8>), dim3(1), dim3(CHOL_THREADS), 0, s, G, D, Linv, R, Rfirst,
                           work, st);
}

// ---------------------------------------------------------------------------
// Hermitian eigendecomposition (cyclic Jacobi) for the two-site split
// ---------------------------------------------------------------------------
namespace {
constexpr int JAC_THREADS = 1024;

// The block form.  Indices are grouped in blocks of JB = 16; a round pairs
// the blocks up (round-robin, all pairs once per sweep), the JW x JW diagonal
// matrix of every pair is rotated in LDS by cyclic Jacobi (k_jacobi_solve, one
// workgroup per pair) -- the JB^2 rotations between its two blocks, and in the
// first round of a sweep those inside the blocks too, so that a sweep meets
// every index pair once -- and the product U of its rotations is applied to
// the rest (k_jacobi_apply): A_PQ <- U_P^H A_PQ U_Q for every two pairs P < Q
// (the mirror image is written with it) and V <- V U by row blocks, on the FP64
// matrix cores.  The rotations, and the tests by which a pair is skipped, are
// those of k_herm_jacobi below.
//   Matrices of up to JAC_ONE rows are one pair of up to that width, rotated to
// the end in one launch (k_jacobi_one; 48 rows take 113 KB of LDS, 64 would take
// 200), where one and two pairs of the block form with their launches were
// slower than the one workgroup in global memory up to 20 and from 33 to 38 rows.
// Measured, us a call with the allocation of its work (that workgroup / the block
// form / this): n = 8 121 / 303 / 73, 16 238 / 365 / 133, 24 480 / 399 / 238, 33
// 864 / 1231 / 569, 40 1270 / 1360 / 616, 48 1930 / 1370 / 946.
//   Bound by the serial chain of rotations (0.6-0.9 us per step of JB
// disjoint rotations in LDS) and its launches: a round takes 13 us in
// k_jacobi_solve and 7 in k_jacobi_apply, a launch after convergence 1.7.
// 144 x 144, spectrum over six decades, 16 sweeps: 44.4 ms in one workgroup
// with the matrix in global memory (31 us per step of 72 rotations) -> 3.8;
// 256 x 256: 264 -> 6.7.  Measured and dropped: every workgroup rotating
// its own copy of P and Q (one launch per round, 28 us), LDS rows of 36 and 48
// doubles (conflicts along columns, 19 us), the products of U formed by the
// threads that rotate the matrix (17 us).
constexpr int JB = 16;
constexpr int JW = 2 * JB;           // width of a pair
constexpr int JS_THREADS = 512;
constexpr int JA_THREADS = 512;
constexpr int JAC_ONE = 48;          // widest matrix of k_jacobi_one
constexpr int JAC_SWEEPS = 28;       // block sweeps enqueued before k_herm_jacobi takes what is left

// State of the iteration.
struct JacState {
    double floor;                    // 4 eps sum |A_ii|
    int exp;                         // the iteration works on A 2^-exp
    int rot[JAC_SWEEPS + 1];         // rot[s]: sweep s rotated something
};

// Rotation [[c, sigma], [-conj(sigma), c]] of columns (p, q).
struct JacRot {
    double c, sr, si;
    bool on;
};

// 1 / sqrt(x) to rounding: the hardware estimate and one third-order step
__device__ inline double jac_rsqrt(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}

// Rotation that diagonalises [[a, b], [conj(b), d]], skipped as in
// k_herm_jacobi; the smaller of the two angles.  With r = sqrt((d - a)^2 / 4 +
// |b|^2), w = r + |d - a| / 2: c = w / sqrt(2 r w), sigma = +-b / sqrt(2 r w).
__device__ inline JacRot jac_rotation(double a, double d, double br, double bi, double floor_, double tol) {
    JacRot r{1.0, 0.0, 0.0, false};
    const double h = br * br + bi * bi;
    if (h > floor_ * floor_ && h > tol * tol * fabs(a * d) && h > 1e-290) {
        const double g = 0.5 * (d - a), x = fma(g, g, h);
        const double rr = x * jac_rsqrt(x), w = rr + fabs(g);
        const double z = jac_rsqrt(2.0 * rr * w), zs = g >= 0.0 ? z : -z;
        r.c = w * z;
        r.sr = br * zs;
        r.si = bi * zs;
        r.on = true;
    }
    return r;
}

// The index pair (p, q) that pair i rotates, round after round: the JB pairs
// between the two blocks, or (ALL) the W / 2 pairs of the round-robin over the
// whole width.
template <int W, bool ALL>
struct JacIndex {
    static_assert(ALL || W == JW, "two blocks");
    int x, y;
    __device__ explicit JacIndex(int i) : x(i), y(ALL ? W - 1 - i : JB + i) {}
    __device__ int p() const { return ALL ? min(x, y) : x; }
    __device__ int q() const { return ALL ? max(x, y) : y; }
    __device__ void next() {
        if (ALL) {   // slot 0 stays, the others go round 1 .. W - 1
            x = x == 0 ? 0 : x == W - 1 ? 1 : x + 1;
            y = y == W - 1 ? 1 : y + 1;
        } else {
            y = JB + ((y + 1) & (JB - 1));
        }
    }
};

// LDS matrix, re and im, [row][column]: with an odd stride of doubles sixteen
// lanes along a row or along a column meet distinct banks.
template <int W>
using JacMatW = double[2][W][W + 1];
typedef JacMatW<JW> JacMat;

// Threads of jac_rotate_pair: whole waves for the matrix, the others for u.
constexpr int jac_mt(int w) { return (w * w / 4 + 63) / 64 * 64; }
constexpr int jac_threads(int w) { return 2 * jac_mt(w) < 256 ? 256 : 2 * jac_mt(w) < 1024 ? 2 * jac_mt(w) : 1024; }

// One pass of rotations over the pair matrix m[cur], its product gathered in
// u; returns the buffer that holds the matrix on exit; rot is set if anything
// rotated.  The first jac_mt(W) threads rotate the matrix, thread (i, j) the 2 x 2
// block of pairs i and j; reading one buffer and writing the other, a round needs
// one barrier.  The others apply the rotations of the round before to u.
template <int W, bool ALL>
__device__ inline int jac_rotate_pair(JacMatW<W> (&m)[2], JacMatW<W>& u, JacRot (&rots)[2][W / 2], int cur,
                                      double floor_, double tol, int* rot) {
    constexpr int P = W / 2, MT = jac_mt(W), UT = jac_threads(W) - MT, ITEMS = (W * P + UT - 1) / UT;
    constexpr int rounds = ALL ? W - 1 : JB;
    const int tid = threadIdx.x, i = tid % P, j = tid / P;
    // p <- c p - conj(sigma) q, q <- sigma p + c q on a pair of columns; on rows
    // sigma and its conjugate change places
    auto rotate = [](double c, double sr, double si, double& pr, double& pm, double& qr, double& qm) {
        const double tr = c * pr - sr * qr - si * qm, tm = c * pm - sr * qm + si * qr;
        qr = c * qr + sr * pr - si * pm;
        qm = c * qm + sr * pm + si * pr;
        pr = tr;
        pm = tm;
    };
    // matrix: pair i's rotation is worked out by every lane that belongs to it,
    // pair j's comes from one of them (a wave holds more than P consecutive tids)
    const int from = (j + P - (tid & ~63) % P) % P;
    JacIndex<W, ALL> ii(i), jj(j);
    // u: item a is row[a] of the columns of pair[a]
    int row[ITEMS], pair[ITEMS], px[ITEMS], py[ITEMS];
#pragma unroll
    for (int a = 0; a < ITEMS; ++a) {
        const int e = max(tid - MT, 0) + UT * a;
        row[a] = e % W;
        pair[a] = e / W;
        const JacIndex<W, ALL> first(pair[a]);
        px[a] = first.x;
        py[a] = first.y;
    }
    for (int t = 0; t <= rounds; ++t) {
        if (tid >= MT) {
#pragma unroll
            for (int a = 0; a < ITEMS; ++a)
                if (t > 0 && (W * P % UT == 0 || pair[a] < P)) {
                    JacIndex<W, ALL> pq(0);
                    pq.x = px[a];
                    pq.y = py[a];
                    const int pj = pq.p(), qj = pq.q(), r = row[a];
                    pq.next();
                    px[a] = pq.x;
                    py[a] = pq.y;
                    const JacRot rj = rots[(t - 1) & 1][pair[a]];
                    double pr = u[0][r][pj], pm = u[1][r][pj], qr = u[0][r][qj], qm = u[1][r][qj];
                    rotate(rj.c, rj.sr, rj.si, pr, pm, qr, qm);
                    u[0][r][pj] = pr;
                    u[1][r][pj] = pm;
                    u[0][r][qj] = qr;
                    u[1][r][qj] = qm;
                }
        } else if (t < rounds) {
            const JacMatW<W>& M = m[(cur + t) & 1];
            JacMatW<W>& O = m[(cur + t + 1) & 1];
            const int pi = ii.p(), qi = ii.q(), pj = jj.p(), qj = jj.q();
            ii.next();
            jj.next();
            const JacRot ri = jac_rotation(M[0][pi][pi], M[0][qi][qi], M[0][pi][qi], M[1][pi][qi], floor_, tol);
            const double cj = __shfl(ri.c, from, 64), srj = __shfl(ri.sr, from, 64), sij = __shfl(ri.si, from, 64);
            if (P * P == MT || j < P) {
                double xr[2][2] = {{M[0][pi][pj], M[0][pi][qj]}, {M[0][qi][pj], M[0][qi][qj]}};
                double xi[2][2] = {{M[1][pi][pj], M[1][pi][qj]}, {M[1][qi][pj], M[1][qi][qj]}};
#pragma unroll
                for (int b = 0; b < 2; ++b) rotate(ri.c, ri.sr, -ri.si, xr[0][b], xi[0][b], xr[1][b], xi[1][b]);
#pragma unroll
                for (int a = 0; a < 2; ++a) rotate(cj, srj, sij, xr[a][0], xi[a][0], xr[a][1], xi[a][1]);
                O[0][pi][pj] = xr[0][0];
                O[0][pi][qj] = xr[0][1];
                O[0][qi][pj] = xr[1][0];
                O[0][qi][qj] = xr[1][1];
                O[1][pi][pj] = xi[0][0];
                O[1][pi][qj] = xi[0][1];
                O[1][qi][pj] = xi[1][0];
                O[1][qi][qj] = xi[1][1];
                if (j == 0) {
                    rots[t & 1][i] = ri;
                    if (ri.on) *rot = 1;
                }
            }
        }
        __syncthreads();
    }
    return (cur + rounds) & 1;
}

// global index of local index l < JW of pair X in round r over nb blocks
__device__ inline int jac_index(int X, int l, int r, int nb) {
    auto player = [&](int slot) { return slot == 0 ? 0 : 1 + (slot - 1 + r) % (nb - 1); };
    const int x = player(X), y = player(nb - 1 - X);
    return JB * (l < JB ? min(x, y) : max(x, y)) + l % JB;
}

typedef double jf64x4 __attribute__((ext_vector_type(4)));

// C = op(A) B for JW x JW complex matrices in LDS on the FP64 matrix cores (op:
// conjugate transpose when HA): wave w < 8 forms plane w / 4 (re, im) of
// output tile w % 4.  Output lane layout of the 16x16x4 FP64 operation with B
// fed first: lane l, register r holds C[m0 + l % 16][n0 + l / 16 + 4 r].
template <bool HA>
__device__ inline jf64x4 jac_product(const JacMat& A, const JacMat& B) {
    const int w = threadIdx.x / 64, lane = threadIdx.x % 64;
    const int m = 16 * (w & 1) + lane % 16, n = 16 * ((w >> 1) & 1) + lane % 16;
    const bool im = w >= 4;
    jf64x4 acc = {0, 0, 0, 0};
#pragma unroll
    for (int k0 = 0; k0 < JW; k0 += 4) {
        const int k = k0 + lane / 16;
        const double ar = HA ? A[0][k][m] : A[0][m][k], ai = HA ? -A[1][k][m] : A[1][m][k];
        const double br = B[0][k][n], bi = B[1][k][n];
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(br, im ? ai : ar, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(im ? bi : -bi, im ? ar : ai, acc, 0, 0, 0);
    }
    return acc;
}

// Exponent of a matrix of `count` doubles: 2^-exp puts the largest entry into
// [1/2, 1), so that squares of entries neither underflow nor overflow whatever
// its scale (exact but for entries 2^-1022 of the largest); the same in every
// thread.  sh: blockDim / 64 doubles.
__device__ inline int jac_exponent(const double* A, int64_t count, double* sh) {
    double mx = 0.0;
    for (int64_t e = threadIdx.x; e < count; e += blockDim.x) mx = fmax(mx, fabs(A[e]));
    for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o, 64));
    if (threadIdx.x % 64 == 0) sh[threadIdx.x / 64] = mx;
    __syncthreads();
    for (int w = 0; w < (int)(blockDim.x / 64); ++w) mx = fmax(mx, sh[w]);
    __syncthreads();
    int ex = 0;
    if (mx > 0.0 && mx <= 1.7976931348623157e308) (void)frexp(mx, &ex);
    return ex;
}

// ---------------------------------------------------------------------------
// Refinement of the eigenvectors (Ogita and Aishima 2018, one step).  The
// rotations leave V = X (1 + O(n eps / gap)) of the exact eigenvectors X, since
// off-diagonal entries at the rounding level of A are never rotated.  With
// R = 1 - V^H V and S = V^H A V, lambda_i = S_ii / (1 - R_ii) and V <- V (1 + E),
// E_ij = (S_ij + lambda_j R_ij) / (lambda_j - lambda_i), is X to second order:
// E + E^H = R keeps V orthonormal, the first-order rotation between i and j takes
// out S_ij.  Pairs without a gap (|S_ij| + |lambda R_ij| > 1e-8 |lambda_j -
// lambda_i|: the square of such a rotation would be visible) take E_ij = R_ij / 2.
// What S and R hold is the rounding of some thousand rotations, so their own
// products are summed in pairs of doubles.
//   Measured, error of the leading projector (a twelfth of the spectrum, over six
// decades) against extended precision, cyclic Jacobi in one workgroup / the block
// form with V (3 - V^H V) / 2 and a last sweep / this: 144 x 144 1.2e-13 / 9.6e-14
// / 1.5e-16, 200 x 200 1.8e-13 / 3.2e-13 / 2.0e-16; the whole call 4.01 -> 3.85 ms
// (144 x 144), 7.24 -> 6.69 (256 x 256) against the block form before.
// ---------------------------------------------------------------------------
constexpr int ET = 16;   // tile of a refinement product, one output a thread

// s + c += a b, c the rounding errors of s (two-product, two-sum)
__device__ inline void dd_add(double& s, double& c, double a, double b) {
#pragma clang fp contract(off)
    const double p = a * b, e = fma(a, b, -p);
    const double t = s + p, z = t - s;
    const double d = (s - (t - z)) + (p - z);
    s = t;
    c += d + e;
}

// Output (m0 + tid % ET, n0 + tid / ET) of op(A) (B + Blo), n x n planar
// column-major, as high and low parts (re, im) (op: conjugate transpose when HA;
// Blo may be null).
struct DD2 {
    double rh, rl, ih, il;
};
template <bool HA>
__device__ inline DD2 dd_product(const double* A, const double* B, const double* Blo, int n, int m0, int n0) {
    __shared__ double As[2][ET][ET + 1], Bs[4][ET][ET + 1];
    const int x = threadIdx.x % ET, y = threadIdx.x / ET;
    const int64_t nn = (int64_t)n * n;
    double rs = 0, rc = 0, is = 0, ic = 0;
    for (int k0 = 0; k0 < n; k0 += ET) {
        const int ra = HA ? k0 + x : m0 + x, ca = HA ? m0 + y : k0 + y, kb = k0 + x, cb = n0 + y;
        const bool oka = ra < n && ca < n, okb = kb < n && cb < n;
        const int64_t oa = oka ? ra + (int64_t)n * ca : 0, ob = okb ? kb + (int64_t)n * cb : 0;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const double a = oka ? A[p * nn + oa] : 0.0;
            As[p][HA ? x : y][HA ? y : x] = HA && p ? -a : a;
            Bs[p][x][y] = okb ? B[p * nn + ob] : 0.0;
            Bs[2 + p][x][y] = okb && Blo ? Blo[p * nn + ob] : 0.0;
        }
        __syncthreads();
        const int kn = min(ET, n - k0);
#pragma unroll 4
        for (int k = 0; k < kn; ++k) {
            const double ar = As[0][k][x], ai = As[1][k][x], br = Bs[0][k][y], bi = Bs[1][k][y];
            dd_add(rs, rc, ar, br);
            dd_add(rs, rc, -ai, bi);
            dd_add(is, ic, ar, bi);
            dd_add(is, ic, ai, br);
            if (Blo) {
                const double lr = Bs[2][k][y], li = Bs[3][k][y];
                rc += ar * lr - ai * li;
                ic += ar * li + ai * lr;
            }
        }
        __syncthreads();
    }
    DD2 o;
    o.rh = rs + rc;
    o.rl = rc - (o.rh - rs);
    o.ih = is + ic;
    o.il = ic - (o.ih - is);
    return o;
}

// One tile of T + Tlo = A V
__device__ inline void eig_av(const double* A, const double* V, int n, int m0, int n0, double* T, double* Tlo) {
    const DD2 o = dd_product<false>(A, V, nullptr, n, m0, n0);
    const int m = m0 + threadIdx.x % ET, c = n0 + threadIdx.x / ET;
    if (m >= n || c >= n) return;
    const int64_t nn = (int64_t)n * n, e = m + (int64_t)n * c;
    T[e] = o.rh;
    T[nn + e] = o.ih;
    Tlo[e] = o.rl;
    Tlo[nn + e] = o.il;
}

// One tile of S = V^H (T + Tlo) (first), or of R = 1 - V^H V
__device__ inline void eig_sr(const double* V, const double* T, const double* Tlo, int n, bool first, int m0, int n0,
                              double* S, double* R) {
    const DD2 o = dd_product<true>(V, first ? T : V, first ? Tlo : nullptr, n, m0, n0);
    const int m = m0 + threadIdx.x % ET, c = n0 + threadIdx.x / ET;
    if (m >= n || c >= n) return;
    const int64_t nn = (int64_t)n * n, e = m + (int64_t)n * c;
    if (first) {
        S[e] = o.rh;
        S[nn + e] = o.ih;
    } else {
        R[e] = ((m == c ? 1.0 : 0.0) - o.rh) - o.rl;
        R[nn + e] = -o.ih - o.il;
    }
}

// One tile of Vout = V + V E; the first one also w[k], the k-th largest eigenvalue
// times 2^ex, and order[k], its column (ties by index, NaN last).
__device__ inline void eig_update(const double* V, const double* S, const double* R, int n, int ex, int m0, int n0,
                                  double* Vout, double* w, int* order) {
    __shared__ double lam[JAC_NMAX], Vs[2][ET][ET + 1], Es[2][ET][ET + 1];
    const int x = threadIdx.x % ET, y = threadIdx.x / ET;
    const int64_t nn = (int64_t)n * n;
    for (int i = threadIdx.x; i < n; i += ET * ET) lam[i] = S[i + (int64_t)n * i] / (1.0 - R[i + (int64_t)n * i]);
    __syncthreads();
    const int m = m0 + x, c = n0 + y;
    double re = 0, im = 0;
    for (int k0 = 0; k0 < n; k0 += ET) {
        const int kv = k0 + y, ke = k0 + x;
#pragma unroll
        for (int p = 0; p < 2; ++p) Vs[p][y][x] = m < n && kv < n ? V[p * nn + m + (int64_t)n * kv] : 0.0;
        double er = 0, ei = 0;
        if (ke < n && c < n) {
            const int64_t e = ke + (int64_t)n * c, h = c + (int64_t)n * ke;
            // the Hermitian parts: E + E^H = R has to hold to rounding over the gap,
            // whatever A is off Hermitian by
            const double sr = 0.5 * (S[e] + S[h]), si = 0.5 * (S[nn + e] - S[nn + h]);
            const double rr = 0.5 * (R[e] + R[h]), ri = 0.5 * (R[nn + e] - R[nn + h]);
            const double li = lam[ke], lj = lam[c];
            const double gap = lj - li;
            const double num = sqrt(sr * sr + si * si) + fmax(fabs(li), fabs(lj)) * sqrt(rr * rr + ri * ri);
            if (num <= 1e-8 * fabs(gap) && gap != 0.0) {
                er = (sr + lj * rr) / gap;
                ei = (si + lj * ri) / gap;
            } else {
                er = 0.5 * rr;
                ei = 0.5 * ri;
            }
        }
        Es[0][x][y] = er;
        Es[1][x][y] = ei;
        __syncthreads();
        const int kn = min(ET, n - k0);
#pragma unroll 4
        for (int k = 0; k < kn; ++k) {
            const double vr = Vs[0][k][x], vi = Vs[1][k][x], fr = Es[0][k][y], fi = Es[1][k][y];
            re += vr * fr - vi * fi;
            im += vr * fi + vi * fr;
        }
        __syncthreads();
    }
    if (m < n && c < n) {
        const int64_t e = m + (int64_t)n * c;
        Vout[e] = V[e] + re;
        Vout[nn + e] = V[nn + e] + im;
    }
    if (m0 || n0) return;
    auto key = [&](int i) { return lam[i] == lam[i] ? lam[i] : -INFINITY; };
    for (int i = threadIdx.x; i < n; i += ET * ET) {
        const double wi = key(i);
        int rank = 0;
        for (int j = 0; j < n; ++j) {
            const double wj = key(j);
            rank += wj > wi || (wj == wi && j < i) ? 1 : 0;
        }
        order[rank] = i;
        w[rank] = ldexp(lam[i], ex);
    }
}

__global__ __launch_bounds__(ET* ET) void k_eig_av(const double* A, const double* V, int n, double* T, double* Tlo) {
    eig_av(A, V, n, ET * blockIdx.x, ET * blockIdx.y, T, Tlo);
}
__global__ __launch_bounds__(ET* ET) void k_eig_sr(const double* V, const double* T, const double* Tlo, int n,
                                                  double* S, double* R) {
    eig_sr(V, T, Tlo, n, blockIdx.z == 0, ET * blockIdx.x, ET * blockIdx.y, S, R);
}
__global__ __launch_bounds__(ET* ET) void k_eig_update(const double* V, const double* S, const double* R, int n,
                                                      const JacState* js, double* Vout, double* w, int* order) {
    eig_update(V, S, R, n, js->exp, ET * blockIdx.x, ET * blockIdx.y, Vout, w, order);
}
// The whole iteration for n <= W <= JAC_ONE: X and A0 = A 2^-exp; for W <= ET, one
// tile, the refinement too (work: T, Tlo, S, R of 2 n^2 doubles).
template <int W>
__global__ __launch_bounds__(jac_threads(W)) void k_jacobi_one(const double* A, int n, int max_sweeps, double tol,
                                                              double* X, double* A0, double* work, double* V,
                                                              double* w, int* order, JacState* js, StepDev* st) {
    constexpr int NT = jac_threads(W);
    __shared__ JacMatW<W> m[2], u;
    __shared__ JacRot rots[2][W / 2];
    __shared__ double sh[NT / 64 + 1];
    __shared__ int s_rot;
    const int nn = n * n;
    const int ex = jac_exponent(A, 2 * nn, sh);
    double tr = 0.0;
    for (int e = threadIdx.x; e < W * W; e += NT) {
        const int a = e % W, b = e / W;
        const bool ok = a < n && b < n;
        const double re = ok ? ldexp(A[a + n * b], -ex) : 0.0, im = ok ? ldexp(A[nn + a + n * b], -ex) : 0.0;
        m[0][0][a][b] = re;
        m[0][1][a][b] = im;
        u[0][a][b] = a == b ? 1.0 : 0.0;
        u[1][a][b] = 0.0;
        if (a == b) tr += fabs(re);
        if (ok) {
            A0[a + n * b] = re;
            A0[nn + a + n * b] = im;
        }
    }
    if (threadIdx.x == 0) js->exp = ex;
    const double floor_ = 4.0 * 2.220446049250313e-16 * block_sum_all(tr, sh);
    int cur = 0;
    bool settled = false;
    for (int q = 0; q < max_sweeps && !settled; ++q) {
        if (threadIdx.x == 0) s_rot = 0;
        __syncthreads();
        cur = jac_rotate_pair<W, true>(m, u, rots, cur, floor_, tol, &s_rot);
        settled = !s_rot;
        __syncthreads();
    }
    if (threadIdx.x == 0 && !settled) atomicExch(&st->bad, 1);
    for (int e = threadIdx.x; e < W * W; e += NT) {
        const int a = e % W, b = e / W;
        if (a >= n || b >= n) continue;
        X[a + n * b] = u[0][a][b];
        X[nn + a + n * b] = u[1][a][b];
    }
    if constexpr (W <= ET) {
        static_assert(NT == ET * ET, "one output a thread");
        double *T = work, *Tlo = T + 2 * nn, *S = Tlo + 2 * nn, *R = S + 2 * nn;
        __syncthreads();
        eig_av(A0, X, n, 0, 0, T, Tlo);
        __syncthreads();
        eig_sr(X, T, Tlo, n, true, 0, 0, S, R);
        eig_sr(X, T, Tlo, n, false, 0, 0, S, R);
        __syncthreads();
        eig_update(X, S, R, n, ex, 0, 0, V, w, order);
    }
}

// V = 1, A0 = B = A 2^-exp (every block finds the exponent for itself), the skip
// level of the rotations.
__global__ __launch_bounds__(JS_THREADS) void k_jacobi_init(const double* A, int n, double* V, double* A0, double* B,
                                                           JacState* js) {
    __shared__ double sh[JS_THREADS / 64 + 1];
    const int64_t nn = (int64_t)n * n;
    const int ex = jac_exponent(A, 2 * nn, sh);
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < nn; e += (int64_t)gridDim.x * blockDim.x) {
        V[e] = e % n == e / n ? 1.0 : 0.0;
        V[nn + e] = 0.0;
        A0[e] = B[e] = ldexp(A[e], -ex);
        A0[nn + e] = B[nn + e] = ldexp(A[nn + e], -ex);
    }
    if (blockIdx.x) return;
    double tr = 0.0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) tr += fabs(ldexp(A[i + (int64_t)n * i], -ex));
    tr = block_sum_all(tr, sh);
    for (int i = threadIdx.x; i <= JAC_SWEEPS; i += blockDim.x) js->rot[i] = 0;
    if (threadIdx.x == 0) {
        js->floor = 4.0 * 2.220446049250313e-16 * tr;
        js->exp = ex;
    }
}

// Round r of sweep s over nb (even) blocks, workgroup X: the diagonal matrix of
// pair X rotated in place, the product of its rotations to U[X] (planar,
// row-major).
__global__ __launch_bounds__(JS_THREADS) void k_jacobi_solve(double* A, int n, int nb, int r, int sweep, double tol,
                                                            double* U, JacState* js) {
    static_assert(JS_THREADS == jac_threads(JW), "threads of a pair");
    if (sweep > 0 && !js->rot[sweep - 1]) return;
    __shared__ JacMat m[2], u;
    __shared__ JacRot rots[2][JB];
    __shared__ int s_rot;
    const int64_t nn = (int64_t)n * n;
    const int X = blockIdx.x;
    if (threadIdx.x == 0) s_rot = 0;
    for (int e = threadIdx.x; e < JW * JW; e += JS_THREADS) {
        const int a = e % JW, b = e / JW, ga = jac_index(X, a, r, nb), gb = jac_index(X, b, r, nb);
        const bool ok = ga < n && gb < n;
        const int64_t o = ok ? ga + (int64_t)n * gb : 0;
        const double re = A[o], im = A[nn + o];
        m[0][0][a][b] = ok ? re : 0.0;
        m[0][1][a][b] = ok ? im : 0.0;
        u[0][a][b] = a == b ? 1.0 : 0.0;
        u[1][a][b] = 0.0;
    }
    const double floor_ = js->floor;
    __syncthreads();
    const int cur = r == 0 ? jac_rotate_pair<JW, true>(m, u, rots, 0, floor_, tol, &s_rot)
                           : jac_rotate_pair<JW, false>(m, u, rots, 0, floor_, tol, &s_rot);
    if (threadIdx.x == 0 && s_rot) js->rot[sweep] = 1;
    double* Ux = U + (int64_t)X * 2 * JW * JW;
    for (int e = threadIdx.x; e < JW * JW; e += JS_THREADS) {
        const int a = e % JW, b = e / JW, ga = jac_index(X, a, r, nb), gb = jac_index(X, b, r, nb);
        Ux[e] = u[0][e / JW][e % JW];
        Ux[JW * JW + e] = u[1][e / JW][e % JW];
        if (ga >= n || gb >= n) continue;
        A[ga + (int64_t)n * gb] = m[cur][0][a][b];
        A[nn + ga + (int64_t)n * gb] = m[cur][1][a][b];
    }
}

// The rest of the round: np (np - 1) / 2 workgroups for the pairs P < Q, then
// ceil(n / JW) x np for the rows of V.
__global__ __launch_bounds__(JA_THREADS) void k_jacobi_apply(double* A, int n, int nb, double* V, int r, int sweep,
                                                            const double* U, const JacState* js) {
    if (sweep > 0 && !js->rot[sweep - 1]) return;
    __shared__ JacMat x, y, up, uq;
    const int np = nb / 2, npp = np * (np - 1) / 2;
    const int64_t nn = (int64_t)n * n;
    const bool isV = (int)blockIdx.x >= npp;
    int P = 0, Q, rb = 0;
    if (isV) {
        Q = (blockIdx.x - npp) % np;
        rb = (blockIdx.x - npp) / np;
    } else {
        Q = 1;
        P = blockIdx.x;
        while (P >= Q) P -= Q++;
    }
    double* D = isV ? V : A;
    auto row = [&](int l) { return isV ? JW * rb + l : jac_index(P, l, r, nb); };
    for (int e = threadIdx.x; e < JW * JW; e += JA_THREADS) {
        const int a = e % JW, b = e / JW, ga = row(a), gb = jac_index(Q, b, r, nb);
        const bool ok = ga < n && gb < n;
        const int64_t o = ok ? ga + (int64_t)n * gb : 0;
        const double re = D[o], im = D[nn + o];
        x[0][a][b] = ok ? re : 0.0;
        x[1][a][b] = ok ? im : 0.0;
#pragma unroll
        for (int pl = 0; pl < 2; ++pl) {
            uq[pl][e / JW][e % JW] = U[((int64_t)Q * 2 + pl) * JW * JW + e];
            up[pl][e / JW][e % JW] = U[((int64_t)P * 2 + pl) * JW * JW + e];
        }
    }
    __syncthreads();
    const int w = threadIdx.x / 64, lane = threadIdx.x % 64;
    const int om = 16 * (w & 1) + lane % 16, on = 16 * ((w >> 1) & 1) + lane / 16;
    jf64x4 z = jac_product<false>(x, uq);
    if (!isV) {
#pragma unroll
        for (int q = 0; q < 4; ++q) y[w >> 2][om][on + 4 * q] = z[q];
        __syncthreads();
        z = jac_product<true>(up, y);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int ga = row(om), gb = jac_index(Q, on + 4 * q, r, nb);
        if (ga >= n || gb >= n) continue;
        D[(w >= 4 ? nn : 0) + ga + (int64_t)n * gb] = z[q];
        if (!isV) D[(w >= 4 ? nn : 0) + gb + (int64_t)n * ga] = w >= 4 ? -z[q] : z[q];
    }
}

// Diagonalises a Hermitian n x n matrix A (planar complex,
// column-major; overwritten) by the cyclic Jacobi method with the round-robin
// ordering: each of the n' - 1 rounds of a sweep (n' = n rounded up to even,
// the extra index a zero row and column) rotates n' / 2 disjoint index pairs
// at once, all rotations taken from the matrix before the round.  Pair
// (p, q), b = A[p, q] = |b| e^{i phi}: J = diag(1, e^{-i phi}) R with the real
// Jacobi rotation R = [[c, s], [-s, c]] that diagonalises
// [[A_pp, |b|], [|b|, A_qq]] (t = sgn(tau) / (|tau| + sqrt(1 + tau^2)),
// tau = (A_qq - A_pp) / (2 |b|), c = 1 / sqrt(1 + t^2), s = t c), applied as
// A <- J^H A J and V <- V J.  A pair is skipped when
// |b| <= tol sqrt(|A_pp A_qq|) (relative accuracy for positive definite
// matrices) or |b| <= 4 eps sum_i |A_ii| (the rounding level of the matrix,
// which pairs of numerically zero eigenvalues cannot get below); the
// iteration stops after a sweep without a rotation, or after max_sweeps
// (then st->bad is set).  Closes the block form: it finds A and V
// as the rounds left them and goes on only if their last sweep still rotated.
__global__ __launch_bounds__(JAC_THREADS) void k_herm_jacobi(double* A, int n, double* V, int block_sweeps,
                                                             int max_sweeps, double tol, const JacState* js,
                                                             StepDev* st) {
    __shared__ double rc[JAC_NMAX / 2], rs[JAC_NMAX / 2], rer[JAC_NMAX / 2], rei[JAC_NMAX / 2];
    __shared__ int rp[JAC_NMAX / 2], rq[JAC_NMAX / 2];
    __shared__ int s_rot, s_done;
    const int tid = threadIdx.x;
    const int np = n + (n & 1), half = np / 2;
    const int64_t nn = (int64_t)n * n;
    double* Ai = A + nn;
    double* Vi = V + nn;
    // off-diagonal entries at the rounding level of the whole matrix cannot
    // be reduced further: a pair is also left alone below 4 eps sum |A_ii|
    const double abs_floor = js->floor;
    // a sweep without rotation ended the rounds
    bool converged = false;
    for (int k = 0; k < block_sweeps; ++k) converged = converged || js->rot[k] == 0;
    if (tid == 0) s_done = converged;
    __syncthreads();
    for (int sweep = 0; sweep < max_sweeps && !converged; ++sweep) {
        if (tid == 0) s_rot = 0;
        __syncthreads();
        for (int r = 0; r < np - 1; ++r) {
            if (tid < half) {
                // circle method: slot 0 holds index 0, slots 1.. rotate
                auto player = [&](int slot) { return slot == 0 ? 0 : 1 + (slot - 1 + r) % (np - 1); };
                int p = player(tid), q = player(np - 1 - tid);
                if (p > q) {
                    const int t = p;
                    p = q;
                    q = t;
                }
                double c = 1.0, sn = 0.0, er = 1.0, ei = 0.0;
                if (q < n) {
                    const double a = A[p + (int64_t)n * p], d = A[q + (int64_t)n * q];
                    const double br = A[p + (int64_t)n * q], bi = Ai[p + (int64_t)n * q];
                    const double ab = sqrt(br * br + bi * bi);
                    if (ab > abs_floor && ab > tol * sqrt(fabs(a * d))) {
                        const double tau = (d - a) / (2.0 * ab);
                        const double t = (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
                        c = 1.0 / sqrt(1.0 + t * t);
                        sn = t * c;
                        er = br / ab;   // e^{-i phi} = conj(b) / |b|
                        ei = -bi / ab;
                        s_rot = 1;
                    }
                }
                rc[tid] = c;
                rs[tid] = sn;
                rer[tid] = er;
                rei[tid] = ei;
                rp[tid] = p;
                rq[tid] = q;
            }
            __syncthreads();
            // A <- J^H A J, one 2 x 2 block (pair P rows, pair Q columns) per item
            for (int e = tid; e < half * half; e += JAC_THREADS) {
                const int P = e % half, Q = e / half;
                const int p0 = rp[P], q0 = rq[P], p1 = rp[Q], q1 = rq[Q];
                const bool rowq = q0 < n, colq = q1 < n;
                // block entries x[row][col], rows (p0, q0), columns (p1, q1)
                double xr[2][2], xi[2][2];
                const int rows[2] = {p0, q0}, cols[2] = {p1, q1};
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int b = 0; b < 2; ++b) {
                        const bool ok = (a == 0 || rowq) && (b == 0 || colq);
                        const int64_t o = rows[a] + (int64_t)n * cols[b];
                        xr[a][b] = ok ? A[o] : 0.0;
                        xi[a][b] = ok ? Ai[o] : 0.0;
                    }
                // rows: r_p = c x_p - s conj(e) x_q,  r_q = s x_p + c conj(e) x_q
                {
                    const double c = rc[P], sn = rs[P], er = rer[P], ei = -rei[P];   // conj(e)
#pragma unroll
                    for (int b = 0; b < 2; ++b) {
                        const double qr = er * xr[1][b] - ei * xi[1][b], qi = er * xi[1][b] + ei * xr[1][b];
                        const double pr = xr[0][b], pi = xi[0][b];
                        xr[0][b] = c * pr - sn * qr;
                        xi[0][b] = c * pi - sn * qi;
                        xr[1][b] = sn * pr + c * qr;
                        xi[1][b] = sn * pi + c * qi;
                    }
                }
                // columns: k_p = c x_p - s e x_q,  k_q = s x_p + c e x_q
                {
                    const double c = rc[Q], sn = rs[Q], er = rer[Q], ei = rei[Q];
#pragma unroll
                    for (int a = 0; a < 2; ++a) {
                        const double qr = er * xr[a][1] - ei * xi[a][1], qi = er * xi[a][1] + ei * xr[a][1];
                        const double pr = xr[a][0], pi = xi[a][0];
                        xr[a][0] = c * pr - sn * qr;
                        xi[a][0] = c * pi - sn * qi;
                        xr[a][1] = sn * pr + c * qr;
                        xi[a][1] = sn * pi + c * qi;
                    }
                }
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int b = 0; b < 2; ++b) {
                        if (!((a == 0 || rowq) && (b == 0 || colq))) continue;
                        const int64_t o = rows[a] + (int64_t)n * cols[b];
                        A[o] = xr[a][b];
                        Ai[o] = xi[a][b];
                    }
            }
            // V <- V J on the columns of every pair
            for (int e = tid; e < n * half; e += JAC_THREADS) {
                const int i = e % n, Q = e / n;
                const int p1 = rp[Q], q1 = rq[Q];
                if (q1 >= n) continue;
                const double c = rc[Q], sn = rs[Q], er = rer[Q], ei = rei[Q];
                const int64_t op = i + (int64_t)n * p1, oq = i + (int64_t)n * q1;
                const double pr = V[op], pi = Vi[op], xr = V[oq], xi = Vi[oq];
                const double qr = er * xr - ei * xi, qi = er * xi + ei * xr;
                V[op] = c * pr - sn * qr;
                Vi[op] = c * pi - sn * qi;
                V[oq] = sn * pr + c * qr;
                Vi[oq] = sn * pi + c * qi;
            }
            __syncthreads();
        }
        const int rotated = s_rot;
        __syncthreads();   // every thread has read s_rot before it is reset
        if (!rotated) {
            if (tid == 0) s_done = 1;
            break;
        }
    }
    __syncthreads();
    if (tid == 0 && !s_done) atomicExch(&st->bad, 1);
}

}  // namespace

namespace {
// dst[c dc + s ds + p dp] = src[c sc + s ss + p sp] (conjugated if conj), for
// c < K, s < S, p < P; planar complex with the given plane distances.
__global__ void k_copy3(const double* src, int64_t src_plane, int64_t sc, int64_t ss, int64_t sp, double* dst,
                        int64_t dst_plane, int64_t dc, int64_t ds, int64_t dp, int K, int S, int P, int conj) {
    const int64_t total = (int64_t)K * S * P;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        const int c = (int)(e % K);
        const int64_t r = e / K;
        const int sidx = (int)(r % S), pidx = (int)(r / S);
        const int64_t i = c * sc + sidx * ss + pidx * sp, o = c * dc + sidx * ds + pidx * dp;
        dst[o] = src[i];
        dst[o + dst_plane] = conj ? -src[i + src_plane] : src[i + src_plane];
    }
}

// out[:, c] = V[:, order[c]] for c < k (n x n planar V, n x k planar out)
__global__ void k_gather_cols(const double* V, int n, const int* order, int k, double* out) {
    const int64_t total = (int64_t)n * k, nn = (int64_t)n * n, nk = (int64_t)n * k;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        const int i = (int)(e % n), c = (int)(e / n);
        const int64_t src = i + (int64_t)n * order[c];
        out[e] = V[src];
        out[e + nk] = V[src + nn];
    }
}

// The kept weight of a truncated split, from the descending eigenvalues w
// of its Gram matrix: kept = w_0 + .. + w_{k-1}, total = the sum of all n.
// Scales the centre tensor x (count complex entries) by sqrt(total / kept),
// restoring the norm of the untruncated tensor, and folds the discarded
// weight 1 - kept / total into the step's maximum.
__global__ void k_split_finish(const double* w, int n, int k, double* x, int64_t count, StepDev* st) {
    __shared__ double sh[8];
    double kept = 0, total = 0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        total += w[i];
        if (i < k) kept += w[i];
    }
    kept = block_sum_all(kept, sh);
    total = block_sum_all(total, sh);
    const double f = kept > 0.0 ? sqrt(total / kept) : 1.0;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < count; e += (int64_t)gridDim.x * blockDim.x) {
        x[e] *= f;
        x[e + count] *= f;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        double disc = total > 0.0 ? 1.0 - kept / total : 0.0;
        if (disc < 0.0) disc = 0.0;
        if (!(kept > 0.0) || !(disc == disc)) atomicExch(&st->bad, 1);
        atomicMax(&st->max_disc_bits, (unsigned long long)__double_as_longlong(disc));
    }
}
}  // namespace

void copy3(const double* src, int64_t src_plane, int64_t sc, int64_t ss, int64_t sp, double* dst, int64_t dst_plane,
           int64_t dc, int64_t ds, int64_t dp, int K, int S, int P, bool conj, hipStream_t s) {
    if (g_dry_run) return;
    const int64_t total = (int64_t)K * S * P;
    hipLaunchKernelGGL(k_copy3, dim3(grid_for(total)), dim3(256), 0, s, src, src_plane, sc, ss, sp, dst, dst_plane, dc,
                       ds, dp, K, S, P, conj ? 1 : 0);
}

void gather_cols(const double* V, int n, const int* order, int k, double* out, hipStream_t s) {
    if (g_dry_run) return;
    hipLaunchKernelGGL(k_gather_cols, dim3(grid_for((int64_t)n * k)), dim3(256), 0, s, V, n, order, k, out);
}

void split_finish(const double* w, int n, int k, double* x, int64_t count, StepDev* st, hipStream_t s) {
    if (g_dry_run) return;
    hipLaunchKernelGGL(k_split_finish, dim3(grid_for(count)), dim3(256), 0, s, w, n, k, x, count, st);
}

int64_t herm_eig_work(int n) {
    const int64_t np = (n + JW - 1) / JW;
    return 6 * 2 * (int64_t)n * n + np * 2 * JW * JW + (int64_t)((sizeof(JacState) + 7) / 8);
}

void herm_eig(const double* A, int n, double* V, double* w, int* order, double* work, StepDev* st, hipStream_t s) {
    if (g_dry_run) return;
    constexpr double TOL = 1e-15;
    const int64_t n2 = 2 * (int64_t)n * n;
    double *A0 = work, *X = A0 + n2, *T = X + n2, *Tlo = T + n2, *S = Tlo + n2, *R = S + n2, *U = R + n2;
    double* B = S;   // the rotated matrix, until S takes its place
    const int np = (n + JW - 1) / JW, nb = 2 * np;
    JacState* js = (JacState*)(U + (int64_t)np * 2 * JW * JW);
#define TTN_ONE(W)                                                                                               \
    hipLaunchKernelGGL(k_jacobi_one<W>, dim3(1), dim3(jac_threads(W)), 0, s, A, n, 60, TOL, X, A0, T, V, w,  \
                       order, js, st)
    if (n <= 2)
        TTN_ONE(2);
    else if (n <= 4)
        TTN_ONE(4);
    else if (n <= 8)
        TTN_ONE(8);
    else if (n <= 16)
        TTN_ONE(16);
    else if (n <= 24)
        TTN_ONE(24);
    else if (n <= 32)
        TTN_ONE(32);
    else if (n <= 40)
        TTN_ONE(40);
    else if (n <= JAC_ONE)
        TTN_ONE(48);
    else {
        hipLaunchKernelGGL(k_jacobi_init, dim3((n * n + 1023) / 1024), dim3(JS_THREADS), 0, s, A, n, X, A0, B, js);
        for (int sweep = 0; sweep < JAC_SWEEPS; ++sweep)
            for (int r = 0; r < nb - 1; ++r) {
                hipLaunchKernelGGL(k_jacobi_solve, dim3(np), dim3(JS_THREADS), 0, s, B, n, nb, r, sweep, TOL, U, js);
                hipLaunchKernelGGL(k_jacobi_apply, dim3(np * (np - 1) / 2 + np * np), dim3(JA_THREADS), 0, s, B, n, nb,
                                   X, r, sweep, (const double*)U, (const JacState*)js);
            }
        hipLaunchKernelGGL(k_herm_jacobi, dim3(1), dim3(JAC_THREADS), 0, s, B, n, X, JAC_SWEEPS, 60, TOL,
                           (const JacState*)js, st);
    }
#undef TTN_ONE
    if (n <= ET) return;
    const int t = (n + ET - 1) / ET;
    hipLaunchKernelGGL(k_eig_av, dim3(t, t), dim3(ET * ET), 0, s, (const double*)A0, (const double*)X, n, T, Tlo);
    hipLaunchKernelGGL(k_eig_sr, dim3(t, t, 2), dim3(ET * ET), 0, s, (const double*)X, (const double*)T,
                       (const double*)Tlo, n, S, R);
    hipLaunchKernelGGL(k_eig_update, dim3(t, t), dim3(ET * ET), 0, s, (const double*)X, (const double*)S,
                       (const double*)R, n, (const JacState*)js, V, w, order);
}

// ---------------------------------------------------------------------------
// leaf operator blocks and product-state contractions
// ---------------------------------------------------------------------------
namespace {
__global__ void k_contract_node_vec(const double* T, int DL, int DR, int DP, const double* a,
                                    const double* b, double* out) {
    __shared__ double sh[16];
    const int p = blockIdx.x;
    const int64_t n = (int64_t)DL * DR * DP;
    const int64_t LR = (int64_t)DL * DR;
    double re = 0, im = 0;
    for (int64_t e = threadIdx.x; e < LR; e += blockDim.x) {
        const int l = (int)(e % DL), r = (int)(e / DL);
        const double ar = a[l], ai = a[l + DL], br = b[r], bi = b[r + DR];
        const double abr = ar * br - ai * bi, abi = ar * bi + ai * br;
        const double tr = T[e + LR * p], ti = T[n + e + LR * p];
        re += abr * tr - abi * ti;
        im += abr * ti + abi * tr;
    }
    const double sr = block_sum(re, sh);
    const double si = block_sum(im, sh);
    if (threadIdx.x == 0) {
        out[p] = sr;
        out[p + DP] = si;
    }
}
}  // namespace

void contract_node_vec(const double* T, int DL, int DR, int DP, const double* a, const double* b,
                       double* out, hipStream_t s) {
    if (g_dry_run) return;
    hipLaunchKernelGGL(k_contract_node_vec, dim3(DP), dim3(256), 0, s, T, DL, DR, DP, a, b, out);
}

}  // namespace ttn
