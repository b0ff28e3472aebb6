// Complex contraction (GEMM) kernels of the TDVP library for gfx950: the
// LDS-tiled MFMA kernel, the wave-sliced kernel of short launches, the kernel
// of FP32 operands split into bf16 pieces and the split-K reduction, with the
// host-side dispatch cgemm().
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstdio>
#include <initializer_list>

#include "lanes.h"
#include "ttn_internal.h"

namespace ttn {

namespace {

// Sum of the split-K partials into C (alpha, beta applied).  G threads share
// an element (G a power of two dividing 256): thread group q sums splits q,
// q + G, ... with four loads in flight, and the G group sums meet in LDS in a
// fixed order, so the result does not depend on timing.  Blocks walk
// (batch, chunk of 256 / G elements) pairs; element indices are 32-bit
// (the host checks M N < 2^31).
template <typename R>
__global__ __launch_bounds__(256) void k_splitk_reduce(Gemm<R> g, int splits, const R* partial, int G) {
    if (g.skip && *g.skip) return;
    __shared__ R sre[256], sim[256];
    const int MN = g.M * g.N;
    const int nbatch = g.B1 * g.B2;
    const int epb = 256 / G;
    const int el = threadIdx.x % epb, grp = threadIdx.x / epb;
    const int chunks = (MN + epb - 1) / epb;
    const int64_t sstride = (int64_t)nbatch * 2 * MN;
    const bool contig = g.scm == 1 && g.scn == g.M;
    for (int64_t blk = blockIdx.x; blk < (int64_t)chunks * nbatch; blk += gridDim.x) {
        const int b = (int)(blk / chunks);
        const int mn = (int)(blk % chunks) * epb + el;
        R re = 0, im = 0;
        if (mn < MN) {
            const R* P = partial + (int64_t)b * 2 * MN + mn;
            R r4[4] = {0, 0, 0, 0}, i4[4] = {0, 0, 0, 0};
            int sp = grp;
            for (; sp + 3 * G < splits; sp += 4 * G) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    r4[u] += P[(int64_t)(sp + u * G) * sstride];
                    i4[u] += P[(int64_t)(sp + u * G) * sstride + MN];
                }
            }
            for (; sp < splits; sp += G) {
                r4[0] += P[(int64_t)sp * sstride];
                i4[0] += P[(int64_t)sp * sstride + MN];
            }
            re = (r4[0] + r4[1]) + (r4[2] + r4[3]);
            im = (i4[0] + i4[1]) + (i4[2] + i4[3]);
        }
        if (G > 1) {
            sre[threadIdx.x] = re;
            sim[threadIdx.x] = im;
            __syncthreads();
            if (grp == 0)
                for (int q = 1; q < G; ++q) {
                    re += sre[q * epb + el];
                    im += sim[q * epb + el];
                }
            __syncthreads();
        }
        if (grp == 0 && mn < MN) {
            const int b1 = b % g.B1, b2 = b / g.B1;
            R* C = g.C + b1 * g.scb1 + b2 * g.scb2;
            const int64_t off = contig ? (int64_t)mn : (int64_t)(mn % g.M) * g.scm + (int64_t)(mn / g.M) * g.scn;
            re *= g.alpha;
            im *= g.alpha;
            if (g.beta) {
                re += C[off];
                im += C[off + g.c_plane];
            }
            C[off] = re;
            C[off + g.c_plane] = im;
        }
    }
}

// k_splitk_reduce for a contiguous, 16-byte aligned output with few splits:
// each thread sums one 16-byte vector of W consecutive elements of every
// split (in split order, as the scalar kernel does with one thread per
// element) and stores it whole.
template <typename R>
__global__ __launch_bounds__(256) void k_splitk_reduce_vec(Gemm<R> g, int splits, const R* partial) {
    if (g.skip && *g.skip) return;
    constexpr int W = 16 / sizeof(R);
    typedef R V __attribute__((ext_vector_type(W)));
    const int MN = g.M * g.N, nbatch = g.B1 * g.B2;
    const int nv = MN / W;
    const int64_t sstride = (int64_t)nbatch * 2 * MN;
    const int total = nv * nbatch;
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < total; e += gridDim.x * blockDim.x) {
        const int b = e / nv, q = e - b * nv;
        const R* P = partial + (int64_t)b * 2 * MN + (int64_t)q * W;
        V re = *(const V*)P, im = *(const V*)(P + MN);
        for (int sp = 1; sp < splits; ++sp) {
            re += *(const V*)(P + sp * sstride);
            im += *(const V*)(P + sp * sstride + MN);
        }
        const int b1 = b % g.B1, b2 = b / g.B1;
        R* C = g.C + b1 * g.scb1 + b2 * g.scb2 + (int64_t)q * W;
        re *= g.alpha;
        im *= g.alpha;
        if (g.beta) {
            re += *(const V*)C;
            im += *(const V*)(C + g.c_plane);
        }
        *(V*)C = re;
        *(V*)(C + g.c_plane) = im;
    }
}

// Launch of the split-K reduction: the vector kernel for contiguous aligned
// outputs and fewer than four splits, else k_splitk_reduce with up to eight
// threads per element when the splits are many and the elements few.
template <typename R>
void splitk_reduce(const Gemm<R>& g, int splits, const R* partial, hipStream_t s) {
    const int64_t MN = (int64_t)g.M * g.N, nbatch = (int64_t)g.B1 * g.B2;
    constexpr int W = 16 / sizeof(R);
    const bool contig = g.scm == 1 && g.scn == g.M;
    if (splits < 4 && contig && MN % W == 0 && MN * nbatch / W < (1LL << 31) && (uintptr_t)g.C % 16 == 0 &&
        (uintptr_t)partial % 16 == 0 && g.c_plane % W == 0 && g.scb1 % W == 0 && g.scb2 % W == 0) {
        const int nb = (int)std::min<int64_t>((MN * nbatch / W + 255) / 256, 8192);
        hipLaunchKernelGGL((k_splitk_reduce_vec<R>), dim3(nb), dim3(256), 0, s, g, splits, partial);
        return;
    }
    int G = 1;
    while (G < 8 && splits >= 8 * 2 * G && MN * nbatch * 2 * G <= 256LL * 1024) G *= 2;
    const int64_t blocks = (MN + 256 / G - 1) / (256 / G) * nbatch;
    const int nb = (int)std::min<int64_t>(blocks, 8192);
    hipLaunchKernelGGL((k_splitk_reduce<R>), dim3(nb), dim3(256), 0, s, g, splits, partial, G);
}

// Consecutive workgroups go to the eight XCDs in turn, each with an L2 of its
// own: block b of n works on tile xcd_order(b, n), which gives every XCD one
// contiguous range of tiles (each of 0 .. n - 1 once).
__device__ inline unsigned xcd_order(unsigned b, unsigned n) {
    const unsigned x = b % 8, q = n / 8, r = n % 8;
    return x * q + min(x, r) + b / 8;
}

// ---------------------------------------------------------------------------
// MFMA contraction kernel (gfx950).  Complex C = A B with three real
// products per complex product (Gauss): P1 = Ar Br, P2 = Ai Bi,
// P3 = (Ar + Ai)(Br + Bi), then Re C = P1 - P2 and Im C = P3 - P1 - P2 -- a
// quarter fewer matrix-core operations than the four-product form, for a
// third accumulator per output tile.  The matrix-core operands are fed
// transposed (B^T as the first, A^T as the second) so that the output lanes
// of each 16x16x4 tile run along m, the contiguous index of C.  Tiles of A
// (BM x BK) and B (BK x BN) are staged through double-buffered LDS; the next
// k-tile is fetched into registers while the current one is multiplied.  A
// k-tile never crosses a boundary of the outer contraction index
// (Kin % BK == 0).  The block holds WGM x WGN waves of (BM/WGM) x (BN/WGN)
// outputs each.
// ---------------------------------------------------------------------------
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

template <typename R>
struct MfmaT;
template <>
struct MfmaT<float> {
    typedef f32x4 acc_t;
    static __device__ inline acc_t mfma(float a, float b, acc_t c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    // row of register r of lane l inside the 16x16 output tile
    static __device__ inline int row(int l, int r) { return 4 * (l / 16) + r; }
    static constexpr int PAD = 16;
};
template <>
struct MfmaT<double> {
    typedef f64x4 acc_t;
    static __device__ inline acc_t mfma(double a, double b, acc_t c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ inline int row(int l, int r) { return (l / 16) + 4 * r; }
    static constexpr int PAD = 8;
};

// RAG: any inner extent and any strides.  The contraction index is walked
// flattened over (k_in, k_out), each element stepping its own address, loads
// past K give zero, and the complex product takes four real products (no
// Re + Im sums), as accurate as a plain FMA loop.
//   WGK > 1: the block is WGK groups of WGM x WGN waves on the same tile; group
// q takes every WGK-th k-tile from tile q, through LDS buffers of its own,
// and the groups' sums meet in LDS once, in group order.
//   FUSE (sampling, FP64):
// MFMA_OUTER: B is an outer product, formed as its tiles are staged:
// B[k, n] = B1[k_in, n] x.f[k_out, n] (B1 through g's own strides; k_out strides
// of 1 in f).
// MFMA_NORMS: also x.norms[n][tm] = sum over the rows m of tile row tm of
// |C[m, n]|^2 (one split, alpha = 1, beta = 0).
constexpr int MFMA_PLAIN = 0, MFMA_OUTER = 1, MFMA_NORMS = 2;
template <typename R>
struct MfmaExtra {
    const R* f = nullptr;
    int64_t f_plane = 0, sfn = 0;
    R* norms = nullptr;
};
template <typename R, int BM, int BN, int WGM, int WGN, int WGK, int MINB, int BK, bool AK, bool BKF,
          bool RAG = false, int FUSE = MFMA_PLAIN>
__global__ __launch_bounds__(64 * WGM * WGN * WGK, MINB) void k_cgemm_mfma(Gemm<R> g, int tilesM, int tilesN,
                                                                          int splits, int kchunk, R* partial,
                                                                          MfmaExtra<R> x) {
    if (g.skip && *g.skip) return;
    constexpr int NT = 64 * WGM * WGN;   // threads of a group
    static_assert(WGK == 1 || !RAG, "K groups are for the aligned form");
    constexpr int WM = BM / WGM, WN = BN / WGN;
    constexpr int TI = WM / 16, TJ = WN / 16;
    static_assert(TI >= 1 && TJ >= 1, "wave tile below 16 x 16");
    constexpr int PAD = MfmaT<R>::PAD;
    constexpr int QA = BM * BK / NT, QB = BN * BK / NT;
    static_assert(QA >= 1 && QB >= 1, "tile smaller than the block");
    typedef typename MfmaT<R>::acc_t acc_t;
    // LDS tiles [buffer][plane][row][col]: an operand whose global layout is
    // contiguous along k is staged k-contiguous with a row stride of BK + 1, so
    // that both the coalesced stash and the MFMA fragment reads hit distinct
    // banks; the others are staged [k][index] with a pad.
    constexpr int KS = BK + 1;
    constexpr int AR = AK ? BM : BK, AC = AK ? KS : BM + PAD;
    constexpr int BR = BKF ? BN : BK, BC = BKF ? KS : BN + PAD;
    constexpr int ASZ = 4 * AR * AC, BSZ = 4 * BR * BC;
    static_assert(WGK == 1 || WGK * (ASZ + BSZ) >= 2 * WGK * 4 * TI * TJ * NT, "sums of the groups in LDS");
    __shared__ R lds[WGK * (ASZ + BSZ)];
    const int kg = WGK == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / NT);
    R(*As)[2][AR][AC] = reinterpret_cast<R(*)[2][AR][AC]>(lds + kg * ASZ);
    R(*Bs)[2][BR][BC] = reinterpret_cast<R(*)[2][BR][BC]>(lds + WGK * ASZ + kg * BSZ);
    int64_t bid = xcd_order(blockIdx.x, gridDim.x);
    const int tm = bid % tilesM;
    bid /= tilesM;
    const int tn = bid % tilesN;
    bid /= tilesN;
    const int sp = bid % splits;
    bid /= splits;
    const int b = (int)bid;
    const int b1 = b % g.B1, b2 = b / g.B1;
    const int m0 = tm * BM, n0 = tn * BN;
    const R* A = g.A + b1 * g.sab1 + b2 * g.sab2 + (int64_t)m0 * g.sam;
    const R* B = g.B + b1 * g.sbb1 + b2 * g.sbb2 + (int64_t)n0 * g.sbn;
    const int K = g.Kin * g.Kout;
    const int ke = min(K, (sp + 1) * kchunk);
    const int kb = sp * kchunk + kg * BK;
    const int tid = WGK == 1 ? threadIdx.x : threadIdx.x % NT, lane = tid % 64, wave = tid / 64;
    const int wm0 = (wave % WGM) * WM, wn0 = (wave / WGM) * WN;
    const R sa = g.conjA ? R(-1) : R(1), sb = g.conjB ? R(-1) : R(1);
    const int mlim = g.M - m0, nlim = g.N - n0;

    // rows past the edge read row 0: masked to zero, or (RAG) left in outputs
    // that are not stored
    int offA[QA], offB[QB];
    R mA[QA], mB[QB];
    // RAG: address of every element's k, its inner index, and the step from the
    // end of one outer index to the next
    const R *ptrA[QA], *ptrB[QB];
    int kinA[QA], kinB[QB];
    const int64_t wrapA = g.sako - g.Kin * g.sak, wrapB = g.sbko - g.Kin * g.sbk;
#pragma unroll
    for (int q = 0; q < QA; ++q) {
        const int e = tid + NT * q;
        const int mm = AK ? e / BK : e % BM, kk = AK ? e % BK : e / BM;
        const bool ok = mm < mlim;
        mA[q] = ok ? R(1) : R(0);
        if constexpr (RAG) {
            const int kout = (kb + kk) / g.Kin;
            kinA[q] = (kb + kk) - kout * g.Kin;
            ptrA[q] = A + (ok ? mm : 0) * g.sam + kinA[q] * g.sak + kout * g.sako;
        } else
            offA[q] = (ok ? mm : 0) * (int)g.sam + kk * (int)g.sak;
    }
#pragma unroll
    for (int q = 0; q < QB; ++q) {
        const int e = tid + NT * q;
        const int nn = BKF ? e / BK : e % BN, kk = BKF ? e % BK : e / BN;
        const bool ok = nn < nlim;
        mB[q] = ok ? R(1) : R(0);
        if constexpr (RAG) {
            const int kout = (kb + kk) / g.Kin;
            kinB[q] = (kb + kk) - kout * g.Kin;
            ptrB[q] = B + (ok ? nn : 0) * g.sbn + kinB[q] * g.sbk + kout * g.sbko;
        } else
            offB[q] = (ok ? nn : 0) * (int)g.sbn + kk * (int)g.sbk;
    }
    R pa[2][QA], pb[2][QB];
    auto fetch = [&](int k0) {
        if constexpr (RAG) {
            // tiles are fetched in k order; only the last one can pass ke
            const bool full = k0 + BK <= ke;
#pragma unroll
            for (int q = 0; q < QA; ++q) {
                const int e = tid + NT * q;
                const bool ok = full || k0 + (AK ? e % BK : e / BM) < ke;
                const R* src = ok ? ptrA[q] : A;
                const R re = src[0], im = src[g.a_plane];
                pa[0][q] = ok ? re : R(0);
                pa[1][q] = ok ? sa * im : R(0);
                ptrA[q] += BK * g.sak;
                for (kinA[q] += BK; kinA[q] >= g.Kin; kinA[q] -= g.Kin) ptrA[q] += wrapA;
            }
#pragma unroll
            for (int q = 0; q < QB; ++q) {
                const int e = tid + NT * q;
                const bool ok = full || k0 + (BKF ? e % BK : e / BN) < ke;
                const R* src = ok ? ptrB[q] : B;
                const R re = src[0], im = src[g.b_plane];
                pb[0][q] = ok ? re : R(0);
                pb[1][q] = ok ? sb * im : R(0);
                ptrB[q] += BK * g.sbk;
                for (kinB[q] += BK; kinB[q] >= g.Kin; kinB[q] -= g.Kin) ptrB[q] += wrapB;
            }
            return;
        }
        const int kin = k0 % g.Kin, kout = k0 / g.Kin;
        const R* Ab = A + (int64_t)kin * g.sak + (int64_t)kout * g.sako;
        const R* Bb = B + (int64_t)kin * g.sbk + (int64_t)kout * g.sbko;
#pragma unroll
        for (int q = 0; q < QA; ++q) {
            pa[0][q] = mA[q] * Ab[offA[q]];
            pa[1][q] = (sa * mA[q]) * Ab[offA[q] + g.a_plane];
        }
#pragma unroll
        for (int q = 0; q < QB; ++q) {
            if constexpr (FUSE == MFMA_OUTER) {
                const R* f = x.f + kout + x.sfn * (n0 + (mB[q] != R(0) ? (tid + NT * q) / BK : 0));
                const R ar = mB[q] * Bb[offB[q]], ai = mB[q] * Bb[offB[q] + g.b_plane];
                const R fr = f[0], fi = f[x.f_plane];
                pb[0][q] = ar * fr - ai * fi;
                pb[1][q] = ar * fi + ai * fr;
            } else {
                pb[0][q] = mB[q] * Bb[offB[q]];
                pb[1][q] = (sb * mB[q]) * Bb[offB[q] + g.b_plane];
            }
        }
    };
    auto stash = [&](int buf) {
#pragma unroll
        for (int q = 0; q < QA; ++q) {
            const int e = tid + NT * q;
            const int mm = AK ? e / BK : e % BM, kk = AK ? e % BK : e / BM;
            As[buf][0][AK ? mm : kk][AK ? kk : mm] = pa[0][q];
            As[buf][1][AK ? mm : kk][AK ? kk : mm] = pa[1][q];
        }
#pragma unroll
        for (int q = 0; q < QB; ++q) {
            const int e = tid + NT * q;
            const int nn = BKF ? e / BK : e % BN, kk = BKF ? e % BK : e / BN;
            Bs[buf][0][BKF ? nn : kk][BKF ? kk : nn] = pb[0][q];
            Bs[buf][1][BKF ? nn : kk][BKF ? kk : nn] = pb[1][q];
        }
    };
    acc_t c1[TI][TJ], c2[TI][TJ], c3[TI][TJ];
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j) {
            c1[i][j] = acc_t{0, 0, 0, 0};
            c2[i][j] = acc_t{0, 0, 0, 0};
            c3[i][j] = acc_t{0, 0, 0, 0};
        }
    // k-tiles of this group, and of the first one, which has the most: every
    // wave takes part in each round's barrier
    constexpr int KSTEP = BK * WGK;
    const int nt = max(0, (ke - kb + KSTEP - 1) / KSTEP);
    const int rounds = WGK == 1 ? nt : (ke - sp * kchunk + KSTEP - 1) / KSTEP;
    if (nt > 0) {
        fetch(kb);
        stash(0);
        if (nt > 1) fetch(kb + KSTEP);
    }
    __syncthreads();
    for (int t = 0; t < rounds; ++t) {
        const int cur = t & 1;
        if (WGK == 1 || t < nt)
#pragma unroll
        for (int kk = 0; kk < BK; kk += 4) {
            const int kr = kk + lane / 16, c16 = lane % 16;
            R br[TJ], bi[TJ], bs[TJ], ar[TI], ai[TI], as[TI];
#pragma unroll
            for (int j = 0; j < TJ; ++j) {
                const int bn = wn0 + 16 * j + c16;
                br[j] = BKF ? Bs[cur][0][bn][kr] : Bs[cur][0][kr][bn];
                bi[j] = BKF ? Bs[cur][1][bn][kr] : Bs[cur][1][kr][bn];
                bs[j] = br[j] + bi[j];
            }
#pragma unroll
            for (int i = 0; i < TI; ++i) {
                const int am = wm0 + 16 * i + c16;
                ar[i] = AK ? As[cur][0][am][kr] : As[cur][0][kr][am];
                ai[i] = AK ? As[cur][1][am][kr] : As[cur][1][kr][am];
                as[i] = ar[i] + ai[i];
            }
            if constexpr (RAG) {   // c1 = Re, c3 = Im
#pragma unroll
                for (int i = 0; i < TI; ++i)
#pragma unroll
                    for (int j = 0; j < TJ; ++j) {
                        c1[i][j] = MfmaT<R>::mfma(br[j], ar[i], c1[i][j]);
                        c3[i][j] = MfmaT<R>::mfma(br[j], ai[i], c3[i][j]);
                        c1[i][j] = MfmaT<R>::mfma(-bi[j], ai[i], c1[i][j]);
                        c3[i][j] = MfmaT<R>::mfma(bi[j], ar[i], c3[i][j]);
                    }
                continue;
            }
            // the three products of one tile are independent: back-to-back
            // MFMAs never share an accumulator
#pragma unroll
            for (int i = 0; i < TI; ++i)
#pragma unroll
                for (int j = 0; j < TJ; ++j) {
                    c1[i][j] = MfmaT<R>::mfma(br[j], ar[i], c1[i][j]);
                    c2[i][j] = MfmaT<R>::mfma(bi[j], ai[i], c2[i][j]);
                    c3[i][j] = MfmaT<R>::mfma(bs[j], as[i], c3[i][j]);
                }
        }
        if (t + 1 < nt) {
            stash(cur ^ 1);
            if (t + 2 < nt) fetch(kb + (t + 2) * KSTEP);
        }
        __syncthreads();
    }
    // sums of the groups, [group][plane][register][thread]
    constexpr int REGS = 4 * TI * TJ;
    if constexpr (WGK > 1) {
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    R* dst = lds + ((2 * kg) * REGS + 4 * (i * TJ + j) + r) * NT + tid;
                    dst[0] = c1[i][j][r] - c2[i][j][r];
                    dst[REGS * NT] = c3[i][j][r] - c1[i][j][r] - c2[i][j][r];
                }
        __syncthreads();
    }
    if constexpr (FUSE == MFMA_NORMS) {
        static_assert(WGK == 1 && !RAG, "whole sums in one wave");
        // rows past M are zero (masked on load): sums over the lanes of a row
        // (m), then over the waves that share the columns
        R* sums = lds;   // [WGM][BN]
        __syncthreads();
#pragma unroll
        for (int j = 0; j < TJ; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                R t = 0;
#pragma unroll
                for (int i = 0; i < TI; ++i) {
                    const R re = c1[i][j][r] - c2[i][j][r], im = c3[i][j][r] - c1[i][j][r] - c2[i][j][r];
                    t += re * re + im * im;
                }
                t = row_total(t);
                if (lane % 16 == 0) sums[BN * (wave % WGM) + wn0 + 16 * j + MfmaT<R>::row(lane, r)] = t;
            }
        __syncthreads();
        if (tid < BN && n0 + tid < g.N) {
            R t = sums[tid];
#pragma unroll
            for (int w = 1; w < WGM; ++w) t += sums[BN * w + tid];
            x.norms[(int64_t)(n0 + tid) * tilesM + tm] = t;
        }
    }
    const int64_t MN = (int64_t)g.M * g.N;
    const int nbatch = g.B1 * g.B2;
    R* C = g.C + b1 * g.scb1 + b2 * g.scb2;
    R* P = partial + ((int64_t)sp * nbatch + b) * 2 * MN;
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = m0 + wm0 + 16 * i + lane % 16;
                const int n = n0 + wn0 + 16 * j + MfmaT<R>::row(lane, r);
                if (m >= g.M || n >= g.N) continue;
                R vre, vim;
                if constexpr (WGK > 1) {   // group q finishes registers q, q + WGK, ...
                    const int e = 4 * (i * TJ + j) + r;
                    if (e % WGK != kg) continue;
                    vre = lds[e * NT + tid];
                    vim = lds[(REGS + e) * NT + tid];
#pragma unroll
                    for (int q = 1; q < WGK; ++q) {
                        vre += lds[(2 * q * REGS + e) * NT + tid];
                        vim += lds[((2 * q + 1) * REGS + e) * NT + tid];
                    }
                } else {
                    vre = RAG ? c1[i][j][r] : c1[i][j][r] - c2[i][j][r];
                    vim = RAG ? c3[i][j][r] : c3[i][j][r] - c1[i][j][r] - c2[i][j][r];
                }
                if (splits == 1) {
                    const int64_t off = (int64_t)m * g.scm + (int64_t)n * g.scn;
                    R re = g.alpha * vre, im = g.alpha * vim;
                    if (g.beta) {
                        re += C[off];
                        im += C[off + g.c_plane];
                    }
                    C[off] = re;
                    C[off + g.c_plane] = im;
                } else {
                    P[m + (int64_t)g.M * n] = vre;
                    P[MN + m + (int64_t)g.M * n] = vim;
                }
            }
}

// ---------------------------------------------------------------------------
// Wave-sliced contraction kernel: any strides, any extents.  A block of WK
// waves owns one 16 x 16 output tile and splits K among its waves;
// every wave reads its matrix-core fragments straight from memory (no LDS
// staging, no barrier in the k loop, the next 16 k in flight while the
// current 16 are multiplied) and the WK partial tiles meet in LDS once, in
// wave order.  This is the kernel of the launches that are bound by latency
// rather than by the matrix cores: few output tiles, short or ragged K.  The
// complex product takes four real products per complex one, as a plain FMA
// loop would.
// Measured (FP64, us per launch inside a replayed graph, where an empty launch
// costs 3.8): parent-leg stack of a 9 x 9 x 64 node, five operators, 11.1 with
// 64 x 64 LDS tiles, 4.2 here; right-leg sum of a 27 x 27 x 64 node 33 -> 6.0;
// parent-leg sum of a 16^3 node over nine operators 12.8 (with its split-K
// reduction) -> 5.6.  16 x 16 tiles beat 32 x 16 and 32 x 32 ones on every one
// of these launches (more blocks, fewer loads ahead of the first product).
//   k order: lane group g = lane / 16 holds k = 16 kb + 4 g + u in its u-th
// of four matrix-core steps, so an operand contiguous along k is read four
// consecutive elements per lane; the contraction index is walked flattened
// over (k_in, k_out), so K is padded once (to 16) and not per outer index.
// ---------------------------------------------------------------------------
template <typename R, int WK>
__device__ inline void wave_tile(const Gemm<R>& g, int64_t bid, int tilesM, int tilesN, int splits, int kbper,
                                 R* partial) {
    if (g.skip && *g.skip) return;
    typedef typename MfmaT<R>::acc_t acc_t;
    const int tm = bid % tilesM;
    bid /= tilesM;
    const int tn = bid % tilesN;
    bid /= tilesN;
    const int sp = bid % splits;
    bid /= splits;
    const int b = (int)bid;
    const int b1 = b % g.B1, b2 = b / g.B1;
    const int m0 = tm * 16, n0 = tn * 16;
    const int K = g.Kin * g.Kout;
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const int c16 = lane % 16, g4 = lane / 16;
    // k blocks of 16: the split's range, then the wave's slice of it
    const int kb0 = sp * kbper, kb1 = min((K + 15) / 16, kb0 + kbper);
    const int per = (kb1 - kb0 + WK - 1) / WK;
    const int wb0 = kb0 + wave * per, wb1 = min(kb1, wb0 + per);
    // rows past the edge read the tile's first (their outputs are not stored)
    const R* A = g.A + b1 * g.sab1 + b2 * g.sab2 + (int64_t)(m0 + c16 < g.M ? m0 + c16 : m0) * g.sam;
    const R* B = g.B + b1 * g.sbb1 + b2 * g.sbb2 + (int64_t)(n0 + c16 < g.N ? n0 + c16 : n0) * g.sbn;
    const R sa = g.conjA ? R(-1) : R(1), sb = g.conjB ? R(-1) : R(1);
    struct Frag {
        R ar[4], ai[4], br[4], bi[4];
    };
    int k = 16 * wb0 + 4 * g4;
    int kout = k / g.Kin, kin = k - kout * g.Kin;
    // the 16 k of the next block: this lane's four, then the step to the block after
    auto fetch = [&](Frag& f) {
        int ki = kin, ko = kout;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const bool ok = k + u < K;
            const int64_t oa = ok ? (int64_t)ki * g.sak + (int64_t)ko * g.sako : 0;
            const int64_t ob = ok ? (int64_t)ki * g.sbk + (int64_t)ko * g.sbko : 0;
            const R ar = A[oa], ai = A[oa + g.a_plane], br = B[ob], bi = B[ob + g.b_plane];
            f.ar[u] = ok ? ar : R(0);
            f.ai[u] = ok ? sa * ai : R(0);
            f.br[u] = ok ? br : R(0);
            f.bi[u] = ok ? sb * bi : R(0);
            if (++ki == g.Kin) {
                ki = 0;
                ++ko;
            }
        }
        k += 16;
        kin += 16;
        while (kin >= g.Kin) {
            kin -= g.Kin;
            ++kout;
        }
    };
    acc_t cre = {0, 0, 0, 0}, cim = {0, 0, 0, 0};
    auto multiply = [&](const Frag& f) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            cre = MfmaT<R>::mfma(f.br[u], f.ar[u], cre);
            cim = MfmaT<R>::mfma(f.br[u], f.ai[u], cim);
            cre = MfmaT<R>::mfma(-f.bi[u], f.ai[u], cre);
            cim = MfmaT<R>::mfma(f.bi[u], f.ar[u], cim);
        }
    };
    if (wb0 < wb1) {
        Frag f0, f1;
        fetch(f0);
        for (int t = wb0; t < wb1; t += 2) {
            if (t + 1 < wb1) fetch(f1);
            multiply(f0);
            if (t + 1 >= wb1) break;
            if (t + 2 < wb1) fetch(f0);
            multiply(f1);
        }
    }
    const int64_t MN = (int64_t)g.M * g.N;
    const int nbatch = g.B1 * g.B2;
    R* C = g.C + b1 * g.scb1 + b2 * g.scb2;
    R* P = partial + ((int64_t)sp * nbatch + b) * 2 * MN;
    auto put = [&](int m, int n, R vre, R vim) {
        if (m >= g.M || n >= g.N) return;
        if (splits == 1) {
            const int64_t off = (int64_t)m * g.scm + (int64_t)n * g.scn;
            R re = g.alpha * vre, im = g.alpha * vim;
            if (g.beta) {
                re += C[off];
                im += C[off + g.c_plane];
            }
            C[off] = re;
            C[off + g.c_plane] = im;
        } else {
            P[m + (int64_t)g.M * n] = vre;
            P[MN + m + (int64_t)g.M * n] = vim;
        }
    };
    if constexpr (WK == 1) {
#pragma unroll
        for (int r = 0; r < 4; ++r) put(m0 + c16, n0 + MfmaT<R>::row(lane, r), cre[r], cim[r]);
    } else {
        // every wave publishes its partial tile, then each thread sums the WK
        // values of its outputs in wave order
        __shared__ R sh[WK][2][16][17];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int n = MfmaT<R>::row(lane, r);
            sh[wave][0][n][c16] = cre[r];
            sh[wave][1][n][c16] = cim[r];
        }
        __syncthreads();
        for (int e = threadIdx.x; e < 256; e += 64 * WK) {
            const int m = e % 16, n = e / 16;
            R re = 0, im = 0;
#pragma unroll
            for (int w = 0; w < WK; ++w) {
                re += sh[w][0][n][m];
                im += sh[w][1][n][m];
            }
            put(m0 + m, n0 + n, re, im);
        }
    }
}

template <typename R, int WK>
__global__ __launch_bounds__(64 * WK, 1) void k_cgemm_wave(Gemm<R> g, int tilesM, int tilesN, int splits,
                                                          int kbper, R* partial) {
    wave_tile<R, WK>(g, blockIdx.x, tilesM, tilesN, splits, kbper, partial);
}

// Several independent contractions in one launch (no split K): block b works
// on the member whose range [first[i], first[i + 1]) holds it.
template <typename R>
struct WaveGroup {
    Gemm<R> g[GROUP_MAX];
    int first[GROUP_MAX + 1];
    int count;
};

template <typename R, int WK>
__global__ __launch_bounds__(64 * WK, 1) void k_cgemm_wave_group(WaveGroup<R> w) {
    int i = 0;
    while (i + 1 < w.count && (int)blockIdx.x >= w.first[i + 1]) ++i;
    const Gemm<R>& g = w.g[i];
    wave_tile<R, WK>(g, blockIdx.x - w.first[i], (g.M + 15) / 16, (g.N + 15) / 16, 1,
                     (g.Kin * g.Kout + 15) / 16, nullptr);
}

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// ---------------------------------------------------------------------------
// FP32 operands on the bf16 matrix cores: x is taken as NP bf16 pieces (each
// the nearest bf16 of what the pieces before it leave of x) and a real product
// as the products of pieces p, q with p + q < NP on v_mfma_f32_32x32x16_bf16
// with FP32 accumulation; the complex product takes four real ones.
//   NP = 3 (FP32 mode): 3 x 8 significant bits hold an FP32 number exactly if
// its pieces lie in the range of bf16, the three dropped products are below
// 2^-24 of the whole.  Against 64 bits the result is closer than that of the
// FP32 matrix-core kernel it replaced (three FP32 products per complex one,
// whose Re + Im sums cancel): left-leg stack of a 128^3 node 2.6e-7 (3.9e-7
// before), parent-leg sum over 33 operators 8.0e-7 (1.17e-6).
//   Range of NP = 3: the first piece overflows from 3.39e38 on (an infinity turns
// into NaN), and below 2^-100 the last ones reach the subnormals of bf16.
// Outputs of operands out of range are taken again in plain FP32 products, with
// the operands read from memory: by a wave whose outputs are not finite, and by a
// block whose operands' largest magnitudes split_in_range refuses, which it looks
// for only if those of its first k-tile are small.  The k loop has no part in it
// (there, the largest magnitudes cost 1-4 % of a launch); what is left shows where
// a block has few k-tiles (128^3 left-leg stack of sixteen, eight tiles: 205 us
// without the checks, 209 with them; sum over 33: 344 / 343).  Sums of finite
// operands that overflow are not looked for: they are infinite or NaN, from 2^-8
// below the largest FP32 number on (the three-product form: from a quarter of it).
//   NP = 2 (BF16x3 mode): hi hi, hi lo, lo hi, relative error 4.4e-6.
// Loads are FP32; pieces are made while staging.  A wave owns 64 x 32 outputs
// (two 32 x 32 tiles); tiles of BM x BN outputs and 16 k, two LDS buffers (98 KB
// at 128 x 128, NP = 3), so one barrier per k-tile, and the stash of the next
// tile lies between the products of the current one.
//   What bounds it (FP32, 256^3 parent-leg sum): the matrix cores are busy
// 71 % of the cycles, but at 1.7 GHz -- 1.2 PFLOP/s of bf16 products is the
// chip's power limit (a library bf16 product of 8192^3 reaches 1.13).
// Measured, us, FP32 matrix cores -> here: 128^3 node, stacks of 17 on the left
// leg 337 -> 219 and of 16 on the right leg 292 -> 199, right-leg sum over 17
// 257 -> 184, parent-leg sum over 33 480 -> 345, 256^3 sum over five 1151 ->
// 823.  BF16x3, kernel with 16x16x32 products and 32-wide k-tiles -> here:
// 226 -> 148, 237 -> 216 (33), 256^3 right-leg sum over nine 953 -> 853.
//   RAG: any inner extent, padded to a whole k-tile for every outer index.
// ---------------------------------------------------------------------------

// Whether the products of operands with these largest magnitudes are those of
// exact pieces: no piece of a large entry below the normal numbers (2^-126, 26
// bits under 2^-100), no product of two of them (26 bits and the sum's growth
// under 2^-96).
__device__ inline bool split_in_range(float a, float b) {
    return a == 0.0f || b == 0.0f || (a >= 0x1p-100f && b >= 0x1p-100f && a * b >= 0x1p-96f);
}

template <int NP, int BM, int BN, bool AK, bool BKF, bool RAG>
__global__ __launch_bounds__(64 * (BM / 64) * (BN / 32), 2) void k_cgemm_split(Gemm<float> g, int tilesM, int tilesN,
                                                                              int splits, int kchunk,
                                                                              float* partial) {
    if (g.skip && *g.skip) return;
    constexpr int BK = 16, NT = 64 * (BM / 64) * (BN / 32);
    constexpr int TI = 2;   // wave: 64 x 32 outputs, two 32 x 32 tiles along m
    constexpr int QA = 4 * BM / NT, QB = 4 * BN / NT;
    static_assert(QA >= 1 && QB >= 1, "tile smaller than the block");
    typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
    typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
    // [buffer][re/im x piece][k / 8][row][8 k]: 16-byte rows, so that the
    // fragment reads (32 rows of one k half) and the stash are contiguous; the
    // halves are 64 bytes off the same banks for the stash of k-fast operands
    __shared__ __attribute__((aligned(16))) __bf16 As[2][2 * NP][2][BM + 4][8];
    __shared__ __attribute__((aligned(16))) __bf16 Bs[2][2 * NP][2][BN + 4][8];
    int64_t bid = blockIdx.x;
    const int tm = bid % tilesM;
    bid /= tilesM;
    const int tn = bid % tilesN;
    bid /= tilesN;
    const int sp = bid % splits;
    bid /= splits;
    const int b = (int)bid;
    const int b1 = b % g.B1, b2 = b / g.B1;
    const int m0 = tm * BM, n0 = tn * BN;
    // k runs over whole k-tiles of every outer index
    const int kinP = RAG ? (g.Kin + BK - 1) / BK * BK : g.Kin;
    const int K = kinP * g.Kout;
    const int kb = sp * kchunk;
    const int ke = min(K, kb + kchunk);
    const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
    const int wm0 = (wave % (BM / 64)) * 64, wn0 = (wave / (BM / 64)) * 32;
    // the thread's share of a tile: four k of QA / QB rows, re and im; rows past
    // the edge read row 0 (their outputs are not stored)
    auto rowA = [&](int q) { return AK ? (tid + NT * q) / 4 : (tid + NT * q) % BM; };
    auto rowB = [&](int q) { return BKF ? (tid + NT * q) / 4 : (tid + NT * q) % BN; };
    auto quadA = [&](int q) { return AK ? tid % 4 : (tid + NT * q) / BM; };
    auto quadB = [&](int q) { return BKF ? tid % 4 : (tid + NT * q) / BN; };
    int kin;
    const float *A[QA], *B[QB];
    auto rewind = [&]() {
        kin = kb % kinP;
        const int kout = kb / kinP;
#pragma unroll
        for (int q = 0; q < QA; ++q) {
            const int r = rowA(q);
            A[q] = g.A + b1 * g.sab1 + b2 * g.sab2 + (int64_t)m0 * g.sam + kin * g.sak + kout * g.sako +
                   (r < g.M - m0 ? r : 0) * g.sam + 4 * quadA(q) * g.sak;
        }
#pragma unroll
        for (int q = 0; q < QB; ++q) {
            const int r = rowB(q);
            B[q] = g.B + b1 * g.sbb1 + b2 * g.sbb2 + (int64_t)n0 * g.sbn + kin * g.sbk + kout * g.sbko +
                   (r < g.N - n0 ? r : 0) * g.sbn + 4 * quadB(q) * g.sbk;
        }
    };
    rewind();
    const int64_t wrapA = g.sako - kinP * g.sak, wrapB = g.sbko - kinP * g.sbk;
    const float sa = g.conjA ? -1.0f : 1.0f, sb = g.conjB ? -1.0f : 1.0f;
    float pa[QA][2][4], pb[QB][2][4];
    // four k of a row, re and im; k0: index of the first of them.  A quad that
    // reaches past Kin reads its row's k = 0 instead and takes zeros.
    auto load = [&](float (&x)[2][4], const float* src, int64_t plane, int64_t sk, bool kfast, int k0) {
        if (RAG && kin + BK > g.Kin) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool ok = k0 + j < g.Kin;
                const float* s = src + (ok ? j : -k0) * sk;
                const float re = s[0], im = s[plane];
                x[0][j] = ok ? re : 0.0f;
                x[1][j] = ok ? im : 0.0f;
            }
            return;
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const float* s = src + (h ? plane : 0);
            if (kfast) {
                const f32x4u t4 = *(const f32x4u*)s;
#pragma unroll
                for (int j = 0; j < 4; ++j) x[h][j] = t4[j];
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) x[h][j] = s[j * sk];
            }
        }
    };
    // loads this thread's share of the tile at (A, B); advance: on to the next
    auto fetch = [&](bool advance) {
        const bool wrap = kin + BK == kinP;
        const int64_t da = advance ? BK * g.sak + (wrap ? wrapA : 0) : 0;
        const int64_t db = advance ? BK * g.sbk + (wrap ? wrapB : 0) : 0;
#pragma unroll
        for (int q = 0; q < QA; ++q) {
            load(pa[q], A[q], g.a_plane, g.sak, AK, kin + 4 * quadA(q));
            A[q] += da;
        }
#pragma unroll
        for (int q = 0; q < QB; ++q) {
            load(pb[q], B[q], g.b_plane, g.sbk, BKF, kin + 4 * quadB(q));
            B[q] += db;
        }
        kin = advance ? (wrap ? 0 : kin + BK) : kin;
    };
    auto stash1 = [&](auto& S, int row, int quad, const float (&x)[2][4], float sg) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            float r[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) r[j] = h ? x[h][j] * sg : x[h][j];
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                bf16x4 v;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    v[j] = (__bf16)r[j];
                    r[j] -= (float)v[j];
                }
                *(bf16x4*)&S[h * NP + p][quad >> 1][row][4 * (quad & 1)] = v;
            }
        }
    };
    auto stash = [&](int buf) {
#pragma unroll
        for (int q = 0; q < QA; ++q) stash1(As[buf], rowA(q), quadA(q), pa[q], sa);
#pragma unroll
        for (int q = 0; q < QB; ++q) stash1(Bs[buf], rowB(q), quadB(q), pb[q], sb);
    };
    f32x16 crr[TI], cii[TI], cim[TI];
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) crr[i][r] = cii[i][r] = cim[i][r] = 0.0f;
    const int nt = (ke - kb) / BK;
    const int r32 = lane % 32, kh = lane / 32;
    float maxA = 0.0f, maxB = 0.0f;   // largest magnitudes of the thread's operands (NaN passed over)
    auto largest = [&]() {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
#pragma unroll
            for (int q = 0; q < QA; ++q) maxA = fmaxf(maxA, fabsf(pa[q][j / 4][j % 4]));
#pragma unroll
            for (int q = 0; q < QB; ++q) maxB = fmaxf(maxB, fabsf(pb[q][j / 4][j % 4]));
        }
    };
    __shared__ int s_box[NP == 3 ? NT / 64 : 1];   // a wave's first tile holds an entry of 2^-48: 1 of A, 2 of B
    if (nt > 0) {
        fetch(nt > 1);
        if constexpr (NP == 3) {
            largest();
            const int bits = (__any(maxA >= 0x1p-48f) ? 1 : 0) | (__any(maxB >= 0x1p-48f) ? 2 : 0);
            s_box[wave] = bits;   // by every lane: a branch here would hold the next loads back
        }
        stash(0);
        fetch(nt > 2);
    }
    __syncthreads();
    for (int t = 0; t < nt; ++t) {
        const int cur = t & 1;
        bf16x8 bf[2 * NP], af[TI][2 * NP];
#pragma unroll
        for (int p = 0; p < 2 * NP; ++p) bf[p] = *(const bf16x8*)&Bs[cur][p][kh][wn0 + r32][0];
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int p = 0; p < 2 * NP; ++p) af[i][p] = *(const bf16x8*)&As[cur][p][kh][wm0 + 32 * i + r32][0];
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int s2 = NP - 1; s2 >= 0; --s2)   // pieces p + q = s2, the smallest products first
#pragma unroll
                for (int p = 0; p <= s2; ++p) {
                    const int q = s2 - p;
                    crr[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[p], af[i][q], crr[i], 0, 0, 0);
                    cii[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[NP + p], af[i][NP + q], cii[i], 0, 0, 0);
                    cim[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[p], af[i][NP + q], cim[i], 0, 0, 0);
                    cim[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[NP + p], af[i][q], cim[i], 0, 0, 0);
                }
        // the next tile (the last one again past the end) into the other
        // buffer, its conversions between the products above
        stash(cur ^ 1);
        fetch(t + 3 < nt);
        // BF16x3: fragment reads first, then five vector operations between
        // two products.  With three pieces the chip runs at its power limit
        // (1.7 GHz) and the compiler's own order is the faster one.
        if constexpr (NP == 2) {
            constexpr int NM = 2 * NP * (NP + 1);       // products per 32 x 32 tile
            __builtin_amdgcn_sched_group_barrier(0x100, 4 * NP, 0);
#pragma unroll
            for (int q = 0; q < 2 * NM; ++q) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                if (q < 2 * NP) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);
                if (q >= 4 && q % 3 == 0) __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
            }
        }
        __syncthreads();
    }
    if constexpr (NP == 3) {
        bool plain = false;
        int box = 0;
#pragma unroll
        for (int w = 0; w < NT / 64; ++w) box |= s_box[w];
        if (__builtin_expect(box != 3 && nt > 0, 0)) {   // the same in every wave
            __shared__ float s_max[2][NT / 64];
            rewind();
            for (int t = 0; t < nt; ++t) {
                fetch(t + 1 < nt);
                largest();
            }
            for (int o = 32; o > 0; o >>= 1) {
                maxA = fmaxf(maxA, __shfl_xor(maxA, o, 64));
                maxB = fmaxf(maxB, __shfl_xor(maxB, o, 64));
            }
            if (lane == 0) {
                s_max[0][wave] = maxA;
                s_max[1][wave] = maxB;
            }
            __syncthreads();
            for (int w = 0; w < NT / 64; ++w) {
                maxA = fmaxf(maxA, s_max[0][w]);
                maxB = fmaxf(maxB, s_max[1][w]);
            }
            plain = !split_in_range(maxA, maxB);
        }
        // an entry out of range makes the imaginary parts of its whole row or column
        // of outputs not finite: one column and one row of every tile tell; z is NaN then
        float z[4] = {0, 0, 0, 0};
#pragma unroll
        for (int i = 1; i < TI; ++i) z[i % 4] = fmaf(cim[i][0], 0.0f, z[i % 4]);
#pragma unroll
        for (int r = 0; r < 16; ++r) z[r % 4] = fmaf(cim[0][r], 0.0f, z[r % 4]);
        if (__builtin_expect(plain || __any((z[0] + z[1]) + (z[2] + z[3]) != 0.0f), 0)) {
            const float* A0 = g.A + b1 * g.sab1 + b2 * g.sab2;
            const float* B0 = g.B + b1 * g.sbb1 + b2 * g.sbb2;
            // both tiles along m share the sixteen columns; those past N read the first
#pragma unroll
            for (int i = 0; i < TI; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) crr[i][r] = cii[i][r] = cim[i][r] = 0.0f;
            int ki = kb % kinP, ko = kb / kinP;
#pragma unroll 1
            for (int k = kb; k < ke; ++k) {
                if (ki < g.Kin) {
                    float ar[TI], ai[TI];
#pragma unroll
                    for (int i = 0; i < TI; ++i) {
                        const int m = m0 + wm0 + 32 * i + r32;
                        const float* a = A0 + (int64_t)(m < g.M ? m : m0) * g.sam + (int64_t)ki * g.sak +
                                         (int64_t)ko * g.sako;
                        ar[i] = a[0];
                        ai[i] = sa * a[g.a_plane];
                    }
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int n = n0 + wn0 + 8 * (r / 4) + 4 * kh + r % 4;
                        const float* b = B0 + (int64_t)(n < g.N ? n : n0) * g.sbn + (int64_t)ki * g.sbk +
                                         (int64_t)ko * g.sbko;
                        const float br = b[0], bi = sb * b[g.b_plane];
#pragma unroll
                        for (int i = 0; i < TI; ++i) {
                            crr[i][r] = fmaf(-ai[i], bi, fmaf(ar[i], br, crr[i][r]));
                            cim[i][r] = fmaf(ai[i], br, fmaf(ar[i], bi, cim[i][r]));
                        }
                    }
                }
                if (++ki == kinP) {
                    ki = 0;
                    ++ko;
                }
            }
        }
    }
    const int64_t MN = (int64_t)g.M * g.N;
    const int nbatch = g.B1 * g.B2;
    float* C = g.C + b1 * g.scb1 + b2 * g.scb2;
    float* P = partial + ((int64_t)sp * nbatch + b) * 2 * MN;
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int m = m0 + wm0 + 32 * i + r32;
            const int n = n0 + wn0 + 8 * (r / 4) + 4 * kh + r % 4;
            if (m >= g.M || n >= g.N) continue;
            const float vre = crr[i][r] - cii[i][r];
            const float vim = cim[i][r];
            if (splits == 1) {
                const int64_t off = (int64_t)m * g.scm + (int64_t)n * g.scn;
                float re = g.alpha * vre, im = g.alpha * vim;
                if (g.beta) {
                    re += C[off];
                    im += C[off + g.c_plane];
                }
                C[off] = re;
                C[off + g.c_plane] = im;
            } else {
                P[m + (int64_t)g.M * n] = vre;
                P[MN + m + (int64_t)g.M * n] = vim;
            }
        }
}

// Launches below this many real flops are bound by latency and take the
// wave-sliced kernel, above it the LDS-tiled kernels.  Measured on both sides
// (us, LDS tiles / wave-sliced, split-K reductions included): FP64 0.15 Gflop
// (a 128 x 128 bond) 16.5 / 11.7, FP32 0.285 Gflop 16.1 / 11.6, FP64 0.54 Gflop
// (a 64^3 node) 15.8 / 19.2, FP32 0.67 Gflop 14.8 / 23.8.
constexpr double WAVE_MAX_FLOPS = 0.3e9;

// Launches of FP32 arrays from here on may take k_cgemm_split.
constexpr double SPLIT_MIN_FLOPS = 1e9;

// Split factor of a launch whose `tiles` output tiles leave the chip idle: up
// to `target` workgroups, at least `minkt` k-tiles each, partial sums within
// the scratch.
template <typename R>
int split_factor(const Gemm<R>& g, const GemmScratch& ws, int64_t tiles, int ktiles, int64_t target, int minkt) {
    if (tiles >= target || ktiles < 2 * minkt || (int64_t)g.M * g.N >= (1LL << 31)) return 1;
    const int64_t per = 2 * (int64_t)g.M * g.N * g.B1 * g.B2 * (int64_t)sizeof(R);
    const int64_t s = std::min<int64_t>((target + tiles - 1) / tiles, ktiles / minkt);
    return (int)std::max<int64_t>(1, std::min<int64_t>(s, ws.bytes / per));
}

// Waves per tile of k_cgemm_wave: one or two k-blocks a wave on short K;
// sixteen waves on long K, unless there are tiles enough for several blocks
// per CU (a stack over a 128 x 128 bond: 11.7 us with eight waves, 14.9 with
// sixteen; 288 to 486 tiles, K = 256 to 450: sixteen 8-15 % slower); one wave
// where the tiles alone are eight waves a CU (FP64, 160 x 36 x 20 node, parent-leg
// stack of sixteen: 49.0 us with four, 27.2 with one; 64 x 208 x 24, stack of four
// 30.4 / 17.9; FP32, 21 x 73 x 245, left-leg stack of four 23.7 / 17.9).
inline int wave_count(int kblocks, int64_t tiles) {
    if (tiles >= 2048) return 1;
    return kblocks >= 16 && tiles <= 256 ? 16 : kblocks >= 8 ? 8 : kblocks >= 2 ? 4 : 1;
}

// Whether k_cgemm_mfma's aligned form takes a Gemm: k-tiles of 16 inside the
// inner extent, unit strides to stage along, and 32-bit element offsets inside
// a tile.
template <typename R>
bool aligned_form(const Gemm<R>& g) {
    const bool off32 = (int64_t)128 * (g.sam + g.sbn) + 32 * (g.sak + g.sbk) + g.a_plane + g.b_plane < (1LL << 31);
    return g.Kout > 0 && g.Kin >= 16 && g.Kin % 16 == 0 && g.M >= 16 && g.N >= 16 && (g.sam == 1 || g.sak == 1) &&
           (g.sbn == 1 || g.sbk == 1) && off32;
}

// Tiles of bm x bn outputs of all batches.
template <typename R>
int64_t tile_count(const Gemm<R>& g, int bm, int bn) {
    return (int64_t)((g.M + bm - 1) / bm) * ((g.N + bn - 1) / bn) * g.B1 * g.B2;
}

// Launches for the wave-sliced kernel: below WAVE_MAX_FLOPS, unless the aligned
// 32 x 32 tiles cover half the chip, where staging through LDS reads the
// operands half as often (us, wave-sliced / tiles: 128 tiles with K = 64, FP64
// 9.9 / 7.8, FP32 8.0 / 6.2; 512 tiles with K = 32, 23.3 / 11.5; below, 64 tiles
// with K = 64 5.9 / 7.4; K = 192 over 144 tiles, FP32, 8.3 / 9.1).  From there on,
// ragged launches of at most 16 rows or columns, which its tiles do not pad to 32
// (FP64, 9 x 208 x 624 node, right-leg product 159 us with 32 x 32 tiles, 91 here;
// FP32, 8 x 256 x 256, left-leg sum over 33 111 / 67), while K is short (K = 4224
// over 12 x 128 outputs of 36 74.6 / 79.7).
template <typename R>
bool takes_wave(const Gemm<R>& g) {
    const int64_t K = (int64_t)g.Kin * g.Kout;
    if (8.0 * g.M * g.N * (double)K * g.B1 * (double)g.B2 >= WAVE_MAX_FLOPS)
        return std::min(g.M, g.N) <= 16 && K <= 1024 && !aligned_form(g);
    return !(aligned_form(g) && g.M >= 32 && g.N >= 32 && tile_count(g, 32, 32) >= (K > 128 ? 256 : 128));
}

template <typename R>
int64_t wave_tiles(const Gemm<R>& g) {
    return (int64_t)((g.M + 15) / 16) * ((g.N + 15) / 16) * g.B1 * g.B2;
}

template <typename R>
int wave_splits(const Gemm<R>& g, const GemmScratch& ws) {
    return split_factor(g, ws, wave_tiles(g), (g.Kin * g.Kout + 15) / 16, 256, 32);
}

// Launch of k_cgemm_wave for any Gemm.
template <typename R>
void launch_wave(const Gemm<R>& g, const GemmScratch& ws, hipStream_t s, CgemmInfo* info) {
    const int K = g.Kin * g.Kout;
    const int kblocks = (K + 15) / 16;
    const int tilesM = (g.M + 15) / 16, tilesN = (g.N + 15) / 16;
    const int64_t tiles = wave_tiles(g);
    const int wk = wave_count(kblocks, tiles);
    int splits = wave_splits(g, ws);
    const int kbper = (kblocks + splits - 1) / splits;
    if (kbper > 0) splits = (kblocks + kbper - 1) / kbper;
    const dim3 grid((unsigned)(tiles * splits));
    R* part = (R*)ws.partial;
    if (info) *info = CgemmInfo{2, splits};
#define TTN_WAVE_LAUNCH(w)                                                                                   \
    hipLaunchKernelGGL((k_cgemm_wave<R, w>), grid, dim3(64 * w), 0, s, g, tilesM, tilesN, splits, kbper, part)
    if (wk == 16)
        TTN_WAVE_LAUNCH(16);
    else if (wk == 8)
        TTN_WAVE_LAUNCH(8);
    else if (wk == 4)
        TTN_WAVE_LAUNCH(4);
    else
        TTN_WAVE_LAUNCH(1);
#undef TTN_WAVE_LAUNCH
    if (splits > 1) splitk_reduce(g, splits, (const R*)ws.partial, s);
}

// Output elements a grid of bm x bn tiles computes, padding included.
inline double padded(int M, int N, int bm, int bn) {
    return (double)((M + bm - 1) / bm) * ((N + bn - 1) / bn) * bm * bn;
}

// Launch of the ragged form of k_cgemm_mfma, 64 x 64 or 32 x 32 tiles.
template <typename R>
void launch_ragged(const Gemm<R>& g, const GemmScratch& ws, hipStream_t s, bool small, bool a_k, bool b_k,
                   CgemmInfo* info) {
    const int K = g.Kin * g.Kout;
    const int bt = small ? 32 : 64;
    const int tilesM = (g.M + bt - 1) / bt, tilesN = (g.N + bt - 1) / bt;
    const int64_t tiles = (int64_t)tilesM * tilesN * g.B1 * g.B2;
    const int ktiles = (K + 15) / 16;
    int splits = split_factor(g, ws, tiles, ktiles, small ? 1024 : 512, 4);
    const int kchunk = (ktiles + splits - 1) / splits * 16;
    splits = (K + kchunk - 1) / kchunk;
    const dim3 grid((unsigned)(tiles * splits));
    R* part = (R*)ws.partial;
    if (info) *info = CgemmInfo{2, splits};
#define TTN_RAG_LAUNCH(bt, minb, ak, bk)                                                                       \
    hipLaunchKernelGGL((k_cgemm_mfma<R, bt, bt, 2, 2, 1, minb, 16, ak, bk, true>), grid, dim3(256), 0, s, g, tilesM, \
                       tilesN, splits, kchunk, part, MfmaExtra<R>{})
#define TTN_RAG_LAUNCHES(bt, minb)             \
    do {                                       \
        if (a_k && b_k)                        \
            TTN_RAG_LAUNCH(bt, minb, true, true);    \
        else if (a_k)                          \
            TTN_RAG_LAUNCH(bt, minb, true, false);   \
        else if (b_k)                          \
            TTN_RAG_LAUNCH(bt, minb, false, true);   \
        else                                   \
            TTN_RAG_LAUNCH(bt, minb, false, false);  \
    } while (0)
    if (small)
        TTN_RAG_LAUNCHES(32, 4);
    else
        TTN_RAG_LAUNCHES(64, 2);
#undef TTN_RAG_LAUNCHES
#undef TTN_RAG_LAUNCH
    if (splits > 1) splitk_reduce(g, splits, (const R*)ws.partial, s);
}

// Estimated time (us) of the pass over split K's partial sums.
template <typename R>
double reduce_us(const Gemm<R>& g, int splits) {
    return splits < 2 ? 0.0 : 1.0 + splits * 4.0 * sizeof(R) * g.M * (double)g.N * g.B1 * g.B2 / 7.2e6;
}

// Launch of the aligned form of k_cgemm_mfma.  64 x 64 tiles (8 waves, two blocks
// per CU) or 32 x 32 ones (4 waves), whichever the estimate below puts first, with
// two or four groups of waves on a 32 x 32 tile when there are few of them, so
// that a CU has 8 to 16 waves; FP64 launches with a long K take 128 x 64 tiles
// (16 waves).  K is split over the grid only where the 32 x 32 tiles leave CUs
// without a block, or where a long K meets few 64 x 64 tiles.
// Measured, FP64, us (128 x 64 tiles or 64 x 64 ones of four waves with K split
// over the grid / the rule here): right-leg sum of a 64^3 node over 4, 8, 16
// operators 28.9 / 14.6, 33.7 / 24.8, 48.9 / 44.1; stack of 8 over 64^3 23.8 /
// 24.2, over 128^3 292 / 267; 96^3 sum over 8 191 / 110; 32 x 32 x 128 node,
// parent-leg stack of 8 34.7 / 23.3.  FP32, 64^3 sum over 4: 23.7 / 10.2.
struct AlignedPlan {
    bool small, big;
    int groups, splits, kchunk;
    int64_t blocks;
};

template <typename R>
AlignedPlan plan_aligned(const Gemm<R>& g, const GemmScratch& ws) {
    const int K = g.Kin * g.Kout, kt = K / 16;
    const int64_t t32 = tile_count(g, 32, 32), t64 = tile_count(g, 64, 64), t128 = tile_count(g, 128, 64);
    // us per k of a 32 x 32 tile on every CU; 32 x 32 tiles reach 0.87 of the larger
    // ones' rate (FP32: 0.8) where both fill the chip (128^3: 305 / 268 us)
    const double ck = sizeof(R) == 8 ? 0.041 : 0.0263, r32 = sizeof(R) == 8 ? 0.87 : 0.8;
    // time in rounds of tiles over the CUs: with a short K, 64 x 64 tiles a little
    // over one to a CU leave most of the second round empty (FP64, 1944 x 48 outputs
    // of nine operators, 279 tiles: 17.8 us, 1098 of 32 x 32 14.9; FP32, 2560 x 64 of
    // nine, 360: 14.8 / 13.7; but 221 of them 11.5, 884 of 32 x 32 12.7; K = 1024,
    // 10368 x 128 outputs, 324 tiles 197, 1296 of 32 x 32 222)
    auto rounds = [&](int64_t blocks) {
        return blocks <= 256 ? 1.0 : K <= 256 ? (double)((blocks + 255) / 256) : blocks / 256.0;
    };
    const double us64 = rounds(t64) * 4 * r32 * ck * K;
    // 32 x 32 tiles that leave CUs without a block split K, into whole rounds where
    // it pays (FP64, 192 x 288 outputs, K = 1536, 54 tiles: 33.7 us with 270 blocks,
    // 25.4 with 216; 1152 x 112, K = 1904, 144 tiles: 77 with one split, 63 with four;
    // FP32, 160 x 96 of twelve, K = 480, 180 tiles: 18.7 with two, 14.6 with one)
    const int64_t per = 2 * (int64_t)g.M * g.N * g.B1 * g.B2 * (int64_t)sizeof(R);
    int s32 = 1;
    double us32 = rounds(t32) * ck * K;
    if (t32 < 256 && (int64_t)g.M * g.N < (1LL << 31))
        for (int q = 2; q <= std::min<int64_t>(std::min(16, kt / 8), ws.bytes / per); ++q) {
            const double u = std::ceil(t32 * q / 256.0) / q * ck * K + reduce_us(g, q);
            if (u < us32) {
                us32 = u;
                s32 = q;
            }
        }
    // few outputs and a long K: 64 x 64 tiles split to 512 blocks, where the 32 x 32
    // ones would be split too (128 x 128 outputs, K = 16384: 53.7 us with 32 x 32
    // tiles, 48.4 with 64 x 64; half the flops: 31.3 / 32.2) or K is so long that
    // the partial sums weigh little (64 x 8192 outputs, K = 4096: 353 / 268; 64 x
    // 4096, K = 2048: 84.9 / 77.6; K = 1024: 46.2 / 51), and only with little
    // padding (24 x 64 outputs of 80, K = 1088: 44.0 with 64 x 64, 31.9 with 32 x 32)
    const bool deep = t64 < 256 && t64 * (kt / 8) >= 512 && (t32 < 256 || kt >= 128) &&
                      3 * padded(g.M, g.N, 64, 64) <= 4 * padded(g.M, g.N, 32, 32);
    AlignedPlan p;
    p.small = !deep && us32 < us64;
    p.big = !p.small && sizeof(R) == 8 && K >= 512 && t128 >= 256 &&
            padded(g.M, g.N, 128, 64) <= padded(g.M, g.N, 64, 64);
    const int64_t tiles = p.small ? t32 : p.big ? t128 : t64;
    p.splits = p.big ? 1 : p.small ? s32 : split_factor(g, ws, tiles, kt, 512, deep ? 8 : 32);
    p.kchunk = (kt + p.splits - 1) / p.splits * 16;
    p.splits = (K + p.kchunk - 1) / p.kchunk;
    p.blocks = tiles * p.splits;
    p.groups = !p.small || p.kchunk < 128 ? 1 : p.blocks <= 256 ? 4 : p.blocks <= 512 ? 2 : 1;
    return p;
}

#define TTN_MFMA_LAUNCH(bm, bn, wgm, wgn, wgk, minb, ak, bk, fuse)                                                   \
    hipLaunchKernelGGL((k_cgemm_mfma<R, bm, bn, wgm, wgn, wgk, minb, 16, ak, bk, false, fuse>),                      \
                       dim3((unsigned)p.blocks), dim3(64 * wgm * wgn * wgk), 0, s, g, (g.M + bm - 1) / bm,           \
                       (g.N + bn - 1) / bn, p.splits, p.kchunk, (R*)ws.partial, x)

template <typename R>
void launch_aligned(const Gemm<R>& g, const GemmScratch& ws, hipStream_t s, bool a_k, bool b_k, CgemmInfo* info) {
    const AlignedPlan p = plan_aligned(g, ws);
    const MfmaExtra<R> x;
    if (info) *info = CgemmInfo{2, p.splits};
#define TTN_MFMA_LAUNCHES(bm, bn, wgm, wgn, wgk, minb)                                \
    do {                                                                              \
        if (a_k && b_k)                                                               \
            TTN_MFMA_LAUNCH(bm, bn, wgm, wgn, wgk, minb, true, true, MFMA_PLAIN);     \
        else if (a_k)                                                                 \
            TTN_MFMA_LAUNCH(bm, bn, wgm, wgn, wgk, minb, true, false, MFMA_PLAIN);    \
        else if (b_k)                                                                 \
            TTN_MFMA_LAUNCH(bm, bn, wgm, wgn, wgk, minb, false, true, MFMA_PLAIN);    \
        else                                                                          \
            TTN_MFMA_LAUNCH(bm, bn, wgm, wgn, wgk, minb, false, false, MFMA_PLAIN);   \
    } while (0)
    if (p.groups == 4)
        TTN_MFMA_LAUNCHES(32, 32, 2, 2, 4, 1);
    else if (p.groups == 2)
        TTN_MFMA_LAUNCHES(32, 32, 2, 2, 2, 2);
    else if (p.small)
        TTN_MFMA_LAUNCHES(32, 32, 2, 2, 1, 4);
    else if (!p.big)
        TTN_MFMA_LAUNCHES(64, 64, 2, 4, 1, 2);
    else if constexpr (sizeof(R) == 8)
        TTN_MFMA_LAUNCHES(128, 64, 4, 4, 1, 1);
#undef TTN_MFMA_LAUNCHES
    if (p.splits > 1) splitk_reduce(g, p.splits, (const R*)ws.partial, s);
}

// Tiles and split factor of a k_cgemm_split launch with np pieces: of 128 x 128, 64 x
// 128 and 128 x 64 tiles and the factors that leave at least four k-tiles to a
// block, the least of the estimated time: rounds of blocks over the CUs (from the
// third on, half of what the last one leaves empty is made up for), each 0.116 us
// per k (two pieces: 0.06) with 34 k of prologue and epilogue, of the half tiles
// 0.78 alone on a CU and 0.61 beside others, and the pass over the partial sums
// (within 7 % on average of 1386 launches of 66 shapes, its choice within 1 % of
// the best one).  Splitting K until a grid covers the chip loses where that pass
// is long or the last round short (us, split so / this: 64 x 26624 outputs, K =
// 256, 208 tiles 44 / 31; 128 x 4320 of five, K = 128, 170 tiles 41 / 22; 972 x 144 of
// seventeen, K = 144 47 / 30).
struct SplitPlan {
    int bm, bn, splits;
};
inline SplitPlan plan_split(const Gemm<float>& g, const GemmScratch& ws, int np) {
    const int K = (g.Kin + 15) / 16 * 16 * g.Kout;
    SplitPlan p{0, 0, 1};
    double least = 0.0;
    for (const auto& t : {SplitPlan{128, 128, 1}, SplitPlan{64, 128, 1}, SplitPlan{128, 64, 1}}) {
        const bool wide = t.bm == t.bn;
        const int64_t tiles = tile_count(g, t.bm, t.bn);
        const int most = split_factor(g, ws, tiles, K / 16, 1024, 4);
        for (int q = 1; q <= most; ++q) {
            const double x = tiles * q / 256.0, rounds = x <= 2 ? std::ceil(x) : 0.5 * (std::ceil(x) + x);
            const double full = wide ? rounds : rounds <= 1 ? 0.78 : 0.61 * rounds;
            const double us = full * (np == 3 ? 0.116 : 0.06) * ((double)K / q + 34) + reduce_us(g, q);
            if (p.bm == 0 || us < least) {
                least = us;
                p = SplitPlan{t.bm, t.bn, q};
            }
        }
    }
    return p;
}

// Launch of k_cgemm_split.
void launch_split(const Gemm<float>& g, const GemmScratch& ws, hipStream_t s, int np, bool a_k, bool b_k,
                  CgemmInfo* info) {
    const SplitPlan p = plan_split(g, ws, np);
    const int bm = p.bm, bn = p.bn;
    const bool rag = g.Kin % 16 != 0;
    const int K = (g.Kin + 15) / 16 * 16 * g.Kout;
    const int tilesM = (g.M + bm - 1) / bm, tilesN = (g.N + bn - 1) / bn;
    const int64_t tiles = (int64_t)tilesM * tilesN * g.B1 * g.B2;
    const bool wide = bm == 128 && bn == 128;
    int splits = p.splits;
    const int kchunk = (K / 16 + splits - 1) / splits * 16;
    splits = (K + kchunk - 1) / kchunk;
    const dim3 grid((unsigned)(tiles * splits)), blk(wide ? 512 : 256);
    float* part = (float*)ws.partial;
    if (info) *info = CgemmInfo{np == 2 ? 3 : 2, splits};
#define TTN_SPLIT_LAUNCH(np, bm, bn, ak, bk, rag)                                                               \
    hipLaunchKernelGGL((k_cgemm_split<np, bm, bn, ak, bk, rag>), grid, blk, 0, s, g, tilesM, tilesN, splits, kchunk, \
                       part)
#define TTN_SPLIT_LAUNCHES(np, bm, bn, rag)                     \
    do {                                                        \
        if (a_k && b_k)                                         \
            TTN_SPLIT_LAUNCH(np, bm, bn, true, true, rag);      \
        else if (a_k)                                           \
            TTN_SPLIT_LAUNCH(np, bm, bn, true, false, rag);     \
        else if (b_k)                                           \
            TTN_SPLIT_LAUNCH(np, bm, bn, false, true, rag);     \
        else                                                    \
            TTN_SPLIT_LAUNCH(np, bm, bn, false, false, rag);    \
    } while (0)
#define TTN_SPLIT_TILES(np, rag)                   \
    do {                                           \
        if (wide)                                  \
            TTN_SPLIT_LAUNCHES(np, 128, 128, rag); \
        else if (bm == 64)                         \
            TTN_SPLIT_LAUNCHES(np, 64, 128, rag);  \
        else                                       \
            TTN_SPLIT_LAUNCHES(np, 128, 64, rag);  \
    } while (0)
    if (np == 2)
        TTN_SPLIT_TILES(2, false);
    else if (rag)
        TTN_SPLIT_TILES(3, true);
    else
        TTN_SPLIT_TILES(3, false);
#undef TTN_SPLIT_TILES
#undef TTN_SPLIT_LAUNCHES
#undef TTN_SPLIT_LAUNCH
    if (splits > 1) splitk_reduce(g, splits, (const float*)ws.partial, s);
}

// Largest element offset an operand can touch (all strides are >= 0).
inline bool inside(const GemmScratch& ws, const void* base, int64_t max_off, int64_t plane, int esz) {
    if (!ws.regions) return true;
    const uintptr_t p = (uintptr_t)base;
    int lo = 0, hi = ws.n_regions - 1, f = -1;
    while (lo <= hi) {
        const int mid = (lo + hi) / 2;
        if (ws.regions[mid].lo <= p) {
            f = mid;
            lo = mid + 1;
        } else {
            hi = mid - 1;
        }
    }
    if (f < 0) return false;
    const uintptr_t end = p + (uintptr_t)(max_off + plane + 1) * esz;
    return p >= ws.regions[f].lo && end <= ws.regions[f].hi;
}

}  // namespace

bool g_dry_run = false;

template <typename R>
bool cgemm_check(const Gemm<R>& g, const GemmScratch& ws, char* why, int whylen) {
    const int64_t km = g.Kin > 0 ? g.Kin - 1 : 0, ko = g.Kout > 0 ? g.Kout - 1 : 0;
    const int64_t b1 = g.B1 - 1, b2 = g.B2 - 1;
    const int64_t amax = (g.M - 1) * g.sam + km * g.sak + ko * g.sako + b1 * g.sab1 + b2 * g.sab2;
    const int64_t bmax = (g.N - 1) * g.sbn + km * g.sbk + ko * g.sbko + b1 * g.sbb1 + b2 * g.sbb2;
    const int64_t cmax = (g.M - 1) * g.scm + (g.N - 1) * g.scn + b1 * g.scb1 + b2 * g.scb2;
    const bool neg = g.sam < 0 || g.sak < 0 || g.sako < 0 || g.sab1 < 0 || g.sab2 < 0 || g.sbn < 0 ||
                     g.sbk < 0 || g.sbko < 0 || g.sbb1 < 0 || g.sbb2 < 0 || g.scm < 0 || g.scn < 0 ||
                     g.scb1 < 0 || g.scb2 < 0 || g.a_plane < 0 || g.b_plane < 0 || g.c_plane < 0;
    const char* bad = neg ? "negative stride"
                      : !inside(ws, g.A, amax, g.a_plane, sizeof(R)) ? "operand A out of its region"
                      : !inside(ws, g.B, bmax, g.b_plane, sizeof(R)) ? "operand B out of its region"
                      : !inside(ws, g.C, cmax, g.c_plane, sizeof(R)) ? "operand C out of its region"
                                                                     : nullptr;
    if (bad) {
        if (why)
            snprintf(why, whylen, "%s (M=%d N=%d Kin=%d Kout=%d B=%dx%d)", bad, g.M, g.N, g.Kin, g.Kout,
                     g.B1, g.B2);
        return false;
    }
    return true;
}

template <typename R>
bool cgemm_groupable(const Gemm<R>& g, const GemmScratch& ws) {
    const bool any = g.M > 0 && g.N > 0 && g.Kin > 0 && g.Kout > 0 && g.B1 > 0 && g.B2 > 0;
    return any && takes_wave(g) && wave_splits(g, ws) == 1;
}

// A wave-sliced launch whose tiles span all the rows (C over A: columns) of its
// outputs and do not split K: every workgroup has then read, when it writes
// (after its last product), all that its own outputs replace, and no other
// workgroup reads that.  Wider legs belong to large tensors, where the copy
// weighs little beside the product.
bool cgemm_in_place(const Gemm<double>& g, const GemmScratch& ws, bool over_a) {
    if (g.M <= 0 || g.N <= 0 || g.Kin * g.Kout <= 0) return false;
    return takes_wave(g) && (over_a ? g.N : g.M) <= 16 && wave_splits(g, ws) == 1;
}

template <typename R>
int cgemm_group(const Gemm<R>* g, int count, const GemmScratch& ws, hipStream_t s) {
    if (g_dry_run || count <= 0) return 0;
    WaveGroup<R> w;
    w.count = count;
    w.first[0] = 0;
    int wk = 1;
    int64_t total = 0, waves = 0;
    for (int i = 0; i < count; ++i) {
        w.g[i] = g[i];
        total += wave_tiles(g[i]);
        w.first[i + 1] = (int)total;
    }
    for (int i = 0; i < count; ++i) {
        const int k = wave_count((g[i].Kin * g[i].Kout + 15) / 16, total);
        wk = std::max(wk, k);
        waves += k * wave_tiles(g[i]);
    }
    // one launch has one wave count: apart, if that would be more than the chip
    // holds (8192 waves) for the sake of a member with few tiles
    if (count == 1 || (wk * total > 8192 && wk * total > 2 * waves)) {
        for (int i = 0; i < count; ++i) launch_wave(g[i], ws, s, nullptr);
        return count;
    }
    const dim3 grid((unsigned)total);
    if (wk == 16)
        hipLaunchKernelGGL((k_cgemm_wave_group<R, 16>), grid, dim3(1024), 0, s, w);
    else if (wk == 8)
        hipLaunchKernelGGL((k_cgemm_wave_group<R, 8>), grid, dim3(512), 0, s, w);
    else if (wk == 4)
        hipLaunchKernelGGL((k_cgemm_wave_group<R, 4>), grid, dim3(256), 0, s, w);
    else
        hipLaunchKernelGGL((k_cgemm_wave_group<R, 1>), grid, dim3(64), 0, s, w);
    return 1;
}

template <typename R>
bool cgemm(const Gemm<R>& g, const GemmScratch& ws, hipStream_t s, char* why, int whylen, hipEvent_t ev0,
           hipEvent_t ev1, CgemmInfo* info) {
    if (info) *info = CgemmInfo{};
    if (g.M <= 0 || g.N <= 0 || g.B1 * g.B2 <= 0) return true;
    if (!cgemm_check(g, ws, why, whylen)) return false;
    if (g_dry_run) return true;
    const int K = g.Kin * g.Kout;
    const int64_t nbatch = (int64_t)g.B1 * g.B2;
    const bool a_k = g.sak == 1 && g.sam != 1, b_k = g.sbk == 1 && g.sbn != 1;
    const double flops = 8.0 * g.M * g.N * (double)K * (double)nbatch;
    // Tile kernels: the one with the least padded work over its rate (relative
    // rates measured on shapes without padding).  Launches bound by latency
    // and K = 0 take the wave-sliced kernel.
    struct Choice {
        int bm, bn;
        double rate;
    };
    auto best = [&](std::initializer_list<Choice> cs) {
        Choice b{0, 0, 0.0};
        double cost = 0.0;
        for (const Choice& c : cs) {
            const double t = padded(g.M, g.N, c.bm, c.bn) / c.rate;
            if (b.bm == 0 || t < cost) {
                b = c;
                cost = t;
            }
        }
        return b;
    };
    if (ev0) (void)hipEventRecord(ev0, s);
    if (K == 0 || takes_wave(g)) {
        // where it would split K over the grid (K >= 1024 over few tiles) and B lies
        // along k, its reads of B are not contiguous: ragged tiles, staged through
        // LDS (FP64, 85 x 117 outputs, K = 1360 21.8 us wave-sliced, 14.2 ragged; FP32,
        // 64 x 96, K = 1088 14.4 / 10.3)
        if (K > 0 && b_k && g.M >= 32 && g.N >= 32 && wave_splits(g, ws) > 1)
            launch_ragged(g, ws, s, true, a_k, b_k, info);
        else
            launch_wave(g, ws, s, info);
        if (ev1) (void)hipEventRecord(ev1, s);
        return true;
    }
    const bool mfma_ok = aligned_form(g);
    if constexpr (sizeof(R) == 4) {
        // BF16x3 mode: outputs of at least one 128 x 128 tile whose inner extent
        // is a multiple of 32, where two blocks in four CUs have work; every
        // other shape is FP32
        const Choice t = best({{128, 128, 1.0}, {64, 128, 0.92}, {128, 64, 0.92}});
        const int64_t tiles128 = (int64_t)((g.M + 127) / 128) * ((g.N + 127) / 128) * nbatch;
        const bool bf16 = g.split && mfma_ok && g.M >= 128 && g.N >= 128 && g.Kin % 32 == 0 &&
                          tiles128 * split_factor(g, ws, tiles128, K / 16, 256, 4) >= 128;
        // FP32 alternatives on the FP32 matrix cores: the aligned tiles (three
        // products), or the ragged tiles (four), which do not pad every outer index
        // to a whole k-tile as k_cgemm_split does (256 x 256 x 20 node, parent-leg sum
        // over five 35.9 us split / 30.1 ragged; 20 x 256 x 128, left-leg sum over 33
        // 102 / 78); below 1 Gflop their shorter
        // prologue wins (64^3 node, right-leg stack of four, 0.54 Gflop: 10.7 us
        // against 13.8; 96^3, left-leg stack of five, 3.4 Gflop: 44.5
        // against 35.7; 208 x 208 x 144, parent-leg sum over three: 305 against
        // 163 with 128 x 64 tiles)
        const Choice f = best(mfma_ok ? std::initializer_list<Choice>{{64, 64, 0.55}, {32, 32, 0.44}}
                                       : std::initializer_list<Choice>{{64, 64, 0.40}, {32, 32, 0.36}});
        const double kpad = (double)((g.Kin + 15) / 16 * 16) / g.Kin;
        const double tf = padded(g.M, g.N, f.bm, f.bn) / f.rate, ts = padded(g.M, g.N, t.bm, t.bn) / t.rate * kpad;
        if (bf16 || (flops >= SPLIT_MIN_FLOPS && ts < tf)) {
            launch_split(g, ws, s, bf16 ? 2 : 3, a_k, b_k, info);
            if (ev1) (void)hipEventRecord(ev1, s);
            return true;
        }
    }
    if (!mfma_ok) {
        // 32 x 32 tiles where 64 x 64 ones compute much more padding (FP64, 81 x
        // 81 outputs: 103 us with 32, 138 with 64; 250 x 10000 outputs: 341 / 329)
        launch_ragged(g, ws, s, best({{64, 64, 1.0}, {32, 32, 0.9}}).bm == 32, a_k, b_k, info);
        if (ev1) (void)hipEventRecord(ev1, s);
        return true;
    }
    launch_aligned(g, ws, s, a_k, b_k, info);
    // the timing window closes after the split-K reduction: a launch's time
    // is the main kernel plus its reduction
    if (ev1) (void)hipEventRecord(ev1, s);
    return true;
}

// Sampling's contractions with the pass beside them folded in (k_cgemm_mfma's
// FUSE).  Both take whole k-tiles and the layouts they state; the caller asks
// cgemm_fusable first and checks g as for cgemm.
bool cgemm_fusable(const Gemm<double>& g) { return aligned_form(g) && g.B1 * g.B2 == 1; }

// C[m, n] = sum A[m, (kin, kout)] B[kin, n] f[kout, n]; A and B contiguous along
// k_in, f planar, contiguous along k_out
int cgemm_outer(const Gemm<double>& g, const double* f, int64_t f_plane, int64_t sfn, const GemmScratch& ws,
                hipStream_t s) {
    typedef double R;
    if (g_dry_run || g.M <= 0 || g.N <= 0) return 1;
    const AlignedPlan p = plan_aligned(g, ws);
    MfmaExtra<R> x;
    x.f = f;
    x.f_plane = f_plane;
    x.sfn = sfn;
    if (p.groups == 4)
        TTN_MFMA_LAUNCH(32, 32, 2, 2, 4, 1, true, true, MFMA_OUTER);
    else if (p.groups == 2)
        TTN_MFMA_LAUNCH(32, 32, 2, 2, 2, 2, true, true, MFMA_OUTER);
    else if (p.small)
        TTN_MFMA_LAUNCH(32, 32, 2, 2, 1, 4, true, true, MFMA_OUTER);
    else if (!p.big)
        TTN_MFMA_LAUNCH(64, 64, 2, 4, 1, 2, true, true, MFMA_OUTER);
    else
        TTN_MFMA_LAUNCH(128, 64, 4, 4, 1, 1, true, true, MFMA_OUTER);
    if (p.splits > 1) splitk_reduce(g, p.splits, (const R*)ws.partial, s);
    return p.splits;
}

// C = A B (A contiguous along m, B along k_in) and norms[n][tm] = sum over the
// 64 rows of tile row tm of |C[m, n]|^2
int cgemm_norms(const Gemm<double>& g, double* norms, hipStream_t s) {
    typedef double R;
    if (g_dry_run || g.M <= 0 || g.N <= 0) return 1;
    const GemmScratch ws;
    AlignedPlan p{};
    p.splits = 1;
    p.kchunk = g.Kin * g.Kout;
    p.blocks = tile_count(g, 64, 64);
    MfmaExtra<R> x;
    x.norms = norms;
    TTN_MFMA_LAUNCH(64, 64, 2, 4, 1, 2, false, true, MFMA_NORMS);
    return 1;
}
#undef TTN_MFMA_LAUNCH

template bool cgemm_check<double>(const Gemm<double>&, const GemmScratch&, char*, int);
template bool cgemm_check<float>(const Gemm<float>&, const GemmScratch&, char*, int);
template bool cgemm_groupable<double>(const Gemm<double>&, const GemmScratch&);
template bool cgemm_groupable<float>(const Gemm<float>&, const GemmScratch&);
template int cgemm_group<double>(const Gemm<double>*, int, const GemmScratch&, hipStream_t);
template int cgemm_group<float>(const Gemm<float>*, int, const GemmScratch&, hipStream_t);
template bool cgemm<double>(const Gemm<double>&, const GemmScratch&, hipStream_t, char*, int, hipEvent_t,
                            hipEvent_t, CgemmInfo*);
template bool cgemm<float>(const Gemm<float>&, const GemmScratch&, hipStream_t, char*, int, hipEvent_t,
                           hipEvent_t, CgemmInfo*);

}  // namespace ttn
