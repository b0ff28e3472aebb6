// Internal interfaces of the TTN/TDVP device library (gfx950).
//
// Storage convention: a complex array of n elements is n real parts followed
// by n imaginary parts ("planar"); stacks of such arrays are concatenated,
// so slot k of a stack of n-element arrays starts at 2*n*k.
#pragma once

#include <hip/hip_runtime.h>

#include <initializer_list>

#include <cstdint>

namespace ttn {

constexpr int KRYLOV_MAX = 16;

// Strided, batched, planar-complex GEMM:
//   C[m, n] = alpha * sum_k opA[m, k] opB[k, n] + beta * C[m, n]
// with k = k_in + Kin * k_out (two-level contraction index) and batch
// b = b1 + B1 * b2.  Offsets are in real elements; *_plane is the distance
// from a real part to its imaginary part.
template <typename R>
struct Gemm {
    int M = 0, N = 0, Kin = 1, Kout = 1, B1 = 1, B2 = 1;
    const R* A = nullptr;
    int64_t a_plane = 0, sam = 0, sak = 0, sako = 0, sab1 = 0, sab2 = 0;
    bool conjA = false;
    const R* B = nullptr;
    int64_t b_plane = 0, sbk = 0, sbko = 0, sbn = 0, sbb1 = 0, sbb2 = 0;
    bool conjB = false;
    R* C = nullptr;
    int64_t c_plane = 0, scm = 0, scn = 0, scb1 = 0, scb2 = 0;
    R alpha = 1;
    int beta = 0;                 // 0 overwrite, 1 accumulate
    const int* skip = nullptr;    // device flag: launch is a no-op when set
    int split = 0;                // FP32 only: products from bf16 hi/lo splits (BF16x3)
};

// A device allocation [lo, hi) of the workspace, for launch extent checks.
struct Region {
    uintptr_t lo, hi;
};

// Scratch for split-K partial sums (real elements) owned by the engine, and
// the table of workspace regions every GEMM operand must stay inside.
struct GemmScratch {
    void* partial = nullptr;
    int64_t bytes = 0;
    const Region* regions = nullptr;   // sorted by lo
    int n_regions = 0;
};

// What a cgemm call launched: the kernel (2 a matrix-core kernel in the
// operands' precision -- k_cgemm_wave, k_cgemm_mfma, or k_cgemm_split with three
// pieces -- 3 k_cgemm_split with two pieces, the BF16x3 products) and the
// split-K factor (> 1: a k_splitk_reduce* launch follows).
struct CgemmInfo {
    int kernel = 0;
    int splits = 0;
};

// Validates every operand extent against the region table and launches.
// Returns false (and launches nothing) when an operand would leave its
// region; `why` receives a description.  ev_begin / ev_end (optional) are
// recorded before the main kernel and after its split-K reduction.
template <typename R>
bool cgemm(const Gemm<R>& g, const GemmScratch& ws, hipStream_t s, char* why, int whylen,
           hipEvent_t ev_begin = nullptr, hipEvent_t ev_end = nullptr, CgemmInfo* info = nullptr);

// The extent check of cgemm alone.
template <typename R>
bool cgemm_check(const Gemm<R>& g, const GemmScratch& ws, char* why, int whylen);

// Whether cgemm may write C over the operand it replaces: over A (same rows m, C's
// n on A's k) or over B (same columns n, C's m on B's k), K = N or M.
bool cgemm_in_place(const Gemm<double>& g, const GemmScratch& ws, bool over_a);

// Contractions of the sampling walk with the pass beside them folded in (see
// contract.hip); usable when cgemm_fusable(g).  They return the split-K factor.
bool cgemm_fusable(const Gemm<double>& g);
int cgemm_outer(const Gemm<double>& g, const double* f, int64_t f_plane, int64_t sfn, const GemmScratch& ws,
                hipStream_t s);
int cgemm_norms(const Gemm<double>& g, double* norms, hipStream_t s);

// Independent short contractions (cgemm_groupable: those that cgemm would give
// to the wave-sliced kernel without split K) in one launch, for sequences
// whose cost is their launches.  The caller has checked their extents and that
// none reads or writes what another writes.  Returns the launches made.
constexpr int GROUP_MAX = 6;
template <typename R>
bool cgemm_groupable(const Gemm<R>& g, const GemmScratch& ws);
template <typename R>
int cgemm_group(const Gemm<R>* g, int count, const GemmScratch& ws, hipStream_t s);

// When set, launchers validate but enqueue nothing (plan checking without a
// device).
extern bool g_dry_run;

// Lanczos state kept on the device so that no host round trip is needed.
struct LanczosDev {
    double beta0;
    double alpha[KRYLOV_MAX];
    double beta[KRYLOV_MAX];
    double c[2 * KRYLOV_MAX];
    int m_eff;
    int done;
    int zero;
    int nonherm;     // Arnoldi: keep the whole Hessenberg projection in hs
    // hs[2 (j KRYLOV_MAX + i)] = H[i][j] (re, im) for i <= j (Arnoldi only;
    // the subdiagonal is beta)
    double hs[2 * KRYLOV_MAX * KRYLOV_MAX];
};

// Step-level device flags and statistics.
struct StepDev {
    int bad;                 // non-zero after a failed Cholesky pivot / NaN
    int min_krylov;
    unsigned long long min_rdiag_bits;   // positive double as ordered bits
    unsigned long long max_disc_bits;    // non-negative double as ordered bits
    double scratch[8];
};

// Krylov bases of the general Lanczos path are stored in chunks of KCH
// elements: element i of slot k, plane p (0 re, 1 im) at
// (i / KCH) S + (2 k + p) KCH + i % KCH, with chunk stride S = 2 KCH (slots);
// a projection pass then reads one contiguous stretch per chunk rather than
// 2 (k + 1) separate streams (measured 6.0 against 4.7 TB/s on 12 vectors of
// 2^21 elements).  S = 0 marks a planar vector (slot stride 2 n).
constexpr int KCH = 256;
__host__ __device__ inline int64_t kch_ofs(int64_t i, int64_t S) { return (i / KCH) * S + (i % KCH); }
// element e < 2 n of a planar vector (e >= n: imaginary part) in a chunked slot
__host__ __device__ inline int64_t kch_elem(int64_t e, int64_t n, int64_t S) {
    const int64_t p = e >= n ? 1 : 0;
    return kch_ofs(e - p * n, S) + p * KCH;
}
inline int64_t kch_pad(int64_t n) { return (n + KCH - 1) / KCH * KCH; }
// planar copy of the first `slots` vectors of a chunked basis
void krylov_unchunk(const double* V, int64_t S, int64_t n, int slots, double* out, const int* skip, hipStream_t s);

// reductions / vector kernels (double master vectors)
// nonherm != 0 starts an Arnoldi basis (non-Hermitian operator): the
// projections of both Gram-Schmidt passes are kept as Hessenberg columns and
// lz_expm exponentiates the Hessenberg matrix instead of the tridiagonal one
// v0f, v0p != nullptr also receive v0 in FP32 or planar FP64 (the next matvec's input)
// v0 planar (S == 0) or slot 0 of a chunked basis
void lz_start(const double* x, int64_t n, double* v0, int64_t S, LanczosDev* lz, double* partial, int nb,
              hipStream_t s, int nonherm = 0, float* v0f = nullptr, double* v0p = nullptr);
// Reductions over at most LZ_FUSE_NB blocks may take their totals inside the
// next kernel of the iteration (every block sums the block partials itself),
// which saves the one-block total kernels; their partials alternate between
// `partial` and partial + LZ_PARTIAL_HALF (the reduction buffer holds both).
constexpr int LZ_FUSE_NB = 256;
constexpr int64_t LZ_PARTIAL_HALF = (int64_t)LZ_FUSE_NB * 2 * KRYLOV_MAX;
// c = V^H w; y0 != nullptr: w is first written as the sum of the matvec outputs
// y0, y1, y2 (y1, y2 may be null; y0 may be w itself).  total = false leaves the
// projections as block partials for a fused lz_subtract_project.
// V: chunked basis (chunk stride S) or planar vectors (S == 0); vnext: a slot of V
template <typename R>
void lz_project(const double* V, int64_t S, int kcount, double* w, int64_t n, double* partial, int nb, LanczosDev* lz,
                int alpha_index, hipStream_t s, const R* y0, const R* y1, const R* y2, bool total);
// w -= V c, then c <- V^H w (second Gram-Schmidt pass), fused
void lz_subtract_project(const double* V, int64_t S, int kcount, double* w, int64_t n, double* partial, int nb,
                         LanczosDev* lz, hipStream_t s, bool fuse = false);
// w -= V c, then beta_j = ||w||, breakdown test, v_{j+1} = w / beta_j
void lz_subtract_next(const double* V, int64_t S, int kcount, double* w, int64_t n, double* vnext, LanczosDev* lz,
                      int j, double* partial, int nb, double tol, hipStream_t s, float* vnextf = nullptr,
                      bool fuse = false, double* vnextp = nullptr);
// Operators of at most LZ_BLOCK_N entries keep a planar basis and run the
// whole iteration between two matvecs (projection, two Gram-Schmidt passes,
// beta_j and breakdown, v_{j+1}) in one block.  The matvec output is y0 + y1 + y2
// (y1, y2 may be null); x / xf (may be null): v_{j+1} for the next matvec, in
// FP64 / FP32.
constexpr int64_t LZ_BLOCK_N = 1536;
void lz_start_block(const double* x, int64_t n, double* v0, LanczosDev* lz, hipStream_t s, int nonherm, double* x0,
                    float* xf);
template <typename R>
void lz_iter(double* V, int j, int m, const R* y0, const R* y1, const R* y2, int64_t n, LanczosDev* lz, double tol,
             double* x, float* xf, hipStream_t s);
// out_q = |x| V exp(-i tau_q H_m) e_1 for every tau (outputs 2 n apart, at most
// LZ_TAUS); V planar (S == 0) or chunked with stride S; fill: x = 0 writes zeros
// (else out is left alone)
constexpr int LZ_TAUS = 8;
void lz_expm_combine(const double* V, int64_t S, int64_t n, double* out, const LanczosDev* lz,
                     std::initializer_list<double> taus, bool fill, StepDev* st, hipStream_t s);
// x <- exp(-i tau Op) x in one workgroup for small operators (the four
// matvec stages, Krylov recursion with two Gram-Schmidt passes, exponential
// and recombination, all in LDS, FP64): usable when n = DL DR DP <=
// SMALL_EVOLVE_N and small_evolve_doubles(...) <= SMALL_EVOLVE_POOL.
// L: [1 + sL] left stack; R: right stack (only its N_j slots are read, and
// only when W != nullptr); B: [1 + sL] right-leg stack or nullptr; W:
// [1 + sL + sR] parent-leg stack or nullptr (the root).
constexpr int64_t SMALL_EVOLVE_N = 1024;
constexpr int SMALL_EVOLVE_POOL = 16384;   // doubles of LDS for vectors and stacks
int64_t small_evolve_doubles(int DL, int DR, int DP, int sL, int sR, int m, bool hasB, bool hasW);
void small_evolve(const double* L, const double* R, const double* B, const double* W, int DL, int DR, int DP,
                  int sL, int sR, int m, double tau, double tol, bool nonherm, double* x, StepDev* st,
                  hipStream_t s);

// conversions and copies
// several FP64 -> FP32 conversions in one launch (null or empty items
// skipped); an item with eye = D > 0 writes the planar D x D identity
// (count 2 D^2) instead of converting x
struct D2FItem {
    const double* x;
    float* y;
    int64_t count;
    int eye = 0;
};
constexpr int D2F_MAX = 10;
struct D2FBatch {
    const double* x[D2F_MAX];
    float* y[D2F_MAX];
    int64_t c[D2F_MAX];
    int eye[D2F_MAX];
    int n;
};
void convert_d2f_many(std::initializer_list<D2FItem> items, const int* skip, hipStream_t s);
void copy_d(const double* x, double* y, int64_t count, const int* skip, hipStream_t s);
void transpose_c(const double* x, double* y, int rows, int cols, hipStream_t s);
void fill_zero_d(double* y, int64_t count, hipStream_t s);
// out_k = (in_k + in_k^H) / 2 for `count` planar D x D FP32 matrices, into FP64;
// with raw_first the first matrix is converted unchanged (a non-Hermitian block)
void herm_f2d(const float* in, double* out, int D, int count, hipStream_t s, bool raw_first = false);
// dst = sum_{k < count} src_k for planar D x D FP64 matrices stored one after another
void sum_mats(const double* src, int D, int count, double* dst, hipStream_t s);

// Eigenvalues (descending, w[k]) and eigenvectors (columns order[k] of V) of
// a Hermitian n x n matrix A (planar, column-major) of any scale, n <= JAC_NMAX,
// by cyclic block Jacobi; st->bad when it does not converge.  work:
// herm_eig_work(n) doubles.
constexpr int JAC_NMAX = 256;
int64_t herm_eig_work(int n);
void herm_eig(const double* A, int n, double* V, double* w, int* order, double* work, StepDev* st, hipStream_t s);
// dst[c dc + s ds + p dp] = (conj) src[c sc + s ss + p sp], c < K, s < S, p < P
void copy3(const double* src, int64_t src_plane, int64_t sc, int64_t ss, int64_t sp, double* dst, int64_t dst_plane,
           int64_t dc, int64_t ds, int64_t dp, int K, int S, int P, bool conj, hipStream_t s);
// out[:, c] = V[:, order[c]], c < k
void gather_cols(const double* V, int n, const int* order, int k, double* out, hipStream_t s);
// scales the centre x (count complex) of a split by sqrt(total / kept) of the
// descending Gram eigenvalues w (n of them, k kept); records the discarded
// weight 1 - kept / total in st->max_disc_bits
void split_finish(const double* w, int n, int k, double* x, int64_t count, StepDev* st, hipStream_t s);

// The whole gauge move (CholeskyQR2) of a small tensor on one of its legs in one
// launch: T <- Q, Rout = R, and (rinvh != nullptr) R^{-H}; usable when
// qr_small_fits.
bool qr_small_fits(int DL, int DR, int DP, int leg);
void qr_small(double* T, int DL, int DR, int DP, int leg, double* Rout, double* rinvh, StepDev* st, hipStream_t s);
// Cholesky of a Hermitian D x D Gram matrix G (planar, column-major):
// G = L L^H.  Writes Linv (lower, L^{-1}) and R = L^H (upper).  Rfirst: the R
// of the gauge move's first factorization when this is its second (G near I);
// min over k of R[k][k] Rfirst[k][k] then goes into st->min_rdiag_bits.  Sets
// st->bad on a non-positive pivot.  work: 2 Dp^2 doubles (Dp = 16 ceil(D / 16))
// for D <= 128, else D (D + 1) + 32 D.
void chol_inv(const double* G, int D, double* Linv, double* R, const double* Rfirst, double* work,
              StepDev* st, hipStream_t s);

// out[p] = sum_{l,r} a[l] b[r] T[l, r, p] (planar complex vectors); used for
// overlaps with product states.
void contract_node_vec(const double* T, int DL, int DR, int DP, const double* a, const double* b,
                       double* out, hipStream_t s);

}  // namespace ttn
