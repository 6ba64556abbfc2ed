// Device-side views and kernel launchers of the shell multigrid (gfx950).
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

namespace mgk {

// The couplings one step of a column sweep needs, in the order a wavefront
// walks its half of the column: record t of direction dir (0: upward from
// layer 0, 1: downward from layer nz-1) and row J is that of layer
// k = dir ? nz-1-t : t (clamped to [0, nz-1]): Tlam[k][J], Tth[k][J],
// Tth[k][J+1], and tc, the vertical coupling to the next layer in that
// direction (Tr[k+1][J] upward, Tr[k][J] downward). Table layout
// [dir][J][t], step_stride(nz) records per row: as many as the layers, and
// as the padded steps of the compiled sweeps and their lanes reach (64).
template <typename T>
struct alignas(4 * sizeof(T)) StepCoef {
    T tl, ts, tn, tc;
};
inline int step_stride(int nz) { return nz <= 72 ? 72 : (nz + 7) / 8 * 8; }

// Geometry and operator data of one level, in the precision T of the kernels
// that read it. Fields are [k][J][i] with i fastest; plane = nI*nJ.
template <typename T>
struct LevelView {
    int nI, nJ, nz;
    long long plane;
    const T* Tlam;   // [nz][nJ]
    const T* Tth;    // [nz][nJ+1], face F south of row F
    const T* Tr;     // [nz+1][nJ], face F below layer F
    const T* M;      // [nz][plane] mass sum(alpha V)
    const T* invp;   // [nz][plane] inverse pivots of the twisted factorisation of H_z
    const StepCoef<T>* sc;   // [2][nJ][scs] step records (see StepCoef)
    int scs;
};

// Maps between a fine level and the next coarser one.
template <typename T>
struct TransferView {
    int nIc, nJc;
    const int* crow_of;      // [nJf]   coarse row of each fine row
    const int* prow;         // [2nJf]  latitude rows used by P
    const T* pw;             // [2nJf]  their weights
    const int* child_first;  // [nJc]   first fine row of each coarse row
    const int* child_count;  // [nJc]   1 or 2
    const int* ptrow;        // [4nJc]  fine rows gathered by P^T (-1 unused)
    const T* ptw;            // [4nJc]
};

constexpr int kBlock = 256;

inline int blocks_for(long long n) { return int((n + kBlock - 1) / kBlock); }

// --- launchers (all asynchronous on `s`) ---------------------------------

// y = H x, or y = f - H x when f != nullptr (difference form).
template <typename T>
void apply(const LevelView<T>& L, const T* x, const T* f, T* y, hipStream_t s);

// One damped block-Jacobi sweep (Eq. 1):
//   xout = (1-omega) xin + omega H_z^{-1}(f + sum_h T_h xin_nb),
// or the sweep from zero xout = omega H_z^{-1} f when xin == nullptr.
// Levels with fewer than staged_columns columns use the staged kernel.
template <typename T>
void smooth(const LevelView<T>& L, const T* f, const T* xin, T* xout, T omega,
            long long staged_columns, hipStream_t s);

// One staged sweep from xin + P xc (the first after a coarse-grid
// correction) on small levels of few layers (prolongs_in_sweep; false,
// launching nothing, elsewhere).
template <typename T>
bool prolongs_in_sweep(const LevelView<T>& L, long long staged_columns);
template <typename T>
bool smooth_prolonged(const LevelView<T>& L, const TransferView<T>& X, const T* f, const T* xin,
                      const T* xc, T* xout, T omega, long long staged_columns, hipStream_t s);

// The same sweep with the kernel for levels that fill the GPU (k_sweep.hip),
// which smooth() uses on every level it does not stage.
template <typename T>
void sweep(const LevelView<T>& L, const T* f, const T* xin, T* xout, T omega, hipStream_t s);

// Two consecutive sweeps (factors om1, om2; the first from zero when xin ==
// nullptr) in one pass, for levels of at least kPairColumns columns with 17 to
// 72 layers, but for some with short rows (sweep_pair_fits; false, launching
// nothing, elsewhere). A block walks a band of rows, three phases longer than the
// band, so a level needs enough rows per CU: with 70 layers, V(2,2) cycles of two
// levels take 431 us against 485 for single sweeps on 768x384, 180 against 189 on
// 384x288 (110,592 columns), 137 against 138 on 384x192. With 38 layers on
// 1152x768 626 against 1046 us. Short columns leave little to share: V(2,4)
// cycles of 1280x780 take 816 against 1049 us with 18 layers, 839 against 773
// with 16 and 744 against 725 with 14 (1536x710x16: 811 against 840).
constexpr long long kPairColumns = 3LL << 15;
bool sweep_pair_fits(const LevelView<float>& L, size_t max_lds);
bool sweep_pair(const LevelView<float>& L, const float* f, const float* xin, float* xout,
                float om1, float om2, size_t max_lds, hipStream_t s);

// Layer and row factors of a level's couplings (FP64):
// Tlam[k][J] = h[k] gl[J], Tth[k][F] = h[k] gt[F], Tr[F][J] = v[F] gr[J].
struct SepView {
    const double *h = nullptr, *v = nullptr, *gl = nullptr, *gt = nullptr, *gr = nullptr;
};

// The whole coarsest-level solve (`sweeps` sweeps from zero, result in x) in
// one launch of one block with the level in its LDS. Returns false,
// launching nothing, where the level does not fit (coarse_solve_fits).
template <typename T>
bool coarse_solve_fits(long long plane, int nJ, int nz, size_t max_lds);
template <typename T>
bool coarse_solve(const LevelView<T>& L, const T* f, T* x, T omega, int sweeps, size_t max_lds,
                  hipStream_t s);

// The coarsest-level solve is a linear map x = C f of the level's n cells, and
// a symmetric one. coarse_basis writes C row by row (row j is the solve applied
// to the j-th unit vector), computed in FP64, into C and rounded to FP32 into
// C32 (n*n values each). Returns false, launching nothing, where the level has
// more than kDenseCoarseMax cells or kDenseCoarseColumns columns or does not
// fit in max_lds bytes of LDS (coarse_basis_fits).
constexpr long long kDenseCoarseMax = 6144;
constexpr long long kDenseCoarseColumns = 128;
bool coarse_basis_fits(long long plane, int nJ, int nz, size_t max_lds);
bool coarse_basis(const LevelView<double>& L, const SepView& sep, double* C, float* C32,
                  double omega, int sweeps, size_t max_lds, hipStream_t s);

// x = A f for an n x n row-major matrix: one wavefront per row, partial sums
// in a fixed order (results are reproducible).
template <typename T>
void dense_matvec(const T* A, long long n, const T* f, T* x, hipStream_t s);

// fc = R (f - H x) (sum over children), or R f when x == nullptr.
template <typename T>
void restrict_residual(const LevelView<T>& F, const TransferView<T>& X, const T* f,
                       const T* x, T* fc, hipStream_t s);

// x += P xc (bilinear, cell-centred).
template <typename T>
void prolong_add(const LevelView<T>& F, const TransferView<T>& X, const T* xc, T* x,
                 hipStream_t s);

// xc = P^T x.
template <typename T>
void prolong_transpose(const LevelView<T>& F, const TransferView<T>& X, const T* x,
                       T* xc, hipStream_t s);

// x += R^T xc (every child cell takes its coarse parent's value).
template <typename T>
void inject_add(const LevelView<T>& F, const TransferView<T>& X, const T* xc, T* x,
                hipStream_t s);

// Block counters of the refinement step: one of the groups of blocks, and one
// per group, a cache line apart.
constexpr unsigned kDoneGroup = 64, kDoneStride = 32;
inline size_t done_values(int blocks) {
    return size_t(kDoneStride) * (1 + (size_t(blocks) + kDoneGroup - 1) / kDoneGroup);
}

// Refinement step on the finest level, in the iterate's precision TU (FP64;
// FP32 in the pure single-precision solve):
//   unew = uin + e (or uin when e == nullptr), written to uout if set;
//   r = b - H unew, stored as TR; the sums of r^2 (and of b^2 when partials_b
//   is not null) in FP64 into norms[0] (norms[1]), host memory, through
//   per-block partial sums; done counts the blocks (done_values(blocks) values,
//   0 before and after).
// uin == nullptr stands for a zero iterate (a solve from u = 0): it is not
// read, and with e == nullptr as well the step is r = b.
// It has residual_update_blocks(L) blocks, hence partial sums.
template <typename TU, typename TE, typename TR>
void residual_update(const LevelView<TU>& L, const TU* b, const TU* uin, const TE* e, TU* uout,
                    TR* r, double* partials, double* partials_b, unsigned* done, double* norms,
                    hipStream_t s);
template <typename TU>
int residual_update_blocks(const LevelView<TU>& L);
// Row tiles of it (blocks per range of layers).
template <typename TU>
int residual_tiles(const LevelView<TU>& L);

// *out = sum of the n partials in a fixed order.
void sum_partials(const double* partials, int n, double* out, hipStream_t s);

// Setup: M = alpha * V (fine level; not written when M is null) and
// per-block counts of alpha values that are not finite and > 0 (as FP64
// partials).
int fine_mass(const LevelView<double>& L, const double* V, const double* alpha,
              double* M, double* partials, hipStream_t s);
// Setup: row-sum pivots of the twisted factorisation of H_z (eliminated from
// both ends toward layer nz/2); inverse pivots in FP64 and FP32 and an FP32
// copy of M.
void pivots(const LevelView<double>& L, double* invp64, float* invp32, float* M32,
            hipStream_t s);

void grad_alpha(const LevelView<double>& L, const double* V, const double* lam,
                const double* u, double* g, hipStream_t s);
void cell_volumes(const LevelView<double>& L, const double* V, double* out, hipStream_t s);
template <typename TA, typename TB>
void cast(const TA* in, TB* out, long long n, hipStream_t s);
template <typename T>
void fill(T* out, T v, long long n, hipStream_t s);

}  // namespace mgk
