// Operator apply, the FP64 refinement step (update + residual + norm), the
// deterministic reductions, and the setup / elementwise kernels.
//
// H is always evaluated in difference form (paper Section 2: Hu with H a
// Laplacian-like matrix):
//   (H x)_c = sum_faces T_f (x_c - x_nb) + M_c x_c.
#include "device.hpp"

namespace mgk {

constexpr int kResidualSync = 4;
// A k_residual_walk block has one wavefront per row of its tile of R
// consecutive rows: R = 16 where that still gives at least
// kResidualTallBlocks blocks, else R = 4 (small levels would leave CUs
// idle). Every kResidualSync layers the block's wavefronts meet at a
// barrier: an XCD's L2 holds only a layer or two of all resident wavefronts'
// rows, so the latitude neighbours a wavefront reads are L2 hits only while
// the wavefronts that own those rows are at about the same layer. Measured
// on the 1024x768x70 shell: 2.03 -> 1.70 GB fetched and 470 -> 448 us per
// launch against 4-row tiles without the barrier.
constexpr int kResidualTallBlocks = 512;
constexpr int kResidualTallRows = 16;
// The walking refinement step: a range of layers per wavefront (at most
// kResidualRange on large levels, shorter ones on smaller levels), the
// layers whose loads are in flight ahead of the one being computed, and the
// same row tiles and barrier interval as above. Measured per launch on the
// 1024x768x70 shell (mixed solve): 446 us with whole columns against 458 us
// with two ranges of 35 layers; loads 2 or 4 layers ahead 467 and 468 us
// against 446; barriers every 8 layers or none 454 and 459 us; longitude
// neighbours loaded instead of shifted from the neighbour lanes 489 us.
// 16-row and 4-row tiles are within 1 % there; on 2560x1920x70 16-row
// tiles take 2.78-2.90 ms against 2.99-3.07 ms (FP64: 3.54-3.59 against
// 3.82-3.83 ms).
//
// A column is cut into as few ranges as that allows and these are of equal
// length, because every XCD takes a contiguous part of the blocks: with 70 + 1
// layers the XCDs that got the last layer of 1024x768x71 waited for the others
// (FP64 740 us, 488 with 36 + 35). A walk ends with its range: steps for layers
// that are not there would issue their loads all the same (1024x768, FP64: 17
// layers 134 us against 268 with 70 steps, 38 layers 263 against 361; mixed 106
// against 204, 211 against 266).
constexpr int kResidualRange = 70;
constexpr int kResidualShortRange = 8;
constexpr int kResidualTinyRange = 4;
constexpr int kResidualAhead = 3;

static int residual_tile_rows(int nI, int nJ) {
    return dev::tiled_blocks(nJ, dev::segments_per_row(nI), kResidualTallRows) >=
                   kResidualTallBlocks
               ? kResidualTallRows
               : 4;
}

// Layers per walk: whole columns on levels with enough tall tiles to fill
// the GPU; ranges of kResidualShortRange layers on smaller levels, whose
// whole-column walks leave a few wavefronts per CU (384x192x70: 54 us with
// whole columns, 47.3 with ranges of 16 layers, 45.4 with 8 and with 4;
// 288x192x38 25.5, 22.8 and 23.4); of kResidualTinyRange on levels that give
// fewer than one block per CU otherwise (FP64 on 64x32x16: 8.4 us with 16
// layers, 6.2 with 8, 4.9 with 4).
static int residual_walk_range(int nI, int nJ, int nz) {
    if (residual_tile_rows(nI, nJ) == kResidualTallRows)
        return nz <= 16 ? 16 : kResidualRange;
    return (long long)dev::tiled_blocks(nJ, dev::segments_per_row(nI), 4) *
                       ((nz + kResidualShortRange - 1) / kResidualShortRange) < 256
               ? kResidualTinyRange
               : kResidualShortRange;
}

namespace {
using namespace dev;

// Rows per block of the operator kernel (64 columns x this many rows: each
// wavefront one row) and layers per lane (a lane walks a chunk of layers of
// its column: the chunk's loads are in flight together, and the vertical
// neighbours come from the layers it already loaded).
constexpr int kApplyRows = 4;
// (FP32 2: adjoint solves on 1024x768x70 0.5-0.9 % slower with 4; FP64 4:
// 0.6 % slower with 2)
template <typename T>
constexpr int apply_layers() {
    return std::is_same<T, float>::value ? 2 : 4;
}
// In FP64 large levels take the walk of the refinement step (MODE 1 and 2) in
// ranges of at most kApplyRange layers, which reads each column once per range.
// It pays where the level's three arrays exceed the 256 MB last-level cache
// (below that the chunks' second reads of a column are cheap) and the column
// is long enough for its pipeline. Whole calls, this kernel against the walk:
// 640x480x50 107 and 88 us, 1152x576x50 209 and 174, x20 95 and 88; about
// 12M cells 1024x768x15 83 and 80, 768x384x40 83 and 78, 512x512x44 75 and 76;
// below 1024x768x14 68 and 77, 640x640x24 66 and 69, 768x384x26 55 and 59;
// few layers 2560x1920x9 303 and 265, x8 228 and 243, x4 128 and 149.
// (Ranges of 16 or 50 layers on 640x480x50: 101 and 89 us a launch, 89 with 25,
// but 358 on 1024x768x70 with whole columns. On fewer columns, 384x192x70, 45
// us with the walk against 41.)
constexpr int kApplyRange = 25;
constexpr long long kApplyWalkColumns = 1LL << 18;
constexpr long long kApplyWalkCells = 3LL << 22;
constexpr int kApplyWalkLayers = 9;

// y = H x (HAS_F = false) or y = f - H x, one lane per column and chunk of
// apply_layers layers, in blocks of 64 columns x kApplyRows rows (grid:
// column groups, row groups, layer chunks): a wavefront takes part of one
// row, so the row's couplings are wave-uniform and no lane divides its index.
template <typename T, bool HAS_F>
__global__ __launch_bounds__(64 * kApplyRows) void k_apply(LevelView<T> L,
                                                           const T* __restrict__ x,
                                                           const T* __restrict__ f,
                                                           T* __restrict__ y) {
    constexpr int NL = apply_layers<T>();
    const int nI = L.nI, nJ = L.nJ, nz = L.nz;
    const int i = int(blockIdx.x) * 64 + int(threadIdx.x);
    const int J = __builtin_amdgcn_readfirstlane(int(blockIdx.y) * kApplyRows +
                                                 int(threadIdx.y));
    const int k0 = int(blockIdx.z) * NL;
    if (i >= nI || J >= nJ) return;
    const size_t P = size_t(L.plane);
    const uint32_t c = uint32_t(J) * uint32_t(nI) + uint32_t(i);
    const uint32_t w = (i == 0) ? c + uint32_t(nI - 1) : c - 1u;
    const uint32_t e = (i == nI - 1) ? c - uint32_t(nI - 1) : c + 1u;
    const uint32_t sth = (J > 0) ? c - uint32_t(nI) : c;
    const uint32_t nth = (J < nJ - 1) ? c + uint32_t(nI) : c;
    auto clampk = [nz](int k) { return k < 0 ? 0 : (k < nz ? k : nz - 1); };
    // the column at layers k0-1 .. k0+NL (clamped: a boundary layer is its
    // own vertical neighbour, and its coupling term vanishes)
    T xv[NL + 2];
#pragma unroll
    for (int d = 0; d < NL + 2; ++d) xv[d] = x[size_t(clampk(k0 - 1 + d)) * P + c];
    T hs[NL];
#pragma unroll
    for (int d = 0; d < NL; ++d) {
        const int k = clampk(k0 + d);
        const T* xk = x + size_t(k) * P;
        const size_t t = size_t(k) * P + c;
        const T xc = xv[d + 1];
        const T xm = (k0 + d > 0) ? xv[d] : xc;
        const T xp = (k0 + d + 1 < nz) ? xv[d + 2] : xc;
        const T h = L.M[t] * xc +
                    hdiff(L.Tlam[k * nJ + J], L.Tth[k * (nJ + 1) + J],
                          L.Tth[k * (nJ + 1) + J + 1], xc, xk[w], xk[e], xk[sth], xk[nth]) +
                    L.Tr[k * nJ + J] * (xc - xm) + L.Tr[(k + 1) * nJ + J] * (xc - xp);
        hs[d] = HAS_F ? f[t] - h : h;
    }
#pragma unroll
    for (int d = 0; d < NL; ++d)
        if (k0 + d < nz) y[size_t(k0 + d) * P + c] = hs[d];
}

// The block's partial sums (in `mine`, written by thread 0) and the sums over
// all blocks, by the block that finishes last: in the fixed order of the
// partials whichever block it is, written to norms[0] (and norms[1] with
// partials_b), which is host memory. That saves two launches per refinement
// step, the reduction and the copy of its result: 9 us of the 92 us of an
// iteration on 64x32x16.
// The partials are stored and read with agent scope, past the XCDs' own
// caches, and a block counts itself done only after its stores have been
// acknowledged. Blocks count in groups of kDoneGroup, each in a cache line of
// its own, and the last of a group counts the group: increments of one address
// wait for each other, about 16 ns each (384x192x70, 2592 blocks: a first step
// that only reads b and writes r 47 us with one counter, 25 now; FP32 steps 44
// and 32, FP64 51.7 and 50.4). The last block of a group and the last of all
// set their counts back to zero for the next step. One wavefront does all of
// it; the others leave.
__device__ __forceinline__ void sum_by_last_block(const double* mine, double* partials,
                                                  double* partials_b, unsigned* done,
                                                  double* norms) {
    if (threadIdx.x >= 64) return;   // the first wavefront's work from here on
    unsigned last = 0;
    if (threadIdx.x == 0) {
        __hip_atomic_store(partials + blockIdx.x, mine[0], __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        if (partials_b)
            __hip_atomic_store(partials_b + blockIdx.x, mine[1], __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        const unsigned g = blockIdx.x / kDoneGroup, first = g * kDoneGroup;
        const unsigned members = gridDim.x - first < kDoneGroup ? gridDim.x - first : kDoneGroup;
        unsigned* group = done + kDoneStride * (1 + g);
        if (__hip_atomic_fetch_add(group, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 ==
            members) {
            __hip_atomic_store(group, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const unsigned groups = (gridDim.x + kDoneGroup - 1) / kDoneGroup;
            if (__hip_atomic_fetch_add(done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 ==
                groups)
                last = 1;
        }
    }
    if (__builtin_amdgcn_readfirstlane(int(last)) == 0) return;
    for (int c = 0; c < (partials_b ? 2 : 1); ++c) {
        const double* p = c ? partials_b : partials;
        double a[4] = {0, 0, 0, 0};
        unsigned t = threadIdx.x;
        for (; t + 192 < gridDim.x; t += 256)
#pragma unroll
            for (int d = 0; d < 4; ++d)
                a[d] += __hip_atomic_load(p + t + 64 * d, __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_AGENT);
        for (; t < gridDim.x; t += 64)
            a[0] += __hip_atomic_load(p + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        double sum = (a[0] + a[1]) + (a[2] + a[3]);
        for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
        if (threadIdx.x == 0)
            __hip_atomic_store(norms + c, sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    if (threadIdx.x == 0)
        __hip_atomic_store(done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Refinement step on the finest level (MODE 0), in the precision TU of the
// iterate (FP64; FP32 in the pure single-precision solve):
//   unew = uin + e (HAS_E; written to uout), r = b - H unew (stored as TR),
//   per-block partial sums of r^2 in FP64, and of b^2 when partials_b is set;
// or the operator alone, r = H uin (MODE 1) or r = b - H uin (MODE 2), with no
// sums. It walks ranges of lr <= LR layers: block b takes range
// b / tiles and the tile of R consecutive rows of one 64-column range
// b % tiles (one wavefront per row), and each wavefront walks its layers
// upward with the loads of the next P layers in flight, the layers below and
// above coming from the steps before and after. A row's couplings are its
// upward step record. FULLI: nI is a multiple of 64, so a lane's longitude
// neighbours are its neighbour lanes' values, and only lanes 0 and 63 load
// theirs. Every S layers the block's wavefronts meet at a barrier, so that
// the latitude neighbours they read are still in L2. HAS_U false: the
// iterate before the update is zero (the first update of a solve from
// u = 0), and uin is not read.
template <typename TU, typename TE, typename TR, bool HAS_E, bool HAS_U, int LR, int P, int R,
          int S, bool FULLI, int MODE = 0>
__global__ __launch_bounds__(64 * R) void k_residual_walk(
    LevelView<TU> L, const TU* __restrict__ bv, const TU* __restrict__ uin,
    const TE* __restrict__ e, TU* __restrict__ uout, TR* __restrict__ r,
    double* partials, double* partials_b, int wpr, int tiles, int lr, unsigned* done,
    double* norms) {
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    const int blk = int(logical_block());
    const int rg = blk / tiles;
    const Seg g = tiled_segment(blk - rg * tiles, wave, R, L.nI, L.nJ, wpr);
    const int nz = L.nz, kb = rg * lr, ke = kb + lr < nz ? kb + lr : nz;
    const uint32_t PU = uint32_t(L.plane) * sizeof(TU), PE = uint32_t(L.plane) * sizeof(TE),
                   PR = uint32_t(L.plane) * sizeof(TR);
    const rsrc_t ru = make_rsrc(HAS_U ? uin : bv, PU * uint32_t(nz)),
                 rb = make_rsrc(MODE == 1 ? uin : bv, PU * uint32_t(nz)),
                 rm = make_rsrc(L.M, PU * uint32_t(nz)),
                 re = make_rsrc(HAS_E ? (const void*)e : (const void*)uin, PE * uint32_t(nz)),
                 rw = make_rsrc(HAS_E ? (const void*)uout : (const void*)uin, PU * uint32_t(nz)),
                 rr = make_rsrc(r, PR * uint32_t(nz));
    const bool lane0 = (threadIdx.x & 63u) == 0;
    const uint32_t gcol = FULLI ? (lane0 ? g.w : g.e) : 0u;
    const uint32_t uc = g.c * sizeof(TU), us = g.s * sizeof(TU), un = g.n * sizeof(TU),
                   uw = (FULLI ? gcol : g.w) * sizeof(TU), ue = g.e * sizeof(TU);
    const uint32_t ec = g.c * sizeof(TE), es = g.s * sizeof(TE), en = g.n * sizeof(TE),
                   ew = (FULLI ? gcol : g.w) * sizeof(TE), ee = g.e * sizeof(TE);
    const uint32_t rc = g.c * sizeof(TR);
    const StepCoef<TU>* qp = L.sc + size_t(g.J) * size_t(L.scs);

    // H is applied to a nonzero iterate (else r = b)
    constexpr bool HOP = HAS_U || HAS_E;
    // u + e at a cell of layer offsets (so_u, so_e); u = 0 without HAS_U
    auto un_at = [&](uint32_t ou, uint32_t oe, uint32_t so_u, uint32_t so_e) -> TU {
        TU v = TU(0);
        if constexpr (HAS_U) v = bld<TU>(ru, ou, so_u);
        if constexpr (HAS_E) v += TU(bld<TE>(re, oe, so_e));
        return v;
    };
    struct Lay {
        TU uc, us, un, uw, ue, b, m;
        TE ec, es, en, ew, ee;
        StepCoef<TU> q;
    };
    // the loads of step t (layer kb + t); only the column itself for the
    // layer above the range. Steps past the range load its last layers again
    // (cache hits), not those of the next range.
    auto fetch = [&](int t, bool column_only) {
        Lay Q;
        if constexpr (!HAS_E) Q.ec = Q.es = Q.en = Q.ew = Q.ee = TE(0);
        if constexpr (!HAS_U) Q.uc = Q.us = Q.un = Q.uw = Q.ue = TU(0);
        const int kc = clampk(kb + t < ke ? kb + t : ke, nz);
        const uint32_t cu = uint32_t(kc) * PU, ce = uint32_t(kc) * PE;
        if constexpr (HAS_U) Q.uc = bld<TU>(ru, uc, cu);
        if constexpr (HAS_E) Q.ec = bld<TE>(re, ec, ce);
        if (!column_only) {
            const int k = kb + t < ke ? kb + t : ke - 1;
            const uint32_t su = uint32_t(k) * PU, se = uint32_t(k) * PE;
            if constexpr (HAS_U) {
                Q.us = bld<TU>(ru, us, su);
                Q.un = bld<TU>(ru, un, su);
                Q.uw = bld<TU>(ru, uw, su);
                if constexpr (!FULLI) Q.ue = bld<TU>(ru, ue, su);
            }
            if constexpr (HAS_E) {
                Q.es = bld<TE>(re, es, se);
                Q.en = bld<TE>(re, en, se);
                Q.ew = bld<TE>(re, ew, se);
                if constexpr (!FULLI) Q.ee = bld<TE>(re, ee, se);
            }
            // b and the mass are read at the cell only: non-temporal loads
            if constexpr (MODE != 1) Q.b = bld<TU, true>(rb, uc, su);
            else Q.b = TU(0);   // (unused)
            if constexpr (HOP) {
                Q.m = bld<TU, true>(rm, uc, su);
                Q.q = step_rec(qp, size_t(k));
            }
        }
        return Q;
    };
    auto sum = [](TU u, TE x) -> TU {
        if constexpr (HAS_U && HAS_E) return u + TU(x);
        else if constexpr (HAS_E) return TU(x);
        else return u;
    };

    // the layer below the range, and its vertical coupling to the first
    // layer (0 at the bottom)
    const int kbm = kb > 0 ? kb - 1 : 0;
    const TU um0 = un_at(uc, ec, uint32_t(kbm) * PU, uint32_t(kbm) * PE);
    const TU tbm = step_rec(qp, size_t(kbm)).tc;
    TU um = um0, tb = kb > 0 ? tbm : TU(0);
    double acc = 0, accb = 0;
    Lay buf[P + 1];
#pragma unroll
    for (int t = 0; t < P; ++t) {
        __builtin_amdgcn_sched_barrier(0);
        buf[t] = fetch(t, t == LR);
    }
#pragma unroll
    for (int t = 0; t < LR; ++t) {
        __builtin_amdgcn_sched_barrier(0);
        if (t + P <= LR) buf[(t + P) % (P + 1)] = fetch(t + P, t + P == LR);
        __builtin_amdgcn_sched_barrier(0);
        const Lay& c = buf[t % (P + 1)];
        const Lay& a = buf[(t + 1) % (P + 1)];
        const TU xc = sum(c.uc, c.ec), xp = sum(a.uc, a.ec);
        const TU xs = sum(c.us, c.es), xn = sum(c.un, c.en);
        TU xw, xe;
        if constexpr (FULLI) {
            const TU edge = sum(c.uw, c.ew);
            xw = from_below(edge, xc);
            xe = from_above(edge, xc);
        } else {
            xw = sum(c.uw, c.ew);
            xe = sum(c.ue, c.ee);
        }
        TU rv = c.b;
        if constexpr (HOP) {
            const StepCoef<TU> q = c.q;
            const TU h = c.m * xc + hdiff(q.tl, q.ts, q.tn, xc, xw, xe, xs, xn) +
                         tb * (xc - um) + q.tc * (xc - xp);
            if constexpr (MODE == 1) rv = h;
            else rv -= h;
            tb = q.tc;
        }
        // computed here, not sunk (with its loads) into the guarded stores
        asm volatile("" : "+v"(rv));
        const int k = kb + t;
        if (k < ke && g.valid) {
            if constexpr (HAS_E) bst(xc, rw, uc, uint32_t(k) * PU);
            bst(TR(rv), rr, rc, uint32_t(k) * PR);
            if constexpr (MODE == 0) {
                acc += double(rv) * double(rv);
                accb += double(c.b) * double(c.b);
            }
        }
        um = xc;
        if (k + 1 >= ke) break;   // the same for every wavefront of the block
        if (t % S == S - 1) __syncthreads();
    }
    if constexpr (MODE == 0) {
        __shared__ double mine[2];
        if (partials_b) block_sum2_to(acc, accb, &mine[0], &mine[1]);
        else block_sum_to(acc, &mine[0]);
        sum_by_last_block(mine, partials, partials_b, done, norms);
    }
}

// One block sums the partials into *out.
__global__ __launch_bounds__(1024) void k_sum_partials(const double* __restrict__ p, int n,
                                                       double* __restrict__ out) {
    __shared__ double red[1024];
    double acc = 0;
    for (int t = threadIdx.x; t < n; t += blockDim.x) acc += p[t];
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int w = blockDim.x / 2; w > 0; w >>= 1) {
        if (int(threadIdx.x) < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = red[0];
}

// Setup: M = alpha V on the finest level; counts alpha values that are not
// finite and > 0.
__global__ __launch_bounds__(kBlock) void k_fine_mass(LevelView<double> L,
                                                      const double* __restrict__ V,
                                                      const double* __restrict__ alpha,
                                                      double* __restrict__ M, long long n,
                                                      double* __restrict__ partials) {
    double bad = 0;
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x; t < n; t += stride) {
        const int k = int(t / L.plane);
        const int J = int((t - k * L.plane) / L.nI);
        const double a = alpha[t];
        if (!(a > 0.0) || !isfinite(a)) bad += 1.0;
        if (M) M[t] = a * V[k * L.nJ + J];
    }
    block_sum_to(bad, partials + blockIdx.x);
}

// Setup: pivots of the twisted (two-sided) factorisation of H_z, per column.
// The column is eliminated from the bottom up to the layer below m = nz/2 and
// from the top down to the layer above it; layer m takes both. In row-sum
// form, with mt_k = M_k + 2 Tlam + Tth(south) + Tth(north) (the row sum of
// H_z at layer k) and Tr_F the coupling across face F (below layer F):
//   below m: g_0 = mt_0, g_k = mt_k + Tr_k g_{k-1} / (Tr_k + g_{k-1}),
//            stored 1 / (Tr_{k+1} + g_k)
//   above m: h_{nz-1} = mt_{nz-1}, h_k = mt_k + Tr_{k+1} h_{k+1} / (Tr_{k+1} + h_{k+1}),
//            stored 1 / (Tr_k + h_k)
//   at m:    stored 1 / (mt_m + Tr_m g_{m-1} / (Tr_m + g_{m-1})
//                            + Tr_{m+1} h_{m+1} / (Tr_{m+1} + h_{m+1}))
// These are the textbook pivots D_k - Tr^2 / p of each elimination without
// the cancellation (every g, h >= mt > 0).
// The recurrences are serial chains of divisions, which bound the smaller
// levels: a column's two halves are two lanes' work (wavefronts 0 and 1 of a
// block of 64 columns), each step has one division (the quotient Tr g / (Tr + g)
// of a layer takes the stored inverse of the layer before), and the masses of
// the next layers are loaded ahead. 21 us per small level of 70 layers against
// 40 with one lane per column and two divisions per layer.
__global__ __launch_bounds__(128) void k_pivots(LevelView<double> L,
                                                double* __restrict__ invp64,
                                                float* __restrict__ invp32,
                                                float* __restrict__ M32) {
    const bool top = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6)) != 0;
    const int lane = int(threadIdx.x & 63u);
    const uint32_t P = uint32_t(L.plane);
    const uint32_t want = logical_block() * 64u + uint32_t(lane);
    const bool valid = want < P;
    const uint32_t col = valid ? want : P - 1;
    const int J = int(col / uint32_t(L.nI)), nJ = L.nJ, nz = L.nz, m = nz / 2;
    auto off = [&](int k) { return size_t(k) * size_t(P) + col; };
    auto mt = [&](int k, double M) {
        return M + 2.0 * L.Tlam[k * nJ + J] + L.Tth[k * (nJ + 1) + J] +
               L.Tth[k * (nJ + 1) + J + 1];
    };
    auto put = [&](int k, double M, double ip) {
        if (!valid) return;
        invp64[off(k)] = ip;
        invp32[off(k)] = float(ip);
        M32[off(k)] = float(M);
    };
    // step t: layer t from the bottom, nz-1-t from the top, m excluded
    const int steps = top ? nz - 1 - m : m;
    const int k0 = top ? nz - 1 : 0, ks = top ? -1 : 1;
    constexpr int D = 4;
    double Mn[D], q = 0;   // q: Tr g / (Tr + g) of the layer before
#pragma unroll
    for (int d = 0; d < D; ++d) Mn[d] = L.M[off(k0 + (d < steps ? d : 0) * ks)];
    for (int t0 = 0; t0 < steps; t0 += D) {
        double Mc[D];
#pragma unroll
        for (int d = 0; d < D; ++d) Mc[d] = Mn[d];
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const int t = t0 + D + d;
            Mn[d] = L.M[off(k0 + (t < steps ? t : 0) * ks)];
        }
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const int t = t0 + d;
            if (t >= steps) break;   // wave-uniform
            const int k = k0 + t * ks;
            const double g = mt(k, Mc[d]) + q;
            const double tr = L.Tr[(top ? k : k + 1) * nJ + J];
            const double ip = 1.0 / (tr + g);
            put(k, Mc[d], ip);
            q = tr * g * ip;
        }
    }
    __shared__ double qt[64];
    if (top) qt[lane] = q;
    __syncthreads();
    if (!top) {
        const double M = L.M[off(m)];
        put(m, M, 1.0 / (mt(m, M) + q + qt[lane]));
    }
}

__global__ __launch_bounds__(kBlock) void k_grad_alpha(LevelView<double> L,
                                                       const double* __restrict__ V,
                                                       const double* __restrict__ lam,
                                                       const double* __restrict__ u,
                                                       double* __restrict__ g, uint32_t n) {
    const uint32_t t = global_index();
    if (t >= n) return;
    const uint32_t P = uint32_t(L.plane);
    const int k = int(t / P);
    const int J = int((t - uint32_t(k) * P) / uint32_t(L.nI));
    g[t] = -lam[t] * V[k * L.nJ + J] * u[t];
}

__global__ __launch_bounds__(kBlock) void k_cell_volumes(LevelView<double> L,
                                                         const double* __restrict__ V,
                                                         double* __restrict__ out, uint32_t n) {
    const uint32_t t = global_index();
    if (t >= n) return;
    const uint32_t P = uint32_t(L.plane);
    const int k = int(t / P);
    const int J = int((t - uint32_t(k) * P) / uint32_t(L.nI));
    out[t] = V[k * L.nJ + J];
}

template <typename TA, typename TB>
__global__ __launch_bounds__(kBlock) void k_cast(const TA* __restrict__ in, TB* __restrict__ out,
                                                 long long n) {
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x; t < n; t += stride)
        out[t] = TB(in[t]);
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_fill(T* __restrict__ out, T v, long long n) {
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x; t < n; t += stride)
        out[t] = v;
}

}  // namespace

template <typename T>
void apply(const LevelView<T>& L, const T* x, const T* f, T* y, hipStream_t s) {
    if constexpr (std::is_same<T, double>::value) {
        if (L.plane >= kApplyWalkColumns && L.nz >= kApplyWalkLayers &&
            L.plane * L.nz >= kApplyWalkCells) {
            const int wpr = segments_per_row(L.nI);
            const int tiles = tiled_blocks(L.nJ, wpr, kApplyRows);
            const int ranges = (L.nz + kApplyRange - 1) / kApplyRange;
            auto go = [&](auto fullc, auto modec) {
                constexpr int MODE = decltype(modec)::value;
                k_residual_walk<double, double, double, false, true, kApplyRange,
                                kResidualAhead, kApplyRows, kResidualSync,
                                decltype(fullc)::value, MODE>
                    <<<tiles * ranges, 64 * kApplyRows, 0, s>>>(
                        L, f, x, nullptr, nullptr, y, nullptr, nullptr, wpr, tiles,
                        (L.nz + ranges - 1) / ranges, nullptr, nullptr);
            };
            using One = std::integral_constant<int, 1>;
            using Two = std::integral_constant<int, 2>;
            if (L.nI % 64 == 0) {
                if (f) go(std::true_type{}, Two{});
                else go(std::true_type{}, One{});
            } else {
                if (f) go(std::false_type{}, Two{});
                else go(std::false_type{}, One{});
            }
            return;
        }
    }
    const dim3 grid(unsigned((L.nI + 63) / 64), unsigned((L.nJ + kApplyRows - 1) / kApplyRows),
                    unsigned((L.nz + apply_layers<T>() - 1) / apply_layers<T>()));
    if (f) k_apply<T, true><<<grid, dim3(64, kApplyRows), 0, s>>>(L, x, f, y);
    else k_apply<T, false><<<grid, dim3(64, kApplyRows), 0, s>>>(L, x, f, y);
}

template <typename TU, typename TE, typename TR>
void residual_update(const LevelView<TU>& L, const TU* b, const TU* uin, const TE* e, TU* uout,
                    TR* r, double* partials, double* partials_b, unsigned* done, double* norms,
                    hipStream_t s) {
    const int wpr = segments_per_row(L.nI);
    const int nb = residual_update_blocks(L), range = residual_walk_range(L.nI, L.nJ, L.nz);
    const int ranges = (L.nz + range - 1) / range, lr = (L.nz + ranges - 1) / ranges;
    const bool tall = residual_tile_rows(L.nI, L.nJ) == kResidualTallRows;
    const int tiles = tiled_blocks(L.nJ, wpr, tall ? kResidualTallRows : 4);
    const bool full = L.nI % 64 == 0;
    auto go = [&](auto lrc, auto rc, auto fullc) {
        constexpr int LR = decltype(lrc)::value, R = decltype(rc)::value;
        constexpr bool FULLI = decltype(fullc)::value;
        constexpr int P = kResidualAhead, S = kResidualSync;
        if (e && uin)
            k_residual_walk<TU, TE, TR, true, true, LR, P, R, S, FULLI>
                <<<nb, 64 * R, 0, s>>>(L, b, uin, e, uout, r, partials, partials_b, wpr, tiles,
                                        lr, done, norms);
        else if (e)
            k_residual_walk<TU, TE, TR, true, false, LR, P, R, S, FULLI>
                <<<nb, 64 * R, 0, s>>>(L, b, uin, e, uout, r, partials, partials_b, wpr, tiles,
                                        lr, done, norms);
        else if (uin)
            k_residual_walk<TU, TE, TR, false, true, LR, P, R, S, FULLI>
                <<<nb, 64 * R, 0, s>>>(L, b, uin, e, uout, r, partials, partials_b, wpr, tiles,
                                        lr, done, norms);
        else   // r = b: no neighbours (the same blocks and sums as with u = 0)
            k_residual_walk<TU, TE, TR, false, false, LR, P, R, S, false>
                <<<nb, 64 * R, 0, s>>>(L, b, uin, e, uout, r, partials, partials_b, wpr, tiles,
                                        lr, done, norms);
    };
    auto low = [&](auto lrc) {
        if (full) go(lrc, std::integral_constant<int, 4>{}, std::true_type{});
        else go(lrc, std::integral_constant<int, 4>{}, std::false_type{});
    };
    auto high = [&](auto lrc) {
        constexpr int R = kResidualTallRows;
        if (full) go(lrc, std::integral_constant<int, R>{}, std::true_type{});
        else go(lrc, std::integral_constant<int, R>{}, std::false_type{});
    };
    if (range == kResidualRange) high(std::integral_constant<int, kResidualRange>{});
    else if (range == 16) high(std::integral_constant<int, 16>{});
    else if (range == kResidualShortRange) low(std::integral_constant<int, kResidualShortRange>{});
    else low(std::integral_constant<int, kResidualTinyRange>{});
}

template <typename TU>
int residual_tiles(const LevelView<TU>& L) {
    return tiled_blocks(L.nJ, segments_per_row(L.nI), residual_tile_rows(L.nI, L.nJ));
}

template <typename TU>
int residual_update_blocks(const LevelView<TU>& L) {
    const int tiles = residual_tiles(L);
    const int lr = residual_walk_range(L.nI, L.nJ, L.nz);
    return tiles * ((L.nz + lr - 1) / lr);
}

void sum_partials(const double* partials, int n, double* out, hipStream_t s) {
    k_sum_partials<<<1, 1024, 0, s>>>(partials, n, out);
}

int fine_mass(const LevelView<double>& L, const double* V, const double* alpha, double* M,
              double* partials, hipStream_t s) {
    const long long n = L.plane * L.nz;
    const int nb = grid_stride_blocks(n);
    k_fine_mass<<<nb, kBlock, 0, s>>>(L, V, alpha, M, n, partials);
    return nb;
}

void pivots(const LevelView<double>& L, double* invp64, float* invp32, float* M32,
            hipStream_t s) {
    k_pivots<<<int((L.plane + 63) / 64), 128, 0, s>>>(L, invp64, invp32, M32);
}

void grad_alpha(const LevelView<double>& L, const double* V, const double* lam,
                const double* u, double* g, hipStream_t s) {
    const long long n = L.plane * L.nz;
    k_grad_alpha<<<blocks_for(n), kBlock, 0, s>>>(L, V, lam, u, g, uint32_t(n));
}

void cell_volumes(const LevelView<double>& L, const double* V, double* out, hipStream_t s) {
    const long long n = L.plane * L.nz;
    k_cell_volumes<<<blocks_for(n), kBlock, 0, s>>>(L, V, out, uint32_t(n));
}

template <typename TA, typename TB>
void cast(const TA* in, TB* out, long long n, hipStream_t s) {
    k_cast<TA, TB><<<grid_stride_blocks(n), kBlock, 0, s>>>(in, out, n);
}

template <typename T>
void fill(T* out, T v, long long n, hipStream_t s) {
    k_fill<T><<<grid_stride_blocks(n), kBlock, 0, s>>>(out, v, n);
}

template void residual_update<double, float, float>(const LevelView<double>&, const double*,
                                                  const double*, const float*, double*,
                                                  float*, double*, double*, unsigned*, double*,
                                                  hipStream_t);
template void residual_update<double, double, double>(const LevelView<double>&,
                                                     const double*, const double*,
                                                     const double*, double*, double*,
                                                     double*, double*, unsigned*, double*,
                                                     hipStream_t);
template void residual_update<float, float, float>(const LevelView<float>&, const float*,
                                                 const float*, const float*, float*, float*,
                                                 double*, double*, unsigned*, double*,
                                                 hipStream_t);
template void apply<float>(const LevelView<float>&, const float*, const float*, float*,
                           hipStream_t);
template void apply<double>(const LevelView<double>&, const double*, const double*, double*,
                            hipStream_t);
template int residual_tiles<double>(const LevelView<double>&);
template int residual_update_blocks<double>(const LevelView<double>&);
template int residual_update_blocks<float>(const LevelView<float>&);
template void cast<double, float>(const double*, float*, long long, hipStream_t);
template void cast<float, double>(const float*, double*, long long, hipStream_t);
template void cast<double, double>(const double*, double*, long long, hipStream_t);
template void fill<float>(float*, float, long long, hipStream_t);
template void fill<double>(double*, double, long long, hipStream_t);
template void fill<unsigned>(unsigned*, unsigned, long long, hipStream_t);

}  // namespace mgk
