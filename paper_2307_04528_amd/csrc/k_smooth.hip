// Block-Jacobi smoother (paper Eq. 1, Section 2.1) on the small levels.
//
// One sweep, with the vertical couplings in H_z solved exactly per column:
//   x_new = (1 - omega) x + omega H_z^{-1} (f + sum_h T_h x_nb)
// which equals x + omega H_z^{-1}(f - H x) since H = H_z + dH and dH holds
// only the horizontal off-diagonals -T_h. Levels that fill the GPU sweep
// with k_sweep (k_sweep.hip); k_smooth_staged here takes the levels below
// staged_columns. (The coarsest level's solve is in k_coarse.hip.)
//
// Column solves use the twisted factorisation of H_z (pivots from setup): one
// wavefront eliminates the layers below the meeting layer m = nz/2 going up,
// another the layers above it going down; after one exchange through LDS
// both know layer m, and each back-substitutes outward. The chain of
// dependent steps is half as long as a one-sided Thomas solve.
#include "device.hpp"

namespace mgk {

namespace {
using namespace dev;

// Staged sweep for small levels. A level of a few thousand columns leaves
// most of the GPU idle: a sweep then costs the critical path of one column
// (its memory round trips and the dependent steps of its solve), not
// bandwidth. Here kStageWaves wavefronts share one segment of 64 columns:
// wavefront w loads layers w, w + kStageWaves, ... (all of its loads in one
// round trip), forms the right-hand sides s = f + sum_h T_h x_nb and writes s
// and the inverse pivots to LDS. After a block barrier the first two
// wavefronts solve the twisted factorisation of H_z, a half column each: s
// and the pivots come from LDS a chunk ahead, the row's vertical couplings
// from the wavefront's lanes, and the forward values stay in registers, so a
// step costs its few instructions. They leave the solution in LDS; after
// another barrier every wavefront damps and stores its own layers, whose old
// iterate it still holds.
//
// In LDS the upper half column lies from the top down after the lower one
// from the bottom up: step t of a half is t * 64 values from the half's base.
//
// Measured: a launch takes 5.6 us on levels of 1-6K columns with 70 layers
// (7.9 with the solve in rolled loops over LDS, where each step waited for
// its loads), 4.7 with 38 layers (6.0), FP64 8.0 with 70 (11.0); 10.9 us of
// 27,648 columns (13.0); with 100 layers, where the LDS now holds the layers
// there are and not 128, 26 us of 51,200 columns (51.7).
constexpr int kStageWaves = 8;

__device__ __forceinline__ float fmad(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double fmad(double a, double b, double c) { return fma(a, b, c); }

// Dynamic LDS of k_smooth_staged: s and pivots by layer (and the rows that
// the padded steps read), and the pair's exchange.
template <typename T>
constexpr size_t staged_lds_bytes(int nz, int pad) {
    return sizeof(T) * (2 * size_t(nz + pad) * 64 + 256);
}

// Whether the couplings times pivots for the way back are kept in registers
// (else formed again), and the wavefronts per SIMD that the registers must allow.
// FP32: two blocks per CU, 128 VGPRs (26 us against 34 with one on 51,200 columns
// of 100 layers). FP64 spills at 128: 20.7 us against 19.1 on 23,552 columns of
// 70 layers. From zero it has fewer values to hold, and more blocks per CU pay on
// the larger levels: two from 49 to 72 layers without the kept products (320x200
// columns of 70 layers 28.0 -> 23.7 us, 200x128 16.3 -> 13.3; 3,072 columns 8.4 ->
// 8.6), four from 17 to 32 (320x200x24 12.4 -> 10.5, x32 14.1 -> 12.3); between,
// LDS holds two either way.
template <typename T, int NS, bool HAS_X>
constexpr bool kept_couplings() {
    if (sizeof(T) == 4) return NS <= 44;
    return HAS_X ? NS <= 36 : NS <= 8 || (NS > 16 && NS <= 24);
}
template <typename T, int NS, bool HAS_X>
constexpr int staged_waves() {
    if (sizeof(T) == 4) return 4;
    return HAS_X || NS > 36 ? 2 : (NS <= 16 ? 8 : (NS <= 24 ? 2 : 4));
}

// NS: steps of a half column compiled for; a half has more than NS - G.
// PRO: the iterate is xin + P xc, formed as it is loaded: the first sweep after
// a coarse-grid correction, without a launch of its own for P (4.7 us on any
// small level; FP32 sweeps of 38 layers take 6.9 us instead of 4.8).
template <typename T, int NS, int G, bool HAS_X, bool PRO>
__global__ __launch_bounds__(64 * kStageWaves)
__attribute__((amdgpu_waves_per_eu(staged_waves<T, NS, HAS_X>()))) void k_smooth_staged(
    LevelView<T> L, const T* __restrict__ f, const T* __restrict__ xin, T* __restrict__ xout,
    T omega, int wpr, TransferView<T> X, const T* __restrict__ xc) {
    // products and sums are contracted by hand: the same bits in every variant
#pragma clang fp contract(off)
    extern __shared__ unsigned char smem_raw[];
    const int nz = L.nz, nJ = L.nJ, m = nz >> 1;
    T* ls = reinterpret_cast<T*>(smem_raw);   // [nz + G][64] s, then the solution
    T* lp = ls + (nz + G) * 64;               // [nz + G][64] inverse pivots
    T* xch = lp + (nz + G) * 64;              // [4][64] the pair's exchange
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    const int lane = int(threadIdx.x & 63u);
    const Seg g = segment(int(blockIdx.x), L.nI, nJ, wpr);
    NbB<T> b(g);
    const int J = g.J;
    // PRO: west and east of a column lie in the neighbour lanes, and one more
    // column brings what the outer two lanes miss: west of lane 0's in the
    // lower lanes, east of lane 63's in the upper. (A lane past the row's end,
    // which stores nothing, takes the row's first column: the last one's east.)
    // Coarse offsets of the four points: this column, south, north, outer.
    uint32_t od = 0, oo[PRO ? 4 : 1][4];
    T pw[PRO ? 4 : 1][2];
    if constexpr (PRO) {
        constexpr uint32_t S = sizeof(T);
        const int nI = L.nI, i0 = (int(blockIdx.x) - J * wpr) * 64;
        const int i = g.valid ? i0 + lane : 0;
        const int io = lane < 32 ? (i0 == 0 ? nI - 1 : i0 - 1) : (i0 + 64 < nI ? i0 + 64 : 0);
        od = uint32_t(J * nI + io) * S;
        if (!g.valid) b.c = uint32_t(J * nI) * S;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const int j = p == 1 ? (J > 0 ? J - 1 : J) : (p == 2 ? (J < nJ - 1 ? J + 1 : J) : J);
            // (with b.s and b.n of a lane past the row's end: any cell will do)
            const int ip = p == 3 ? io : (p == 0 ? i : (g.valid ? i0 + lane : nI - 1));
            const int I = ip >> 1, In = prolong_neighbour(ip, X.nIc);
            const int J0 = tab(X.prow, 2 * j), J1 = tab(X.prow, 2 * j + 1);
            pw[p][0] = tab(X.pw, 2 * j);
            pw[p][1] = tab(X.pw, 2 * j + 1);
            oo[p][0] = uint32_t(J0 * X.nIc + I) * S;
            oo[p][1] = uint32_t(J0 * X.nIc + In) * S;
            oo[p][2] = uint32_t(J1 * X.nIc + I) * S;
            oo[p][3] = uint32_t(J1 * X.nIc + In) * S;
        }
    }
    const uint64_t Pb = uint64_t(L.plane) * sizeof(T);
    constexpr int Q = (2 * NS + kStageWaves - 1) / kStageWaves;
    // position of layer k in LDS
    auto pos = [&](int k) { return k < m ? k : m + (nz - 1 - k); };
    const bool top = wave == 1;
    // the vertical couplings of the solving wavefronts' row: lane t holds that
    // of step t to the next layer toward the meeting layer
    T tr = T(0);
    if (wave < 2) {
        int F = top ? nz - 1 - lane : lane + 1;
        F = F < 0 ? 0 : (F < nz ? F : nz);
        tr = L.Tr[size_t(F) * size_t(nJ) + size_t(J)];
    }
    T rc[HAS_X ? Q : 1];
    {
        // the horizontal couplings of this wavefront's layers: lane q holds
        // those of layer wave + q kStageWaves (vector loads issued with the
        // stencil loads, read back with readlane)
        T ctl = T(0), cts = T(0), ctn = T(0);
        if (HAS_X && lane < Q) {
            const int kq = clampk(wave + lane * kStageWaves, nz);
            ctl = L.Tlam[size_t(kq) * size_t(nJ) + size_t(J)];
            cts = L.Tth[size_t(kq) * size_t(nJ + 1) + size_t(J)];
            ctn = L.Tth[size_t(kq) * size_t(nJ + 1) + size_t(J) + 1];
        }
        T rf[Q], rp[Q], rw[HAS_X ? Q : 1], re[HAS_X ? Q : 1], rs[HAS_X ? Q : 1],
            rn[HAS_X ? Q : 1];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int kk = clampk(wave + q * kStageWaves, nz);
            rf[q] = ldb<T>(layer(f, kk, Pb), b.c);
            rp[q] = ldb<T>(layer(L.invp, kk, Pb), b.c);
            if constexpr (HAS_X) {
                gcptr xl = layer(xin, kk, Pb);
                rc[q] = ldb<T>(xl, b.c);
                if constexpr (PRO) {
                    rw[q] = ldb<T>(xl, od);
                } else {
                    rw[q] = ldb<T>(xl, b.w);
                    re[q] = ldb<T>(xl, b.e);
                }
                rs[q] = ldb<T>(xl, b.s);
                rn[q] = ldb<T>(xl, b.n);
            }
        }
        if constexpr (PRO) {
            const uint64_t Pcb = uint64_t(X.nIc) * uint64_t(X.nJc) * sizeof(T);
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                gcptr cl = layer(xc, clampk(wave + q * kStageWaves, nz), Pcb);
                auto add = [&](T v, int p) {
                    return prolonged(v, ldb<T>(cl, oo[p][0]), ldb<T>(cl, oo[p][1]),
                                     ldb<T>(cl, oo[p][2]), ldb<T>(cl, oo[p][3]), pw[p][0],
                                     pw[p][1]);
                };
                rc[q] = add(rc[q], 0);
                rs[q] = add(rs[q], 1);
                rn[q] = add(rn[q], 2);
                const T ro = add(rw[q], 3);
                rw[q] = from_below(ro, rc[q]);
                re[q] = from_above(ro, rc[q]);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int k = wave + q * kStageWaves;
            if (k < nz) {
                T s = rf[q];
                if constexpr (HAS_X) {
                    const T h = lane_value(cts, q) * rs[q];
                    s += fmad(lane_value(ctn, q), rn[q],
                              fmad(lane_value(ctl, q), rw[q] + re[q], h));
                }
                ls[pos(k) * 64 + lane] = s;
                lp[pos(k) * 64 + lane] = rp[q];
            }
        }
    }
    __syncthreads();
    const int elim = top ? nz - 1 - m : m;   // steps a half eliminates
    const int own = top ? elim + 1 : elim;   // and the layers it solves for
    T* hs = ls + (top ? m * 64 : 0) + lane;
    const T* hp = lp + (top ? m * 64 : 0) + lane;
    constexpr bool KEEPCB = kept_couplings<T, NS, HAS_X>();
    constexpr int D = sizeof(T) == 4 ? 6 : 3;
    constexpr int NC = (NS + D - 1) / D;
    T y[NS], cb[KEEPCB ? NS : 1];
    if (wave < 2) {
        T bs[2][D], bp[2][D];
        auto fetch = [&](int c) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                const int t = c * D + d < NS ? c * D + d : NS - 1;
                bs[c & 1][d] = hs[t * 64];
                bp[c & 1][d] = hp[t * 64];
            }
        };
        T vp = T(0), cp = T(0), sm = T(0), im = T(0);
        fetch(0);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if (c + 1 < NC) fetch(c + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int d = 0; d < D; ++d) {
                const int t = c * D + d;
                if (t >= NS) continue;
                const T s = bs[c & 1][d], ip = bp[c & 1][d], cn = lane_value(tr, t);
                T v = fmad(cp, vp, s) * ip;
                // computed here, not sunk (with its operands) to later blocks
                asm volatile("" : "+v"(v));
                y[t] = v;
                if constexpr (KEEPCB) cb[t] = cn * ip;
                if (t < NS - G - 1 || t < elim) {   // wave-uniform
                    vp = v;
                    cp = cn;
                } else if (t == elim) {
                    sm = s;
                    im = ip;
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (!top) {
            xch[lane] = vp;
        } else {
            xch[64 + lane] = vp;
            xch[128 + lane] = sm;
            xch[192 + lane] = im;
        }
    }
    __syncthreads();
    if (wave < 2) {
        // meeting layer: x_m = (s_m + Tr_m y_{m-1} + Tr_{m+1} z_{m+1}) / d_m
        // (the couplings' faces have no lane where a half is empty; Tr is 0)
        const T cm = m > 0 ? L.Tr[size_t(m) * size_t(nJ) + size_t(J)] : T(0);
        const T cm1 = m + 1 < nz ? L.Tr[size_t(m + 1) * size_t(nJ) + size_t(J)] : T(0);
        T z = fmad(cm1, xch[64 + lane], fmad(cm, xch[lane], xch[128 + lane])) * xch[192 + lane];
        T bp[2][KEEPCB ? 1 : D];
        auto fetch = [&](int c) {
            if constexpr (!KEEPCB) {
#pragma unroll
                for (int d = 0; d < D; ++d)
                    bp[c & 1][d] = hp[(c * D + d < NS ? c * D + d : NS - 1) * 64];
            }
        };
        fetch(NC - 1);
#pragma unroll
        for (int c = NC - 1; c >= 0; --c) {
            if (c > 0) fetch(c - 1);
            if constexpr (!KEEPCB) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int d = D - 1; d >= 0; --d) {
                const int t = c * D + d;
                if (t >= NS) continue;
                T k_;
                if constexpr (KEEPCB) k_ = cb[t];
                else k_ = lane_value(tr, t) * bp[c & 1][d];
                if (t < NS - G - 1 || t < elim) z = fmad(k_, z, y[t]);
                if (t < NS - G || t < own) hs[t * 64] = z;
            }
        }
    }
    __syncthreads();
    const T keep = T(1) - omega;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int k = wave + q * kStageWaves;
        if (k < nz) {
            const T z = ls[pos(k) * 64 + lane];
            T out = omega * z;
            if constexpr (HAS_X) {
                const T old = keep * rc[q];
                out = fmad(omega, z, old);
            }
            if (g.valid) stb<T>(layer_w(xout, k, Pb), b.c, out);
        }
    }
}

}  // namespace

// Half columns that smooth_prolonged is compiled for: as many layers per
// wavefront as keep the four points' coarse values in one or two round trips.
// (160x96, per V-cycle with P apart and in the sweep: FP32 16 layers 134 and
// 124 us, 40 layers 173 and 164, 48 layers 181.5 and 182; FP64 8 layers 131 and
// 122, 16 layers 155 and 152, 24 layers 174 and 176. With 70 layers a sweep
// that spills takes 19 us against 5.5 + 4.7.)
template <typename T>
constexpr int prolong_steps() { return sizeof(T) == 4 ? 20 : 8; }
// And the blocks of it: two per CU (390 blocks of 38 layers 9.6 us against 6.7
// + 4.9; 960 blocks 17.6 against 11.0 + 6.1).
constexpr long long kProlongBlocks = 512;

// The staged sweep of a small level (with X: of xin + P xc); false where the
// level is not small or the staging buffers do not fit in LDS.
template <typename T>
bool launch_staged(const LevelView<T>& L, const T* f, const T* xin, T* xout, T omega,
                   const TransferView<T>* X, const T* xc, long long staged_columns,
                   hipStream_t s) {
    if (L.plane >= staged_columns) return false;
    const int wpr = segments_per_row(L.nI);
    const int nb = L.nJ * wpr;
    bool launched = false;
    with_half((L.nz + 1) / 2, [&](auto ns, auto gc) {
        constexpr int NS = decltype(ns)::value, G = decltype(gc)::value;
        const size_t lds = staged_lds_bytes<T>(L.nz, G);
        if (lds > kMaxLds) return;
        auto go = [&](auto hx, auto pro) {
            const auto fn = &k_smooth_staged<T, NS, G, decltype(hx)::value, decltype(pro)::value>;
            if (!allow_lds(fn, lds)) return;
            fn<<<nb, 64 * kStageWaves, lds, s>>>(L, f, xin, xout, omega, wpr,
                                                 X ? *X : TransferView<T>{}, xc);
            launched = true;
        };
        if (X) {
            if constexpr (NS <= prolong_steps<T>()) go(std::true_type{}, std::true_type{});
        } else if (xin) {
            go(std::true_type{}, std::false_type{});
        } else {
            go(std::false_type{}, std::false_type{});
        }
    });
    return launched;
}

template <typename T>
bool prolongs_in_sweep(const LevelView<T>& L, long long staged_columns) {
    return L.plane < staged_columns && (L.nz + 1) / 2 <= prolong_steps<T>() &&
           (long long)L.nJ * segments_per_row(L.nI) <= kProlongBlocks;
}

template <typename T>
bool smooth_prolonged(const LevelView<T>& L, const TransferView<T>& X, const T* f, const T* xin,
                      const T* xc, T* xout, T omega, long long staged_columns, hipStream_t s) {
    return prolongs_in_sweep<T>(L, staged_columns) &&
           launch_staged<T>(L, f, xin, xout, omega, &X, xc, staged_columns, s);
}

template <typename T>
void smooth(const LevelView<T>& L, const T* f, const T* xin, T* xout, T omega,
            long long staged_columns, hipStream_t s) {
    if (launch_staged<T>(L, f, xin, xout, omega, nullptr, nullptr, staged_columns, s)) return;
    sweep<T>(L, f, xin, xout, omega, s);
}

template void smooth<float>(const LevelView<float>&, const float*, const float*, float*, float,
                            long long, hipStream_t);
template bool prolongs_in_sweep<float>(const LevelView<float>&, long long);
template bool prolongs_in_sweep<double>(const LevelView<double>&, long long);
template bool smooth_prolonged<float>(const LevelView<float>&, const TransferView<float>&,
                                      const float*, const float*, const float*, float*, float,
                                      long long, hipStream_t);
template bool smooth_prolonged<double>(const LevelView<double>&, const TransferView<double>&,
                                       const double*, const double*, const double*, double*,
                                       double, long long, hipStream_t);
template void smooth<double>(const LevelView<double>&, const double*, const double*, double*,
                             double, long long, hipStream_t);

}  // namespace mgk
