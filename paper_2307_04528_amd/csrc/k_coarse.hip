// Coarsest-level solve (paper Section 2.3): `sweeps` damped block-Jacobi
// sweeps (Eq. 1) from zero with the level held in the LDS of one block, and
// the explicit matrix of that solve.
//
// A level of a few hundred columns is a serial chain of sweeps: what a sweep
// costs is the dependent steps of its column solves and the LDS traffic of
// its stencil. A lane owns half a column (the twisted factorisation of H_z,
// pivots from setup): the first half of the block's wavefronts eliminates
// the layers below the meeting layer m = nz/2 upward, the second half the
// layers above it downward; they exchange three values per column through
// LDS and substitute back outward. Only the iterate is read from LDS in the
// forward pass (the four neighbours); the inverse pivots, which no sweep
// changes, stay in registers (IPREG), as do the forward values. Two block
// barriers per sweep: before the exchange is read (every lane has then read
// the old neighbours, so the new iterate overwrites them in place) and after
// the new iterate is written.
//
// UNIT: the block solves for U unit vectors at once, U copies of a layer side
// by side in its lanes and LDS, and writes U rows of the matrix (which is
// symmetric, as H is: x = C f with C = sum_k (I - omega H_z^{-1} H)^k omega
// H_z^{-1}). With all of its U * columns lanes packed, a block wastes no
// wavefront on a ragged tail, and the pivots are shared. The couplings are
// products of a layer and a row factor (the metric terms separate): layer k's
// unknowns are scaled by the square root of its horizontal factor h_k, which
// takes that factor out of the stencil and leaves the matrix symmetric, and
// the eliminated values by the row's vertical factor; the row factors stay in
// registers and the vertical layer factors in a lane each, so no coupling is
// read from LDS.
//
// Measured, matrix of 5,040 cells in columns of 70 layers: 1.50 ms (6.94 with
// one unit vector per block and the couplings in LDS; 1.68 with unscaled
// unknowns, whose steps take half as many instructions again). The vector
// units are busy half of that and LDS for two fifths: what bounds it is the
// steps' latency, with the eight wavefronts that registers and LDS hold. Plain
// solve, 40 sweeps of 252 columns of 38 layers in FP32: 54 us (101 with the
// couplings in LDS, 75 with the iterate by layer, whose addresses each step
// computes), 1.35 us per sweep on one CU, latency again.
#include "device.hpp"

namespace mgk {

namespace {
using namespace dev;

// Threads of a block at most (eight wavefronts, two per SIMD: a lane may use
// 256 VGPRs, which FP64 needs for its pivots and forward values).
constexpr int kCoarseThreads = 512;

// Short FP32 columns of a plain solve: what no sweep changes (right-hand side
// and couplings) stays in registers.
template <typename T, int NS, bool UNIT>
constexpr bool coarse_hold() { return !UNIT && std::is_same<T, float>::value && NS <= 24; }

// Steps whose LDS loads are in flight ahead of the ones being solved. (FP32
// columns of 38 layers: 54 us with 2, 58 with 4, 61 with 1 or 5. Unit vectors,
// 70 layers: 1.50 ms with 3, 1.60 with 2, 1.56 with 4.)
template <typename T, int NS, bool UNIT>
constexpr int coarse_ahead() {
    if (UNIT) return 3;
    return std::is_same<T, float>::value && NS <= 44 && !coarse_hold<T, NS, UNIT>() ? 4 : 2;
}

// Whether the iterate lies in LDS by half and step, kStride values per step
// whatever the block's lanes: then a step's addresses are immediate offsets.
// (Where that fits: all that coarse_hold() covers, and FP64 columns up to 36
// steps. Otherwise by layer, as many values as there are lanes.)
constexpr int kStride = kCoarseThreads / 2;
template <typename T, int NS, bool UNIT>
constexpr bool fixed_stride() { return UNIT ? NS <= 36 : coarse_hold<T, NS, UNIT>(); }

// The LDS loads of one step: the four neighbours, and (not UNIT) the
// right-hand side and the couplings of the layer, cn the vertical one to the
// next layer in the half's direction.
template <typename T>
struct CoarseNb {
    T w, e, s, n, f, ip, tl, ts, tn, cn;
};
// The LDS loads of one step of the back-substitution.
template <typename T>
struct CoarseBack {
    T x, ip, cn;
};

// NS: steps compiled for; a half has more than NS - G of them, so only the
// last G + 1 steps need a look at where its layers end.
template <typename T, int NS, int G, bool IPREG, bool UNIT>
__global__ __launch_bounds__(kCoarseThreads) void k_coarse_sweeps(
    LevelView<T> L, SepView sep, const T* __restrict__ f, T* __restrict__ xout,
    float* __restrict__ xout32, T omega, int sweeps, int U) {
    extern __shared__ unsigned char smem_raw[];
    const int P = int(L.plane), nz = L.nz, nJ = L.nJ, n = P * nz;
    const int H = int(blockDim.x) >> 1;          // lanes of one half (whole wavefronts)
    constexpr bool FIXED = fixed_stride<T, NS, UNIT>();
    const int nx = FIXED ? 2 * NS * kStride : U * n;
    T* sx = reinterpret_cast<T*>(smem_raw);      // [2][NS][kStride] or [nz][U][P] iterate
    T* xch = sx + nx;                            // [3][H] exchange
    T* sp = xch + 3 * H;                         // [nz][P] pivots (not IPREG)
    T* sf = sp + (IPREG ? 0 : n);                // [nz][P] right-hand side (not UNIT)
    T* stl = sf + (UNIT ? 0 : n);                // [nz][nJ] (not UNIT)
    T* sth = stl + (UNIT ? 0 : nz * nJ);         // [nz][nJ+1] (not UNIT)
    T* str = sth + (UNIT ? 0 : nz * (nJ + 1));   // [nz+1][nJ] (not UNIT)
    for (int t = threadIdx.x; t < nx; t += blockDim.x) sx[t] = T(0);
    if constexpr (!IPREG)
        for (int t = threadIdx.x; t < n; t += blockDim.x) {
            sp[t] = L.invp[t];
            if constexpr (UNIT) sp[t] *= T(sep.h[t / P]) * T(sep.gr[(t % P) / L.nI]);
        }
    constexpr bool HOLD = coarse_hold<T, NS, UNIT>(), STAGE = !UNIT && !HOLD;
    if constexpr (STAGE) {
        for (int t = threadIdx.x; t < n; t += blockDim.x) sf[t] = f[t];
        for (int t = threadIdx.x; t < nz * nJ; t += blockDim.x) stl[t] = L.Tlam[t];
        for (int t = threadIdx.x; t < nz * (nJ + 1); t += blockDim.x) sth[t] = L.Tth[t];
        for (int t = threadIdx.x; t < (nz + 1) * nJ; t += blockDim.x) str[t] = L.Tr[t];
    }

    const bool top = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >= H ? 1 : 0) != 0;
    const int idx = int(threadIdx.x) - (top ? H : 0);
    const int u0 = idx / P;
    const bool active = u0 < U;
    const int u = active ? u0 : 0, col = active ? idx - u0 * P : 0;
    const Nb b = neighbours(uint32_t(col), L.nI, nJ);
    const int J = b.J;
    // UNIT: the block's unit vectors are 1 in layer ku, columns cu .. cu + U - 1
    const int per_layer = UNIT ? (P + U - 1) / U : 1;
    const int ku = UNIT ? int(blockIdx.x) / per_layer : -1;
    const int cu = UNIT ? (int(blockIdx.x) - ku * per_layer) * U : 0;
    // row factors of the couplings (UNIT)
    const T gl = UNIT ? T(sep.gl[J]) : T(0), gs = UNIT ? T(sep.gt[J]) : T(0),
            gn = UNIT ? T(sep.gt[J + 1]) : T(0), gr = UNIT ? T(sep.gr[J]) : T(0);
    const int m = nz >> 1;
    const int elim = top ? nz - 1 - m : m;   // steps this half eliminates
    const int own = top ? elim + 1 : elim;   // and the layers it writes
    // step t is layer t (bottom) or nz-1-t (top)
    const int k0 = top ? nz - 1 : 0, ks = top ? -1 : 1;
    T ip[IPREG ? NS : 1];
    if constexpr (IPREG) {
#pragma unroll
        for (int t = 0; t < NS; ++t) {
            const int k = k0 + (t < own ? t : 0) * ks;
            ip[t] = L.invp[size_t(k) * size_t(P) + col];
            if constexpr (UNIT) ip[t] *= T(sep.h[k]) * gr;
        }
    }
    // UNIT: the vertical couplings of the scaled unknowns by step, step t's in
    // lane t (read back with a readlane: scalar loads in the chain would each
    // be waited for)
    const int lane = int(threadIdx.x & 63u);
    T vv = T(0), fu = T(0);
    if constexpr (UNIT) {
        const int kl = k0 + (lane < own ? lane : 0) * ks;
        const int kn = kl + ks < 0 ? 0 : clampk(kl + ks, nz);
        vv = T(sep.v[top ? kl : kl + 1]) / (sqrt(T(sep.h[kl])) * sqrt(T(sep.h[kn])));
        fu = active && col == cu + u ? T(1) / sqrt(T(sep.h[ku])) : T(0);
    }
    // not UNIT, FP32: couplings times pivots kept for the back-substitution
    constexpr bool KEEPCB = !UNIT && std::is_same<T, float>::value;
    T hf[HOLD ? NS : 1], hl[HOLD ? NS : 1], hs_[HOLD ? NS : 1], hn[HOLD ? NS : 1],
        hc[HOLD ? NS : 1];
    if constexpr (HOLD) {
#pragma unroll
        for (int t = 0; t < NS; ++t) {
            const int k = k0 + (t < own ? t : 0) * ks;
            hf[t] = f[size_t(k) * size_t(P) + col];
            hl[t] = L.Tlam[k * nJ + J];
            hs_[t] = L.Tth[k * (nJ + 1) + J];
            hn[t] = L.Tth[k * (nJ + 1) + J + 1];
            hc[t] = L.Tr[(top ? k : k + 1) * nJ + J];
        }
    }
    const T keep = T(1) - omega, damp = UNIT ? omega / gr : omega;
    // byte addresses in the iterate: this column and its neighbours, first step
    // (FIXED) or layer 0
    const uint32_t xb = uint32_t(u) * uint32_t(P) + (FIXED && top ? NS * kStride : 0);
    // UNIT: this half's step with the unit values (-1: none)
    const int tu = !UNIT ? -1 : (top ? (ku >= m ? nz - 1 - ku : -1) : (ku < m ? ku : -1));
    // (unit vectors: a lane without a column has a place of its own beyond the
    // columns, where the layout has one)
    constexpr bool SPARE = UNIT && FIXED;
    const uint32_t xc = (SPARE ? uint32_t(idx) + (top ? NS * kStride : 0) : xb + uint32_t(col)) *
                        uint32_t(sizeof(T)),
                   xw = (xb + b.w) * uint32_t(sizeof(T)), xe = (xb + b.e) * uint32_t(sizeof(T)),
                   xs = (xb + b.s) * uint32_t(sizeof(T)), xn = (xb + b.n) * uint32_t(sizeof(T));
    auto at = [&](uint32_t base, uint32_t off) -> T& {
        return *reinterpret_cast<T*>(smem_raw + (base + off));
    };
    constexpr int D = coarse_ahead<T, NS, UNIT>();
    constexpr int NC = (NS + D - 1) / D;
    __syncthreads();

    for (int s = 0; s < sweeps; ++s) {
        // opaque copies, once per chunk, of what the steps' addresses and role
        // decisions depend on: they are formed where they are used, not
        // hoisted out of the loops into hundreds of registers
        int pl = P, xl = U * P * int(sizeof(T)), kb = k0, ow = own, el = elim,
            un = tu;
        auto opaque = [&]() {
            asm volatile("" : "+s"(pl), "+s"(xl), "+s"(kb), "+s"(ow), "+s"(el), "+s"(un));
        };
        T vs = vv;
        if constexpr (UNIT) asm volatile("" : "+v"(vs));
        // steps past a half's layers load a real layer; what they compute is
        // discarded
        auto layer_of = [&](int t) { return kb + (t < NS - G || t < ow ? t : 0) * ks; };
        auto offset_of = [&](int t) -> uint32_t {
            if constexpr (FIXED) return uint32_t(t * kStride) * uint32_t(sizeof(T));
            else return uint32_t(layer_of(t) * xl);
        };
        auto fetch = [&](int t) {
            CoarseNb<T> r;
            const int k = layer_of(t);
            const uint32_t o = offset_of(t < NS ? t : NS - 1);
            r.w = at(xw, o);
            r.e = at(xe, o);
            r.s = at(xs, o);
            r.n = at(xn, o);
            if constexpr (!IPREG) r.ip = sp[k * pl + col];
            if constexpr (!UNIT && !HOLD) {
                r.f = sf[k * pl + col];
                r.tl = stl[k * nJ + J];
                r.ts = sth[k * (nJ + 1) + J];
                r.tn = sth[k * (nJ + 1) + J + 1];
                r.cn = str[(top ? k : k + 1) * nJ + J];
            }
            return r;
        };
        auto fetch_back = [&](int t) {
            CoarseBack<T> r;
            const int k = layer_of(t);
            r.x = at(xc, offset_of(t < NS ? t : NS - 1));
            if constexpr (!IPREG) r.ip = sp[k * pl + col];
            if constexpr (!UNIT && !KEEPCB) r.cn = str[(top ? k : k + 1) * nJ + J];
            return r;
        };
        T y[NS], cb[KEEPCB ? NS : 1];
        // y of the layer eliminated before, and its coupling to this one
        T vp = T(0), cp = T(0), sm = T(0), im = T(0);
        CoarseNb<T> q[2][D];
#pragma unroll
        for (int d = 0; d < D; ++d) q[0][d] = fetch(d);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            opaque();
            if (c + 1 < NC) {
#pragma unroll
                for (int d = 0; d < D; ++d) q[(c + 1) & 1][d] = fetch((c + 1) * D + d);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int d = 0; d < D; ++d) {
                const int t = c * D + d;
                if (t >= NS) continue;
                const CoarseNb<T>& r = q[c & 1][d];
                T sv, cn;
                if constexpr (UNIT) {
                    const T one = t == un ? T(1) : T(0);   // wave-uniform
                    sv = gl * (r.w + r.e) + one * fu + gs * r.s + gn * r.n;
                    cn = lane_value(vs, t);
                } else if constexpr (HOLD) {
                    const int h = HOLD ? t : 0;
                    sv = hf[h] + hl[h] * (r.w + r.e) + hs_[h] * r.s + hn[h] * r.n;
                    cn = hc[h];
                } else {
                    sv = r.f + r.tl * (r.w + r.e) + r.ts * r.s + r.tn * r.n;
                    cn = r.cn;
                }
                const T p = IPREG ? ip[IPREG ? t : 0] : r.ip;   // (UNIT: scaled)
                sv += cp * vp;
                y[t] = sv * p;
                if constexpr (KEEPCB) cb[t] = cn * p;
                if (t < NS - G - 1) {
                    vp = y[t];
                    cp = cn;
                } else if (t < el) {   // wave-uniform
                    vp = y[t];
                    cp = cn;
                } else if (t == el) {
                    sm = sv;
                    im = p;
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        // meeting layer (step elim of the top half):
        // x_m = (s_m + Tr_{m+1} y_{m+1} + Tr_m y_{m-1}) / d_m
        if (!top) {
            xch[idx] = cp * vp;
        } else {
            xch[H + idx] = sm;
            xch[2 * H + idx] = im;
        }
        if constexpr (UNIT) asm volatile("" : "+v"(vs));   // formed again below, not kept
        CoarseBack<T> rb[2][D];
#pragma unroll
        for (int d = 0; d < D; ++d) rb[(NC - 1) & 1][d] = fetch_back((NC - 1) * D + d);
        __syncthreads();
        T z = (xch[H + idx] + xch[idx]) * xch[2 * H + idx];
        // Unit vectors: every lane takes part, also those without a column, since
        // the steps' couplings lie in the lanes of vs, which a branch here would
        // leave out of any copy of it. Only stores are guarded (none with SPARE).
        if (UNIT || active) {
#pragma unroll
            for (int c = NC - 1; c >= 0; --c) {
                opaque();
                if (c > 0) {
#pragma unroll
                    for (int d = 0; d < D; ++d) rb[(c - 1) & 1][d] = fetch_back((c - 1) * D + d);
                }
                __builtin_amdgcn_sched_barrier(0);
                T out[D];
#pragma unroll
                for (int d = D - 1; d >= 0; --d) {
                    const int t = c * D + d;
                    if (t >= NS) continue;
                    const CoarseBack<T>& r = rb[c & 1][d];
                    T k_;
                    if constexpr (KEEPCB) {
                        k_ = cb[t];
                    } else {
                        const T p = IPREG ? ip[IPREG ? t : 0] : r.ip;
                        if constexpr (UNIT) k_ = lane_value(vs, t) * p;
                        else k_ = r.cn * p;
                    }
                    if (t < NS - G - 1 || t < el) z = y[t] + k_ * z;
                    out[d] = damp * z + keep * r.x;
                    if constexpr (!UNIT || SPARE)
                        if (t < NS - G || t < ow) at(xc, offset_of(t)) = out[d];
                }
                if constexpr (UNIT && !SPARE)
                    if (active) {
#pragma unroll
                        for (int d = D - 1; d >= 0; --d) {
                            const int t = c * D + d;
                            if (t >= NS) continue;
                            if (t < NS - G || t < ow) at(xc, offset_of(t)) = out[d];
                        }
                    }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __syncthreads();
    }
    auto place = [&](int k, int c) {
        if constexpr (FIXED) return (k < m ? k : NS + nz - 1 - k) * kStride + c;
        else return k * U * P + c;
    };
    if constexpr (UNIT) {
        // the unit vectors' rows of the matrix, n values each
        const int count = (P - cu < U ? P - cu : U) * n;
        const size_t base = (size_t(ku) * size_t(P) + size_t(cu)) * size_t(n);
        for (int t = threadIdx.x; t < count; t += blockDim.x) {
            const int uu = t / n, kk = (t - uu * n) / P, cc = t - uu * n - kk * P;
            const T v = sx[place(kk, uu * P + cc)] / sqrt(T(sep.h[kk]));
            xout[base + t] = v;
            xout32[base + t] = float(v);
        }
    } else {
        for (int t = threadIdx.x; t < n; t += blockDim.x)
            xout[t] = sx[FIXED ? place(t / P, t % P) : t];
    }
}

inline int lanes64(long long c) { return int((c + 63) / 64 * 64); }

// Pivots in registers up to 36 steps in FP64 (72 VGPRs beside as many for
// the forward values), up to 64 in FP32.
template <typename T>
constexpr bool pivots_in_registers(int ns) {
    return std::is_same<T, float>::value || ns <= 36;
}

// LDS values of a block (see the kernel's layout).
template <typename T, int NS, bool UNIT>
size_t coarse_values(long long plane, int nJ, int nz, int U) {
    const size_t n = size_t(plane) * size_t(nz);
    const size_t staged = size_t(nz) * nJ + size_t(nz) * (nJ + 1) + size_t(nz + 1) * nJ + n;
    return (fixed_stride<T, NS, UNIT>() ? size_t(2 * NS * kStride) : size_t(U) * n) +
           3 * size_t(lanes64(plane * U)) + (pivots_in_registers<T>(NS) ? 0 : n) +
           (UNIT || coarse_hold<T, NS, UNIT>() ? 0 : staged);
}
template <typename T, bool UNIT>
size_t coarse_values_for(long long plane, int nJ, int nz, int U) {
    size_t v = 0;
    with_half((nz + 1) / 2, [&](auto ns, auto) {
        v = coarse_values<T, decltype(ns)::value, UNIT>(plane, nJ, nz, U);
    });
    return v;
}

template <typename T, int NS, int G, bool UNIT>
bool launch(const LevelView<T>& L, const SepView& sep, const T* f, T* x, float* x32, T omega,
            int sweeps, int U, int blocks, hipStream_t s) {
    constexpr bool IPREG = pivots_in_registers<T>(NS);
    const size_t lds = coarse_values<T, NS, UNIT>(L.plane, L.nJ, L.nz, U) * sizeof(T);
    const auto fn = &k_coarse_sweeps<T, NS, G, IPREG, UNIT>;
    if (!allow_lds(fn, lds)) return false;
    fn<<<blocks, 2 * lanes64(L.plane * U), lds, s>>>(L, sep, f, x, x32, omega, sweeps, U);
    return true;
}

}  // namespace

template <typename T>
bool coarse_solve_fits(long long plane, int nJ, int nz, size_t max_lds) {
    return 2 * lanes64(plane) <= kCoarseThreads &&
           coarse_values_for<T, false>(plane, nJ, nz, 1) * sizeof(T) <= max_lds;
}

template <typename T>
bool coarse_solve(const LevelView<T>& L, const T* f, T* x, T omega, int sweeps, size_t max_lds,
                  hipStream_t s) {
    if (!coarse_solve_fits<T>(L.plane, L.nJ, L.nz, max_lds)) return false;
    bool done = false;
    with_half((L.nz + 1) / 2, [&](auto ns, auto g) {
        done = launch<T, decltype(ns)::value, decltype(g)::value, false>(
            L, SepView{}, f, x, nullptr, omega, sweeps, 1, 1, s);
    });
    return done;
}

// Unit vectors per block: as many as its LDS and lanes hold, but not so many
// that fewer than two blocks per CU remain (a smaller level then spreads over
// more CUs instead).
static int basis_vectors(long long plane, int nJ, int nz, size_t max_lds) {
    const long long n = plane * nz;
    int U = 0;
    while (2 * lanes64(plane * (U + 1)) <= kCoarseThreads &&
           coarse_values_for<double, true>(plane, nJ, nz, U + 1) * sizeof(double) <= max_lds &&
           (U == 0 || (U + 1) * 512LL <= n))
        ++U;
    return U;
}

bool coarse_basis_fits(long long plane, int nJ, int nz, size_t max_lds) {
    return plane * nz <= kDenseCoarseMax && plane <= kDenseCoarseColumns &&
           basis_vectors(plane, nJ, nz, max_lds) > 0;
}

bool coarse_basis(const LevelView<double>& L, const SepView& sep, double* C, float* C32,
                  double omega, int sweeps, size_t max_lds, hipStream_t s) {
    const long long n = L.plane * L.nz;
    if (n < 1 || !coarse_basis_fits(L.plane, L.nJ, L.nz, max_lds)) return false;
    const int U = basis_vectors(L.plane, L.nJ, L.nz, max_lds);
    bool done = false;
    with_half((L.nz + 1) / 2, [&](auto ns, auto g) {
        done = launch<double, decltype(ns)::value, decltype(g)::value, true>(
            L, sep, nullptr, C, C32, omega, sweeps, U, int((L.plane + U - 1) / U * L.nz), s);
    });
    return done;
}

template bool coarse_solve_fits<float>(long long, int, int, size_t);
template bool coarse_solve_fits<double>(long long, int, int, size_t);
template bool coarse_solve<float>(const LevelView<float>&, const float*, float*, float, int,
                                  size_t, hipStream_t);
template bool coarse_solve<double>(const LevelView<double>&, const double*, double*, double, int,
                                   size_t, hipStream_t);

}  // namespace mgk
