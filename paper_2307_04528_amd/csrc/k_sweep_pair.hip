// Two consecutive sweeps (paper Eq. 1, Section 2.1) of a large level in one
// pass over memory, FP32:
//   x1 = (1 - om1) x + om1 H_z^{-1} (f + sum_h T_h x_nb)     (or om1 H_z^{-1} f)
//   x2 = (1 - om2) x1 + om2 H_z^{-1} (f + sum_h T_h x1_nb)
// A sweep by itself reads f, the pivots and x and writes x: 16 B per cell, at
// the rate of HBM. Two sweeps in one pass move the same 16 B: x1 never leaves
// the CU, and f and the pivots are read once for both.
//
// Tiling. A block owns a strip of up to 62 longitudes (64 lanes: x1 is
// needed one column beyond the outputs on either side) and a band of rows,
// and walks the band row by row. Five pairs of wavefronts take the rows in
// turn (one wavefront per half column: the twisted factorisation, as in
// k_sweep): in phase p a pair does the first sweep of row p, in phase p + 2,
// when x1 of row p + 1 is there, the second sweep of row p, with f and the
// pivots of the row still in its registers, and from phase p + 3 it loads
// those of its next row, p + 5. So each phase does one first and one second
// sweep of a row, and loads have two phases to arrive. Two more wavefronts
// load the rows of x straight into LDS, three rows ahead.
//
// LDS. A ring of eight row slots holds x and x1: row r of x lies in slot r,
// and x1 of row r replaces x of row r - 1, which the first sweep of row r was
// the last to read (slots modulo 8). In phase p the first sweep reads x of
// p-1, p, p+1, the second x1 of p-3, p-2, p-1 (slots p-4 .. p-2), and x of
// p+2 and p+3 is arriving. Within a slot the upper half column is stored from
// the top down, so that step t of either half lies t * 256 B from the half's
// base: an immediate offset. 70 layers take 140 KB: one block per CU.
//
// Barriers. Two per phase. The one in mid phase publishes the meeting
// exchange of both pairs and ends the reads of the row that x1 replaces; the
// one at the end publishes x1 and the arrived rows. Every wavefront of the
// block reaches both in every phase, whatever its role.
//
// What bounds it: on 1024x768x70 a launch takes 261 us (single sweeps: 2 x
// 191) and 195 us from zero (120 + 191), at 1.11 and 0.81 GB of counted
// traffic, 4.2 TB/s; the rows' misaligned ends cost 1.25x the bytes
// of f and the pivots, and without its loads a launch takes 141 us. Measured
// on the way: three pairs that keep the next row in a second set of registers
// 305 us, non-temporal hints 291 us, the step records as scalar loads of the
// steps 490 us, taller bands on fewer blocks 264-285 us.
#include "device.hpp"

namespace mgk {

namespace {
using namespace dev;

constexpr int kOut = 62;          // output columns of a strip at most
constexpr int kSlots = 8;         // row slots of the ring
constexpr int kPairs = 5;         // pairs of compute wavefronts
constexpr int kLoadWaves = 2;     // loading wavefronts
constexpr int kEdgeRow = 192;     // edge values of a row slot (2 per layer, padded)
constexpr int kZeros = 96;        // zeros read by the lanes that have no edge

struct Strips {
    int count, width;   // strips, output columns of each (the last may have fewer)
    int band;           // rows per band
};

// LDS values of a block: the ring, the edge columns (from an iterate), the
// meeting exchange of the pairs and the zeros.
inline size_t pair_lds_values(int nz, bool zero) {
    return size_t(zero ? 4 : kSlots) * size_t(nz) * 64 + (zero ? 0 : size_t(kSlots) * kEdgeRow) +
           kPairs * 4 * 64 + kZeros;
}

// NS: steps of a half column compiled for; a half has more than NS - G.
// ZERO: the first sweep starts from zero (x is not read). Plain loads and
// stores at every size: neighbouring strips share the cache lines at their
// borders, and with the non-temporal hint each fetches (or writes part of)
// its own.
template <int NS, int G, bool ZERO>
__global__ __launch_bounds__(64 * (2 * kPairs + kLoadWaves))
__attribute__((amdgpu_waves_per_eu(3)))
void k_sweep_pair(LevelView<float> L, const float* __restrict__ f, const float* __restrict__ xin,
                  float* __restrict__ xout, float om1, float om2, Strips st) {
    extern __shared__ float ring[];
    const int nI = L.nI, nJ = L.nJ, nz = L.nz, m = nz >> 1;
    const int lb = int(logical_block());
    const int band = lb / st.count, strip = lb - band * st.count;
    const int j0 = band * st.band;                       // first output row
    const int B = nJ - j0 < st.band ? nJ - j0 : st.band; // output rows
    const int c0 = strip * st.width;                     // first output column
    const int cn = nI - c0 < st.width ? nI - c0 : st.width;
    const int r0 = j0 - 1;                               // row of phase 0
    const int phases = B + 3;
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    const int lane = int(threadIdx.x & 63u);
    // this lane's column (wrapping around the circle of longitude)
    auto wrap = [&](int c) { return c < 0 ? c + nI : c % nI; };
    const int col = wrap(c0 - 1 + lane);
    const uint32_t Pb = uint32_t(L.plane) * 4u, bytes = Pb * uint32_t(nz);
    const int slot_values = nz * 64;
    float* edges = ring + (ZERO ? 4 : kSlots) * slot_values;
    float(*xch)[4][64] =
        reinterpret_cast<float(*)[4][64]>(edges + (ZERO ? 0 : kSlots * kEdgeRow));
    typedef float f4 __attribute__((ext_vector_type(4)));
    float* zeros = &xch[kPairs][0][0];
    if (threadIdx.x < kZeros) zeros[threadIdx.x] = 0.0f;
    auto xslot = [&](int r) { return (r & (kSlots - 1)) * slot_values; };
    auto x1slot = [&](int r) {
        return (ZERO ? (r & 3) : ((r - 1) & (kSlots - 1))) * slot_values;
    };

    if (wave >= 2 * kPairs) {
        // a loading wavefront (every second layer): rows of x, straight into LDS
        typedef __attribute__((address_space(3))) void* lptr;
        const int part = wave - 2 * kPairs;
        const rsrc_t rx = make_rsrc(ZERO ? f : xin, bytes);
        const int ec = wrap((lane & 1) ? c0 + 63 : c0 - 2);   // this lane's edge column
        // (always NS + 2 loads, layers past the last one loading it again: the
        // wait below counts them)
        auto load_row = [&](int r) {
            if constexpr (!ZERO) {
                const uint32_t ov = uint32_t(r * nI + col) * 4u;
                float* dst = ring + xslot(r);
                for (int i = 0; i < NS; ++i) {
                    const int pi = part + kLoadWaves * i, p = pi < nz ? pi : nz - 1;
                    const int k = p < m ? p : nz - 1 - (p - m);
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lptr)(dst + p * 64), 4, int(ov),
                                                             int(uint32_t(k) * Pb), 0, 0);
                }
                float* de = edges + (r & (kSlots - 1)) * kEdgeRow;
                for (int h = 0; h < 2; ++h) {
                    const int i = part + kLoadWaves * h < 3 ? part + kLoadWaves * h : 2;
                    const int e = i * 64 + lane;
                    const int p = (e >> 1) < nz ? (e >> 1) : nz - 1;
                    const int k = p < m ? p : nz - 1 - (p - m);
                    const uint32_t oe = uint32_t(k) * Pb + uint32_t(r * nI + ec) * 4u;
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lptr)(de + i * 64), 4, int(oe),
                                                             0, 0, 0);
                }
            }
        };
        // barriers of this wavefront: no wait but the one on its own loads
        auto barrier = []() {
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        };
        const int last = r0 + B + 2 < nJ - 1 ? r0 + B + 2 : nJ - 1;   // last row needed
        for (int r = r0 - 1 < 0 ? 0 : r0 - 1; r <= r0 + 2; ++r)
            if (r <= last) load_row(r);
        __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
        barrier();
        for (int p = 0; p < phases; ++p) {
            const int r = r0 + p + 3;
            const bool more = !ZERO && r <= last;
            if (more) load_row(r);
            barrier();
            // the row that the next phase reads first, loaded in the phase
            // before, must be in LDS; this phase's NS + 2 loads may still be in
            // flight
            constexpr int C = NS + 2;
            if (more) __builtin_amdgcn_s_waitcnt(0x0f70 | (C & 15) | ((C >> 4) << 14));
            else __builtin_amdgcn_s_waitcnt(0x0f70);
            barrier();
        }
        return;
    }

    // The hardware deals a block's wavefronts to the four SIMDs in turn; this
    // order puts the two pairs that sweep in the same phase (p and p - 2) on
    // different SIMDs in all but one phase of five.
    const int place = wave >> 1;
    const int pair = place == 2 ? 3 : (place == 3 ? 2 : place);
    const bool top = (wave & 1) != 0;
    const int elim = top ? nz - 1 - m : m;   // steps this half eliminates
    const int own = top ? elim + 1 : elim;   // and the layers it writes
    const int hb = top ? m * 64 : 0;         // the half's base in a row slot
    const rsrc_t rf = make_rsrc(f, bytes), rp = make_rsrc(L.invp, bytes),
                 ro = make_rsrc(xout, bytes);
    // Byte offsets of the layers by step (steps past the half: of step 0),
    // from copies that opaque() hides: formed where they are used, not kept in
    // scalar registers.
    struct Offsets {
        uint32_t first, step;
        int own;
        __device__ __forceinline__ void opaque() {
            asm volatile("" : "+s"(first), "+s"(step), "+s"(own));
        }
        __device__ __forceinline__ uint32_t operator()(int t) const {
            return first + uint32_t(t < NS - G || t < own ? t : 0) * step;
        }
    };
    const Offsets offsets{top ? uint32_t(nz - 1) * Pb : 0u, top ? 0u - Pb : Pb, own};
    constexpr int D = 4, NC = (NS + D - 1) / D;    // steps per chunk, forward
    constexpr int E = 6, NE = (NS + E - 1) / E;    // and back
    float fr[NS], ir[NS];
    f4 q = {0, 0, 0, 0};   // step records, step t's in lane t
#pragma unroll
    for (int t = 0; t < NS; ++t) fr[t] = ir[t] = 0.0f;

    // f (part 0), pivots and records (part 1) of row r into registers
    auto load_part = [&](auto part, int r) {
        constexpr int PART = decltype(part)::value;
        const uint32_t ov = uint32_t(r * nI + col) * 4u;
        Offsets soff = offsets;
#pragma unroll
        for (int t = 0; t < NS; ++t) {
            if (t % 4 == 0) soff.opaque();
            if constexpr (PART == 0) fr[t] = bld<float>(rf, ov, soff(t));
            else ir[t] = bld<float>(rp, ov, soff(t));
        }
        if constexpr (PART == 1)
            q = *reinterpret_cast<const f4*>(
                &L.sc[(size_t(top) * size_t(nJ) + size_t(r)) * size_t(L.scs) + lane]);
    };
    using Part0 = std::integral_constant<int, 0>;
    using Part1 = std::integral_constant<int, 1>;

    // One sweep of row r (first: x -> x1 in LDS; second: x1 -> xout).
    // Products and sums are contracted by hand, as the compiler does in k_sweep:
    // the two kernels give the same bits.
    auto sweep_row = [&](auto first_c, int r, float omega) {
#pragma clang fp contract(off)
        constexpr bool FIRST = decltype(first_c)::value;
        constexpr bool HAS_X = !(FIRST && ZERO);
        const float keep = 1.0f - omega;
        const int rs = r > 0 ? r - 1 : r, rn = r < nJ - 1 ? r + 1 : r;
        const float* pc = ring + (FIRST ? xslot(r) : x1slot(r)) + hb + lane;
        const float* ps = ring + (FIRST ? xslot(rs) : x1slot(rs)) + hb + lane;
        const float* pn = ring + (FIRST ? xslot(rn) : x1slot(rn)) + hb + lane;
        const float* pe = lane == 0 || lane == 63
                              ? edges + (r & (kSlots - 1)) * kEdgeRow + (top ? 2 * m : 0) +
                                    (lane >> 5)
                              : zeros;
        // Software pipeline over chunks of D steps, so that a step costs its
        // instructions and not their latencies: while chunk c is eliminated
        // (two dependent operations per step), the right-hand sides of chunk
        // c + 1 are formed and the LDS loads of chunk c + 2 are in flight.
        struct Nbs {
            float c, s, n, e;
        } b[2][D];
        auto fetch = [&](int c) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                const int t = c * D + d;
                Nbs& v = b[c & 1][d];
                if constexpr (HAS_X) {
                    v.c = pc[t * 64];
                    v.s = ps[t * 64];
                    v.n = pn[t * 64];
                    if constexpr (FIRST) v.e = pe[t * 2];
                }
            }
        };
        float sv[2][D];
        auto form = [&](int c) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                const Nbs& v = b[c & 1][d];
                const int t = c * D + d < NS ? c * D + d : NS - 1;
                float s = fr[t];
                if constexpr (HAS_X) {
                    // west + east: the neighbour lanes', and the edge value
                    float we = FIRST ? v.e + from_below0(v.c) : from_below0(v.c);
                    we += from_above0(v.c);
                    s += fmaf(lane_value(q.z, t), v.n,
                              fmaf(lane_value(q.y, t), v.s, lane_value(q.x, t) * we));
                }
                sv[c & 1][d] = s;
            }
        };
        float y[NS];
        float vp = 0, cp = 0, sm = 0, im = 0;
        fetch(0);
        __builtin_amdgcn_sched_barrier(0);
        if (NC > 1) fetch(1);
        form(0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if (c + 1 < NC) form(c + 1);
            if (c + 2 < NC) fetch(c + 2);
#pragma unroll
            for (int d = 0; d < D; ++d) {
                const int t = c * D + d;
                if (t >= NS) continue;
                const float s = sv[c & 1][d];
                float w = fmaf(cp, vp, s) * ir[t];
                // computed here, not sunk (with its operands) to later blocks
                asm volatile("" : "+v"(w));
                y[t] = w;
                if (t < NS - G - 1 || t < elim) {
                    vp = w;
                    cp = lane_value(q.w, t);
                } else if (t == elim) {
                    sm = s;
                    im = ir[t];
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        float(*xc)[64] = xch[pair];
        if (!top) {
            xc[0][lane] = cp * vp;
        } else {
            xc[1][lane] = cp * vp;
            xc[2][lane] = sm;
            xc[3][lane] = im;
        }
        __syncthreads();
        const float xm = (xc[2][lane] + xc[0][lane] + xc[1][lane]) * xc[3][lane];
        float z = xm;
        float* po = ring + x1slot(r) + hb + lane;
        const uint32_t ov = uint32_t(r * nI + col) * 4u;
        // Every lane takes part, also those with no output column: the steps'
        // couplings lie in the lanes of q, which a branch here would leave out of
        // any copy of it. Only the stores are guarded, a chunk of them at a time.
        float xo[2][E];
        auto fetch_x = [&](int c) {
            if constexpr (HAS_X) {
#pragma unroll
                for (int d = 0; d < E; ++d) xo[c & 1][d] = pc[(c * E + d) * 64];
            }
        };
        fetch_x(NE - 1);
        Offsets soff = offsets;
#pragma unroll
        for (int c = NE - 1; c >= 0; --c) {
            soff.opaque();
            if (c > 0) fetch_x(c - 1);
            __builtin_amdgcn_sched_barrier(0);
            float out[E];
#pragma unroll
            for (int d = E - 1; d >= 0; --d) {
                const int t = c * E + d;
                if (t >= NS) continue;
                if (t < NS - G - 1 || t < elim)
                    z = fmaf(lane_value(q.w, t) * ir[t], z, y[t]);
                out[d] = omega * z;
                if constexpr (HAS_X) out[d] = fmaf(keep, xo[c & 1][d], out[d]);
                if constexpr (FIRST)
                    if (t < NS - G || t < own) po[t * 64] = out[d];
            }
            if constexpr (!FIRST)
                if (lane >= 1 && lane <= cn) {
#pragma unroll
                    for (int d = E - 1; d >= 0; --d) {
                        const int t = c * E + d;
                        if (t >= NS) continue;
                        if (t < NS - G || t < own) bst<false>(out[d], ro, ov, soff(t));
                    }
                }
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
    };
    auto idle = [&]() {
        __syncthreads();
        __syncthreads();
    };
    // rows of phase p with a first sweep, and with a second one two phases on
    auto has_first = [&](int p) { return p >= 0 && p <= B + 1 && r0 + p >= 0 && r0 + p < nJ; };
    auto has_second = [&](int p) { return p >= 1 && p <= B; };

    if (has_first(pair)) {
        load_part(Part0{}, r0 + pair);
        load_part(Part1{}, r0 + pair);
    }
    __syncthreads();   // the first rows of x are there
    for (int p = 0; p < pair && p < phases; ++p) idle();
    for (int p = pair; p < phases; p += kPairs) {
        if (has_first(p)) sweep_row(std::true_type{}, r0 + p, om1);
        else idle();
        if (p + 1 >= phases) break;
        idle();
        if (p + 2 >= phases) break;
        if (has_second(p)) sweep_row(std::false_type{}, r0 + p, om2);
        else idle();
        if (p + 3 >= phases) break;
        // the next row's loads, in two halves: a wavefront can have 63
        // memory operations in flight, and a 64th would hold up the phase
        const bool load = has_first(p + kPairs);
        if (load) load_part(Part0{}, r0 + p + kPairs);
        __syncthreads();
        if (load) load_part(Part1{}, r0 + p + kPairs);
        __syncthreads();
        if (p + 4 >= phases) break;
        idle();
    }
}

// The strips and bands of a level: strips as wide as possible, and about as
// many bands as fill every CU once (a block per CU; a band's first and last
// rows cost it three phases more than it has rows).
inline Strips strips_of(int nI, int nJ) {
    Strips s;
    s.count = (nI + kOut - 1) / kOut;
    s.width = (nI + s.count - 1) / s.count;
    const int bands = 256 / s.count > 0 ? 256 / s.count : 1;
    s.band = (nJ + bands - 1) / bands;
    return s;
}

}  // namespace

bool sweep_pair_fits(const LevelView<float>& L, size_t max_lds) {
    // A row takes more strips than single sweeps take segments of it, most so
    // short rows: 2 against 1 with 64 columns, 3 against 2 with 128. Single sweeps
    // are the faster there where they are compiled for about as many layers as
    // there are. V(2,2) cycles of two levels, single sweeps and pairs: 64x2048
    // with 17, 32 and 70 layers 104, 126, 232 and 109, 139, 237 us (33 and 69
    // layers, not compiled so: 174, 258 and 145, 235); 128x768 with 24 and 70
    // layers 95, 160 and 100, 166, 128x1024 101 (17), 212 and 100, 206.
    const bool close = L.nz <= 32 || L.nz == 70;
    const long long strips = strips_of(L.nI, L.nJ).count, segments = segments_per_row(L.nI);
    if (close && (2 * strips > 3 * segments ||
                  7 * segments * L.plane < 6 * strips * kPairColumns))
        return false;
    return L.nz >= 17 && L.nz <= 72 && L.nI >= 4 && L.plane >= kPairColumns &&
           pair_lds_values(L.nz, false) * sizeof(float) <= max_lds;
}

bool sweep_pair(const LevelView<float>& L, const float* f, const float* xin, float* xout,
                float om1, float om2, size_t max_lds, hipStream_t s) {
    if (!sweep_pair_fits(L, max_lds)) return false;
    const Strips st = strips_of(L.nI, L.nJ);
    const int nb = st.count * ((L.nJ + st.band - 1) / st.band);
    const size_t lds = pair_lds_values(L.nz, xin == nullptr) * sizeof(float);
    bool done = false;
    auto go = [&](auto ns, auto g, auto zero) {
        constexpr bool ZERO = decltype(zero)::value;
        auto* fn = &k_sweep_pair<decltype(ns)::value, decltype(g)::value, ZERO>;
        if (!allow_lds(fn, lds)) return;
        fn<<<nb, 64 * (2 * kPairs + kLoadWaves), lds, s>>>(L, f, xin, xout, om1, om2, st);
        done = true;
    };
    auto by_start = [&](auto ns, auto g) {
        if (xin) go(ns, g, std::false_type{});
        else go(ns, g, std::true_type{});
    };
    const int half = (L.nz + 1) / 2;
    using std::integral_constant;
    if (half <= 12) by_start(integral_constant<int, 12>{}, integral_constant<int, 4>{});
    else if (half <= 16) by_start(integral_constant<int, 16>{}, integral_constant<int, 4>{});
    else if (half <= 20) by_start(integral_constant<int, 20>{}, integral_constant<int, 4>{});
    else if (half <= 24) by_start(integral_constant<int, 24>{}, integral_constant<int, 4>{});
    else if (half <= 28) by_start(integral_constant<int, 28>{}, integral_constant<int, 4>{});
    else if (half <= 32) by_start(integral_constant<int, 32>{}, integral_constant<int, 4>{});
    else by_start(integral_constant<int, 36>{}, integral_constant<int, 4>{});
    return done;
}

}  // namespace mgk
