// group_dp.h -- exact chain TV prox with the deque spread over lanes (gfx950).
// Included by seg_kernels.h, whose types and helpers it uses.
//
// A lane that owns a whole deque (seg_kernels.h) takes a serial walk over the
// window per node: about 135-200 instructions and two LDS round trips, 0.5 to
// 1 us a node when a SIMD holds one wave.  That is the time of a launch with
// few chains (one 512 x 512 image: 128 waves on 1024 SIMDs).  Here a group of
// GW lanes (16, one DPP row, or a whole wave) owns the deque, one breakpoint
// per lane in registers, the deque's front at any lane of the group (a ring):
//  - a lane reads its neighbours by DPP rotation, no LDS;
//  - the message derivative at the breakpoints is the same chain of FMAs from
//    the front as dp_step_window's, run as rounds in which every lane takes its
//    left neighbour's value (round m completes lane m);
//  - every lane forms the two roots on the segments beside it, and wave masks
//    pick the lane whose root is lambda^- (the last breakpoint below w^-, or
//    the lane before the front) and the one whose root is lambda^+;
//  - those two lanes keep their root as the new breakpoint, the lanes outside
//    them empty themselves: nothing moves.
// Every rounded operation and its operands are those of dp_step_ring /
// dq_scan, so states, lambda pairs and x are the same bits.
//
// One workgroup solves one chain: its groups run the chain's segments with a
// halo, compare their halo state with the neighbour's end state through LDS,
// rerun from the true state where they differ until nothing changes (round k
// makes the first k + 1 segments final), and the clips are composed by a scan
// over the nodes (clips are closed under composition, and composing them
// rounds nothing).  So a launch is one kernel instead of five.  A step takes 0.4 us
// (FP64 0.75) at up to three waves a SIMD and 0.13 us more for each further one.
#pragma once

namespace tvc {
#pragma clang fp contract(off)

template <int CTRL> __device__ __forceinline__ int dpp_mov(int v) {
    return __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, true);
}
template <int CTRL> __device__ __forceinline__ float dpp_mov(float v) {
    return __int_as_float(dpp_mov<CTRL>(__float_as_int(v)));
}
template <int CTRL> __device__ __forceinline__ double dpp_mov(double v) {
    const long long b = __double_as_longlong(v);
    const unsigned lo = (unsigned)dpp_mov<CTRL>((int)(unsigned)b), hi = (unsigned)dpp_mov<CTRL>((int)(b >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
// Lane t of the lane's row of 16.
template <int t, typename T> __device__ __forceinline__ T row_bcast(T v) { return dpp_mov<0x150 + t>(v); }

// kGrpRounds rounds of v = fma(a, d, m ? b : v of the lane before), the rotation
// taken as the select's DPP operand; the compiler makes a move, a select and the
// FMA of each (1024 x 1024, us a 2D iteration: FP32 143 -> 138, FP64 252 -> 242).
// A DPP operand has to be two wait states old.
constexpr int kGrpRounds = 5;  // run between tests that every crossing was reached
#define TVC_GRP_ROUND32(rot) \
    "s_nop 1\n\tv_cndmask_b32_dpp %0, %0, %1, vcc " rot " row_mask:0xf bank_mask:0xf\n\tv_fmac_f32 %0, %2, %3\n\t"
#define TVC_GRP_ROUND64(rot)                                                             \
    "s_nop 1\n\tv_cndmask_b32_dpp %0, %2, %4, vcc " rot " row_mask:0xf bank_mask:0xf\n\t" \
    "v_cndmask_b32_dpp %1, %3, %5, vcc " rot " row_mask:0xf bank_mask:0xf"
#define TVC_GRP_ROUNDS(name, rot)                                                                         \
    __device__ __forceinline__ void name(float &v, float b, float a, float d, uint64_t m) {               \
        register uint64_t vcc asm("vcc") = m;                                                             \
        static_assert(kGrpRounds == 5, "");                                                               \
        asm(TVC_GRP_ROUND32(rot) TVC_GRP_ROUND32(rot) TVC_GRP_ROUND32(rot) TVC_GRP_ROUND32(rot)           \
                TVC_GRP_ROUND32(rot) "s_nop 1"                                                            \
            : "+v"(v)                                                                                     \
            : "v"(b), "v"(a), "v"(d), "s"(vcc));                                                          \
    }                                                                                                     \
    __device__ __forceinline__ void name(double &v, double b, double a, double d, uint64_t m) {           \
        register uint64_t vcc asm("vcc") = m;                                                             \
        _Pragma("unroll") for (int r = 0; r < kGrpRounds; ++r) {                                          \
            int lo, hi;                                                                                   \
            asm(TVC_GRP_ROUND64(rot)                                                                      \
                : "=&v"(lo), "=&v"(hi)                                                                    \
                : "v"(__double2loint(v)), "v"(__double2hiint(v)), "v"(__double2loint(b)),                 \
                  "v"(__double2hiint(b)), "s"(vcc));                                                      \
            v = fmav(a, d, __hiloint2double(hi, lo));                                                     \
        }                                                                                                 \
    }
TVC_GRP_ROUNDS(row_rounds, "row_ror:1")
TVC_GRP_ROUNDS(wave_rounds, "wave_ror:1")
#undef TVC_GRP_ROUND32
#undef TVC_GRP_ROUND64
#undef TVC_GRP_ROUNDS

// The lanes of a group as a ring: neighbours' values, and masks moved one lane
// towards the front.
// (A rotation reads lanes that take part in it only: no lane of the wave may be
// masked off where one is taken.)
template <int GW> struct Ring;
template <> struct Ring<16> {
    static constexpr uint64_t kFirst = 0x0001000100010001ull, kLast = 0x8000800080008000ull;
    template <typename T> static __device__ __forceinline__ T prev(T v) { return dpp_mov<0x121>(v); }  // row_ror:1
    template <typename T> static __device__ __forceinline__ T next(T v) { return dpp_mov<0x12F>(v); }  // row_ror:15
    template <typename T> static __device__ __forceinline__ void rounds(T &v, T b, T a, T d, uint64_t m) {
        row_rounds(v, b, a, d, m);
    }
    static __device__ __forceinline__ uint64_t before(uint64_t m) {
        return ((m >> 1) & ~kLast) | ((m & kFirst) << 15);
    }
    static __device__ __forceinline__ uint64_t bits(uint64_t m, int lane) { return (m >> (lane & 48)) & 0xffff; }
};
template <> struct Ring<64> {
    static constexpr uint64_t kFirst = 1ull, kLast = 1ull << 63;
    template <typename T> static __device__ __forceinline__ T prev(T v) { return dpp_mov<0x13C>(v); }  // wave_ror:1
    template <typename T> static __device__ __forceinline__ T next(T v) { return dpp_mov<0x134>(v); }  // wave_rol:1
    template <typename T> static __device__ __forceinline__ void rounds(T &v, T b, T a, T d, uint64_t m) {
        wave_rounds(v, b, a, d, m);
    }
    static __device__ __forceinline__ uint64_t before(uint64_t m) { return (m >> 1) | (m << 63); }
    static __device__ __forceinline__ uint64_t bits(uint64_t m, int) { return m; }
};

__device__ __forceinline__ bool lane_in(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }
__device__ __forceinline__ uint64_t lanes_where(bool p) { return __builtin_amdgcn_ballot_w64(p); }

// A deque per group.  front / back: the lanes of the first and last
// breakpoint (the last step's lambda^- and lambda^+); pre: the lane before the
// front; valid: the lanes that hold breakpoints (the others hold +inf).
template <typename T, typename G> struct GDeque {
    T l;
    G k;
    uint64_t front, pre, back, valid;
    uint64_t ovf;  // groups' lanes where a deque did not fit (fewer than GW breakpoints)
};

// One step (dp_step_ring) of every group of the wave.
template <typename T, typename G, bool kGen, int GW>
__device__ __forceinline__ void grp_step(GDeque<T, G> &S, const StepIn<T, G> &in) {
    using R = Ring<GW>;
    const EndSlope<T, G, kGen> es(in.sf, in.sprev);
    const T lo = in.lo, hi = in.hi;
    const T lamP = R::prev(S.l), lamN = R::next(S.l);
    const T slP = slope_of<T, G>(in.sf, R::prev(S.k)), sl = slope_of<T, G>(in.sf, S.k);
    const bool at0 = lane_in(S.front), pre = lane_in(S.pre);
    const T d = at0 ? (T)0 : S.l - lamP;
    const T v0 = es.mul(S.l) + (in.lop - in.yi);
    // v at this lane's breakpoint; lanes not reached yet hold +inf, above both levels
    T v = at0 ? v0 : pos_inf<T>();
    auto rounds = [&]() { R::rounds(v, v0, slP, d, S.front); };
    uint64_t mlo, left, right, keep;
    T vR;  // what lambda^+ is solved from: v at the breakpoint left of it
    bool deep = false;
    if constexpr (GW > kTwoEnded) deep = __popcll(S.valid) >= kTwoEnded;
    if (!deep) {
        uint64_t mhi;
        // the w^+ crossing; true if it is at a breakpoint not reached yet
        auto cross = [&]() {
            vR = R::prev(v);
            mhi = lanes_where(v <= hi);
            right = (lanes_where(vR <= hi) | S.front) & ~mhi;
            return (right & lanes_where(v == pos_inf<T>()) & S.valid) != 0;
        };
        rounds();
        if (cross()) {
            rounds();
            if (cross()) {
                rounds();
                cross();
            }
        }
        mlo = lanes_where(v < lo);
        left = (mlo | S.pre) & ~lanes_where(R::next(v) < lo);
        keep = mhi & ~mlo & S.valid;
    } else if constexpr (GW == 64) {
        // from kTwoEnded breakpoints on: w^- crossing from the front, w^+ crossing
        // walking from the back (dq_scan), one group per wave
        const int t = __popcll(S.valid);
        rounds();
        for (int done = kGrpRounds;; done += kGrpRounds) {
            mlo = lanes_where(v < lo);
            const uint64_t nxt = (lanes_where(R::prev(v) < lo) | S.front) & ~mlo;
            if (!(nxt & lanes_where(v == pos_inf<T>()) & S.valid) || done >= t) break;
            rounds();
        }
        left = (mlo | S.pre) & ~lanes_where(R::next(v) < lo);
        const bool atB = lane_in(S.back);
        const T u0 = es.mul(S.l) + (in.hip - in.yi), dN = S.l - lamN;
        T u = atB ? u0 : pos_inf<T>();
        for (int done = 1; !(lanes_where(u <= hi) & S.valid) && done < t; done += 4) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const T e = fmav(sl, dN, R::next(u));
                u = atB ? u0 : e;
            }
        }
        vR = R::prev(u);
        const uint64_t ulo = lanes_where(u <= hi) & S.valid;
        right = ((ulo << 1) | (ulo >> 63)) & ~ulo;
        const uint64_t after = (left << 1) | (left >> 63);
        if (!right || (right & mlo)) right = after;  // r is raised to p
        const int lane = threadIdx.x & 63, h = __ffsll((unsigned long long)S.front) - 1;
        const int j = (lane - h) & 63, p = (__ffsll((unsigned long long)left) - h) & 63,
                  r = (__ffsll((unsigned long long)right) - 1 - h) & 63;
        keep = lanes_where(j >= p && j < r) & S.valid;
    }
    const uint64_t on_left = ((GW == 64) ? ((left << 1) | (left >> 63))
                                         : (((left & ~R::kLast) << 1) | ((left & R::kLast) >> 15)));
    // lambda^- on the segment right of this lane's breakpoint, or on the left
    // end piece (slope a_s) for the lane before the front
    const T vN = R::next(v);
    const T X = pre ? vN : v, base0 = pre ? lamN : S.l;
    const T rr = pre ? es.ra : recip(sl);
    const T lm = clampv(fmav(lo - X, rr, base0), pre ? -pos_inf<T>() : S.l, lamN);
    // lambda^+ on the segment left of this lane's breakpoint; from lambda^-
    // where both lie on one segment
    const bool same = lane_in(on_left);
    // (every lane takes part in each rotation: none may sit behind a condition)
    const T lmP = R::prev(lm), rrP = R::prev(rr);
    const T base = same ? lmP : lamP, span = hi - lo, gap = hi - vR;
    const T lp = clampv(fmav(same ? span : gap, rrP, base), base, S.l);
    const bool isL = lane_in(left), isR = lane_in(right);
    const G kk = pre ? in.sprev : S.k;
    S.k = isR ? in.sf : kk;
    const T kept = lane_in(keep) ? S.l : pos_inf<T>(), lr = isR ? lp : kept;
    S.l = isL ? lm : lr;
    S.front = left;
    S.back = right;
    S.pre = R::before(left);
    S.valid = left | right | keep;
    S.ovf |= right & (left | S.pre);
}

// ---------------------------------------------------------------------------
// One chain per workgroup.
// ---------------------------------------------------------------------------
struct GrpLds {
    void *lam;    // [S * L] pairs (lds_lam)
    void *l, *k;  // end states [2 * threads] (group g's entries from 2 g * GW, at most 64)
    int *size;    // [groups] (-1: no end state yet)
    int *need;    // [groups + 1] the state entering a segment changed
    int *wide;    // [groups + 1] the segments of a pass that outgrew 16 lanes; their number first
    int *deep;    // a deque outgrew a wave
    void *w;      // [2 * waves] the waves' composed clips
};
template <class Prob>
struct GroupOk : std::bool_constant<!IsL1<Prob>::value> {};

// Solves chain c with groups of GW lanes; false (for the whole workgroup) if a
// deque outgrew a wave (then *sh.deep too), or an end state its 2 GW entries.  Where the
// block has `side` chains, also (and *sh.deep) if more than 3 / side of the segments of a
// pass outgrow 16 lanes: a wave runs neighbouring ones one after the other, 0.8 us a node
// (FP64 1.6), grp_deep_chains the chains side by side, 1.2 us and more (us, 16384 x 512
// ramps at w = 3: 2260, all by waves 25400; 4096 x 4096 random walks, a part of whose
// segments are wide, with 0.4 in place of 3 / side 11200, 3780 by waves).  A segment whose deque
// outgrows 16 lanes is run again in the same pass by a whole wave, from its
// neighbour's end state (the wide segments of a pass, a wave each): deques of 16
// to 23 breakpoints come up in a few segments of many chains of a 2D iteration
// from lambda = 1.5 sigma on (us an iteration, FP32, sigma = 0.1; in brackets with
// the whole chain run again by waves: 512 x 512 at lambda = 0.2 237 (342), 1024 x
// 1024 at 0.15 457 (742), at 0.25 726 (924)).  kStream: lambda may be kept in the
// stream (without a store to it in the step loop, the next tile's loads are waited
// for a tile later; with one, before the loop).
template <typename T, class Prob, int GW, bool kStream>
__device__ bool grp_chain(const WsOf<T, Prob> &ws, const typename Prob::Params &pp, const ChainSpan &sp, int64_t c,
                          const GrpGeom &gm, const GrpLds &sh, int L, int side = 0) {
    using R = Ring<GW>;
    using G = typename Prob::Tag;
    constexpr bool kGen = Prob::kGen;
    constexpr int E = GW == 16 ? 32 : 64;  // entries of a saved end state
    const int tid = threadIdx.x, lane = tid & 63, gl = tid & (GW - 1), g = tid / GW;
    const int n = (int)sp.n, H = gm.H, nw = blockDim.x >> 6, wave = tid >> 6;
    const bool act = g * L < n;
    const auto src = Prob::src(pp, sp);
    T *lamL = (T *)sh.lam;
    T *const esl = (T *)sh.l;
    G *const esk = (G *)sh.k;
    // the lambda pair of node i: (lo, hi) at lds + 2 i, or in the stream
    auto put = [&](int i, int which, T v) {
        if (!kStream || gm.lds_lam)
            lamL[2 * i + which] = v;
        else if (i < n)
            ((T *)(ws.lam + (int64_t)i * ws.C + c))[which] = v;
    };
    // Runs the nodes from `halo` before a to the segment's end in tiles of 16
    // (nodes before the chain's start are skipped) with groups of W lanes;
    // `fresh`: from an empty deque at the first node, else continuing S.  at_a()
    // is called before node a.
    auto run = [&](auto width, GDeque<T, G> &S, int a, int halo, bool fresh, bool store, auto at_a) {
        constexpr int W = decltype(width)::value;
        using RW = Ring<W>;
        const int gw = tid & (W - 1);
        const int from = a - halo, tiles = (halo + L) / 16;
        // tiles before the chain's start in every group of the wave (2D 64 x 64: 59 -> 44
        // us an iteration)
        int q = 0;
        while (16 * q < halo && !lanes_where(a < n && from + 16 * q >= 0)) ++q;
        int i0 = from + 16 * q;
        const int h0 = from > 0 ? from : 0;
        StepIn<T, G> in;
        in.lop = (T)0;
        in.hip = (T)0;
        G first = (G)0, last = (G)0;  // general a_i: the sums before the first node and of the chain
        if (from > 0 && a < n) {
            if constexpr (kGen) first = src.prefix_before(from);
            if (!fresh) {
                const auto pv = src.load(from - 1);
                if constexpr (kGen) {
                    in.lop = src.wlo(pv);
                    in.hip = src.whi(pv);
                } else {
                    in.hip = src.weight(pv);
                }
            }
        }
        if constexpr (kGen) {
            if (a < n && a + L > n) last = src.prefix_before(n);
        }
        in.sprev = first;
        // A lane's node of a tile: what is loaded, and the step's inputs from it.  The
        // root has a zero edge; nodes past the chain's end, run to fill a tile, get
        // constant data and weight, on which a deque stays short.
        struct Tile {
            T y, lo, hi;
            G s;
        };
        auto load = [&](int i) {
            const int j = i + (lane & 15);
            return src.load(j < 0 ? 0 : (j < n ? j : n - 1));
        };
        auto inputs = [&](const typename Prob::Pre &pv, int i, Tile &t) {
            const int j = i + (lane & 15);
            t.y = src.data(pv);
            const T end = j == n - 1 ? (T)0 : (T)1;
            if constexpr (kGen) {
                t.lo = j < n - 1 ? src.wlo(pv) : -end;
                t.hi = j < n - 1 ? src.whi(pv) : end;
                // the anchor's group of 8 summed left to right
                t.s = src.prefix(pv, j, (G)0);
#pragma unroll
                for (int r = 0; r < 7; ++r) t.s = src.prefix(pv, j, Ring<16>::prev(t.s));
                if (j >= n) t.s = last + (G)(j - n + 1);
            } else {
                t.hi = j < n - 1 ? src.weight(pv) : end;
            }
        };
        Tile t, tn;
        typename Prob::Pre pn = load(i0);
        if constexpr (!kGen) inputs(pn, i0, t);
        S.ovf = 0;
        for (; q < tiles; ++q, i0 += 16) {
            if (16 * q == halo) at_a();
            if constexpr (kGen) {  // (its sums wait for the loads: formed a tile later)
                inputs(pn, i0, t);
                pn = load(i0 + 16);
            } else {
                pn = load(i0 + 16);
                inputs(pn, i0 + 16, tn);
            }
            const uint64_t im = lanes_where(fresh && i0 == h0);
            const uint64_t st = lanes_where(store && a < n && i0 >= a);
            const uint64_t live = lanes_where(i0 >= h0);
            if constexpr (kGen)
                in.sprev = lane_in(im) ? first : in.sprev;
            else
                in.sf = (G)(i0 + 1);
            uint64_t init = im;
            // lane k of the row holds node i0 + k: the tile turns by one lane a node
#pragma unroll 1
            for (int k = 0; k < 16; ++k) {
                in.yi = row_bcast<0>(t.y);
                in.hi = row_bcast<0>(t.hi);
                t.y = Ring<16>::next(t.y);
                t.hi = Ring<16>::next(t.hi);
                if constexpr (kGen) {
                    in.lo = row_bcast<0>(t.lo);
                    in.sf = row_bcast<0>(t.s);
                    t.lo = Ring<16>::next(t.lo);
                    t.s = Ring<16>::next(t.s);
                } else {
                    in.lo = -in.hi;
                    in.lop = -in.hip;
                    in.sprev = in.sf - (G)1;
                }
                grp_step<T, G, kGen, W>(S, in);
                if (init) {  // an empty message: breakpoints (b_s + w^-) / a_s and (b_s + w^+) / a_s
                    if (lane_in(init)) {
                        const EndSlope<T, G, kGen> es(in.sf, in.sprev);
                        S.l = gw == 0 ? es.div(in.yi + in.lo) : (gw == 1 ? es.div(in.yi + in.hi) : pos_inf<T>());
                        S.k = gw == 0 ? in.sprev : in.sf;
                    }
                    S.front = (S.front & ~init) | (RW::kFirst & init);
                    S.pre = (S.pre & ~init) | (RW::kLast & init);
                    S.back = (S.back & ~init) | ((RW::kFirst << 1) & init);
                    S.valid = (S.valid & ~init) | ((RW::kFirst | (RW::kFirst << 1)) & init);
                    S.ovf &= ~init;
                    init = 0;
                }
                S.ovf &= live;
                if (lane_in((S.front | S.back) & st)) put(i0 + k, lane_in(S.back) ? 1 : 0, S.l);
                in.hip = in.hi;
                if constexpr (kGen) {
                    in.lop = in.lo;
                    in.sprev = in.sf;
                } else {
                    in.sf += (G)1;
                }
            }
            if constexpr (!kGen) t = tn;
        }
    };
    // The deque of m breakpoints at esl / esk[at ..], or an empty one.
    auto load = [&](auto width, GDeque<T, G> &S, int m, int at) {
        constexpr int W = decltype(width)::value;
        const int gw = tid & (W - 1);
        S.l = gw < m ? esl[at + gw] : pos_inf<T>();
        S.k = gw < m ? esk[at + gw] : (G)0;
        S.front = Ring<W>::kFirst;
        S.pre = Ring<W>::kLast;
        S.valid = lanes_where(gw < m);
        S.back = lanes_where(gw == (m > 0 ? m - 1 : 0));
        S.ovf = 0;
    };
    // breakpoints of S in order: this lane's place, and the deque's size
    auto order = [&](auto width, const GDeque<T, G> &D, int &j, int &size) {
        constexpr int W = decltype(width)::value;
        const int h = __ffsll((unsigned long long)Ring<W>::bits(D.front, lane)) - 1;
        j = (tid - h) & (W - 1);
        size = __popcll(Ring<W>::bits(D.valid, lane));
    };
    // S as the end state of segment q, whose breakpoint j this lane holds; a
    // state that differs from the last one is written and told to q's neighbour
    auto end_state = [&](auto width, const GDeque<T, G> &S, int q, int j, int size, bool on) {
        constexpr int W = decltype(width)::value;
        bool differs = on && size != sh.size[on ? q : 0];
        if (on && !differs && j < size) differs = !ent_same<T>(esl[q * E + j], esk[q * E + j], S.l, S.k);
        if (Ring<W>::bits(lanes_where(differs), lane)) {
            if (j < size) {
                esl[q * E + j] = S.l;
                esk[q * E + j] = S.k;
            }
            if ((tid & (W - 1)) == 0) {
                sh.size[q] = size;
                sh.need[q + 1] = 1;
            }
        }
    };
    constexpr auto kGroup = std::integral_constant<int, GW>{};
    constexpr auto kWave = std::integral_constant<int, 64>{};
    // the state a segment was last run from (first the deque after its halo)
    T hl = pos_inf<T>();
    G hk = (G)0;
    int hj = 0, hsize = 0;
    auto group_any = [&](bool p) { return R::bits(lanes_where(p), lane) != 0; };
    // The first pass runs every segment with its halo; later ones run the
    // segments whose incoming deque was not the true one again from it.  A pass
    // makes at least one more segment final, so there are at most as many as
    // segments.
    bool mine = act, wide = false;
    if (gl == 0) sh.size[g] = -1;
#pragma unroll 1
    for (int pass = 0; pass <= (int)blockDim.x / GW; ++pass) {
        GDeque<T, G> S;
        const int m = (pass > 0 && mine) ? sh.size[g - 1] : 0;
        if (GW == 16 && m >= GW) wide = true;
        const bool here = mine && !wide;
        load(kGroup, S, here ? m : 0, (g - 1) * E);
        if (GW == 16 && tid == 0) sh.wide[0] = 0;
        __syncthreads();  // the states have been read
        if (gl == 0) sh.need[g + 1] = 0;
        bool bad = false;
        if (lanes_where(here)) {
            if (pass > 0 && here) {
                hl = S.l;
                hk = S.k;
                hj = gl;
                hsize = m;
            }
            run(kGroup, S, g * L, pass == 0 ? H : 0, pass == 0, here, [&]() {
                if (pass == 0) {
                    order(kGroup, S, hj, hsize);
                    hl = S.l;
                    hk = S.k;
                }
            });
            bad = here && R::bits(S.ovf, lane) != 0;
            int j, size;
            order(kGroup, S, j, size);
            end_state(kGroup, S, g, j, size, here && !bad);
        }
        if constexpr (GW == 16) {
            if (bad) wide = true;
            if (mine && wide && gl == 0) sh.wide[1 + atomicAdd(sh.wide, 1)] = g;
            __syncthreads();
            const int count = sh.wide[0];
            if ((int64_t)count * L * side > 3 * (int64_t)n) {
                if (tid == 0) *sh.deep = 1;
                return false;
            }
            bad = false;
            for (int q0 = 0; q0 < count; q0 += nw) {
                // (a segment whose neighbour has no end state yet waits for it)
                const int q = __builtin_amdgcn_readfirstlane(q0 + wave < count ? sh.wide[1 + q0 + wave] : -1);
                const int mq = __builtin_amdgcn_readfirstlane(q > 0 ? sh.size[q - 1] : 0);
                const bool go = q >= 0 && mq >= 0;
                load(kWave, S, go ? mq : 0, (q - 1) * E);
                if (go && lane == 0) sh.need[q] = 0;
                __syncthreads();
                if (go) {
                    run(kWave, S, q * L, 0, q == 0, true, []() {});
                    int j, size;
                    order(kWave, S, j, size);
                    bad = S.ovf != 0 || size > E;
                    if (S.ovf != 0) *sh.deep = 1;
                    if (!bad) end_state(kWave, S, q, j, size, true);
                }
                if (__syncthreads_or(bad)) return false;
            }
        } else if (__syncthreads_or(bad)) {
            if (tid == 0) *sh.deep = 1;
            return false;
        }
        bool need = act && g > 0 && sh.need[g] != 0;
        if (need && !wide) {
            need = sh.size[g - 1] != hsize;
            if (!need && hj < hsize) need = !ent_same<T>(esl[(g - 1) * E + hj], esk[(g - 1) * E + hj], hl, hk);
        }
        mine = group_any(need);
        if (!__syncthreads_or(mine)) break;
    }
    // x from the composed clips, a block of blockDim.x nodes at a time from the
    // end: a suffix scan of (lo, hi) over the wave, then over the waves
    const auto sink = Prob::sink(pp, sp);
    T *sw = (T *)sh.w;
    T xin = (T)0;
    for (int c0 = (n - 1) / (int)blockDim.x * (int)blockDim.x; c0 >= 0; c0 -= (int)blockDim.x) {
        const int i = c0 + tid;
        T lo = -pos_inf<T>(), hi = pos_inf<T>();
        typename Prob::SinkPre sv;
        if (i < n) {
            sv = sink.load(i);
            if (!kStream || gm.lds_lam) {
                lo = lamL[2 * i];
                hi = lamL[2 * i + 1];
            } else {
                const LamPair<T> p = ws.lam[(int64_t)i * ws.C + c];
                lo = p.lo;
                hi = p.hi;
            }
            if (i == n - 1) hi = lo;
        }
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const T olo = __shfl_down(lo, off, 64), ohi = __shfl_down(hi, off, 64);
            if (lane + off < 64) {
                const T l2 = clampv(olo, lo, hi), h2 = clampv(ohi, lo, hi);
                lo = l2;
                hi = h2;
            }
        }
        if (lane == 0) {
            sw[2 * wave] = lo;
            sw[2 * wave + 1] = hi;
        }
        __syncthreads();
        T xr = xin;
        for (int q = nw - 1; q >= 0; --q) {
            if (q == wave) xr = xin;
            xin = clampv(xin, sw[2 * q], sw[2 * q + 1]);
        }
        if (i < n) sink.store(i, clampv(xr, lo, hi), sv);
        __syncthreads();
    }
    return true;
}

// A deque of one lane in LDS: a ring of cap entries, for dq_scan and dq_update.
template <typename T, typename G> struct LdsDeque {
    G *k;
    T *l;
    int cap, head, size;
    __device__ __forceinline__ int at(int j) const {
        const int i = head + j;
        return i < 0 ? i + cap : (i >= cap ? i - cap : i);
    }
    __device__ __forceinline__ Ent<T, G> ld(int j) const { return mk_ent<T, G>(l[at(j)], k[at(j)]); }
    __device__ __forceinline__ void put(int j, const Ent<T, G> &e) const {
        l[at(j)] = e.l;
        k[at(j)] = e.k;
    }
    __device__ __forceinline__ void shift(int d) { head = at(d); }
};

// The whole chain on one lane with its deque in LDS (cap entries at k and l), lambda in
// the stream; false if the deque outgrew them.
template <typename T, class Prob>
__device__ bool grp_lane_chain(const WsOf<T, Prob> &ws, const typename Prob::Params &pp, const ChainSpan &sp, int64_t c,
                               typename Prob::Tag *k, T *l, int cap) {
    using G = typename Prob::Tag;
    constexpr bool kGen = Prob::kGen;
    const auto src = Prob::src(pp, sp);
    auto cy = carry_before<T, Prob>(src, 0);
    LdsDeque<T, G> D{k, l, cap, 0, 0};
    D.put(0, mk_ent<T, G>(pos_inf<T>(), (G)0));
    for (int64_t i = 0; i < sp.n; ++i) {
        if (D.size + 3 > cap) return false;  // a step writes one entry before the front and two past the back
        const auto pr = src.load(i);
        const auto in = step_in<T, Prob>(src, pr, i, i == sp.n - 1, cy);
        const EndSlope<T, G, kGen> es(in.sf, in.sprev);
        const DqScan<T> sc = dq_scan<T, G, kGen, true>(D, D.size, in, es);
        const int i0 = sc.p > 0 ? sc.p - 1 : 0, i1 = sc.r > 0 ? sc.r - 1 : 0;
        T lm, lp;
        G tnew;
        dq_solve<T, G, kGen>(sc, in, es, D.size == 0, D.ld(i0), D.ld(i0 + 1), D.ld(i1), D.ld(i1 + 1), lm, lp, tnew);
        D.size = dq_update<T, G>(D, sc, in.sf, lm, lp, tnew);
        put_lam<T>(ws.lam, i, ws.C, c, lm, i == sp.n - 1 ? lm : lp);
    }
    full_backward<T, Prob>(ws, pp, sp, c);
    return true;
}

// The block's chains with more than 63 breakpoints (the first `nd` of its slots of the
// list), a lane of its first wave each, all of the block's LDS shared out among them;
// those that outgrow their share again with fewer lanes, and at last in HBM.  A single
// chain goes there at once where its block has an HBM deque (1000 x 300 ramps, w = 30:
// 570 us, 735 in LDS).  us, many chains, ramps at w = 30, the ring of a lane each of the
// kernel for TV-l1 / one lane of a block in HBM / this: 4096 x 4096 20100 / 50000 / 8030,
// FP64 64500 / 109000 / 16700, 16384 x 512 12700 / 30000 / 2910.
template <typename T, class Prob, bool kList>
__device__ void grp_deep_chains(const WsOf<T, Prob> &ws, const typename Prob::Params &pp, int64_t nd, char *mem,
                                int lds) {
    using G = typename Prob::Tag;
    const int lane = threadIdx.x, all = lds / (int)(sizeof(T) + sizeof(G));
    const int64_t slots = ws.fb_lanes / gridDim.x;
    for (int most = kList || slots < 1 ? 64 : 0; nd > 0; most /= 8) {
        const bool hbm = most == 0;  // after 64, 8 and 1 lanes
        int lanes = hbm ? (int)(slots < 64 ? slots : 64) : most;
        if (lanes < 1) return;  // (the LDS holds any deque of a launch without slots)
        lanes = nd < lanes ? (int)nd : lanes;
        const int cap = (all / lanes - 1) | 1;  // odd: the lanes' deques lie in different banks
        int64_t failed = 0;
        for (int64_t at = 0; at < nd; at += lanes) {
            int *const slot = ws.ovf_list + blockIdx.x;
            bool bad = false;
            int c = 0;
            if (lane < lanes && at + lane < nd) {
                c = slot[(at + lane) * gridDim.x];
                const ChainSpan sp = Prob::span(pp, c, ws.n);
                if (hbm)
                    seg_full_chain<T, Prob>(ws, pp, sp, c, blockIdx.x + (int64_t)lane * gridDim.x);
                else
                    bad = !grp_lane_chain<T, Prob>(ws, pp, sp, c, (G *)mem + (int64_t)lane * cap,
                                                   (T *)((G *)mem + (int64_t)lanes * cap) + (int64_t)lane * cap, cap);
            }
            const uint64_t m = lanes_where(bad);
            if (bad) slot[(failed + __popcll(m & ((1ull << lane) - 1))) * gridDim.x] = c;
            failed += __popcll(m);
            __threadfence_block();
        }
        nd = failed;
    }
}

// A launch over all chains (kList false, a block each), or over the chains in ws.ovf_list.
// Segments whose deque outgrows a group of 16 are run by a whole wave (grp_chain),
// chains with more than 31 breakpoints at a segment's end with a wave per segment,
// and chains with more than 63 breakpoints are left for the end (grp_deep_chains).
template <typename T, class Prob, bool kList>
__global__ __launch_bounds__(1024) void k_chain_wg(WsOf<T, Prob> ws, typename Prob::Params pp, GrpGeom gm) {
    extern __shared__ __align__(16) char s_grp[];
    if (seg_stopped(ws)) return;
    const int S16 = (int)blockDim.x / 16;
    GrpLds sh;
    {
        char *p = s_grp;
        sh.k = p;
        p += 2 * sizeof(typename Prob::Tag) * blockDim.x;
        sh.l = p;
        p += 2 * sizeof(T) * blockDim.x;
        sh.w = p;
        p += 2 * sizeof(T) * (blockDim.x / 64);
        sh.size = (int *)p;
        p += sizeof(int) * S16;
        sh.need = (int *)p;
        p += sizeof(int) * (S16 + 4);
        sh.wide = (int *)p;
        p += sizeof(int) * (S16 + 4);
        sh.deep = (int *)p;
        p += 4 * sizeof(int);
        sh.lam = p;
    }
    const int64_t count = kList ? (int64_t)*ws.ovf_count : ws.C;
    const int side = kList ? (int)((count + gridDim.x - 1) / gridDim.x) : 0;
    int64_t deep = 0;
    for (int64_t q = blockIdx.x; q < count; q += gridDim.x) {
        // neighbouring chains on one XCD (blocks go round the eight XCDs in turn):
        // neighbouring columns share cache lines
        const int64_t x = q & 7, per = count >> 3, rem = count & 7;
        const int64_t c = kList ? (int64_t)ws.ovf_list[q] : x * per + (x < rem ? x : rem) + (q >> 3);
        const ChainSpan sp = Prob::span(pp, c, ws.n);
        if (sp.n <= 0) continue;
        if (threadIdx.x == 0) *sh.deep = 0;
        bool done = grp_chain<T, Prob, 16, kList>(ws, pp, sp, c, gm, sh, gm.L, side);
        if (!done) {
            __syncthreads();
            if (*sh.deep == 0) {
                const int waves = (int)blockDim.x / 64;
                const int Lw = (int)((sp.n + waves - 1) / waves + 15) / 16 * 16;
                done = grp_chain<T, Prob, 64, kList>(ws, pp, sp, c, gm, sh, Lw);
            }
        }
        if (!done) {
            if (threadIdx.x == 0) ws.ovf_list[blockIdx.x + deep * gridDim.x] = (int)c;
            ++deep;
        } else if constexpr (kList) {  // the segments' tails are done
            for (int64_t s = threadIdx.x; s * ws.L < sp.n; s += blockDim.x)
                ws.seg_unc[s * ws.C + c] = (int)((s + 1) * ws.L < sp.n ? (s + 1) * ws.L : sp.n);
        }
        __syncthreads();
    }
    if (deep && threadIdx.x < 64) grp_deep_chains<T, Prob, kList>(ws, pp, deep, s_grp, gm.lds);
}

#pragma clang fp contract(fast)
}  // namespace tvc
