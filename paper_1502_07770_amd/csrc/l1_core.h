// l1_core.h -- one step of the TV-l1 chain prox (Sec. 4.2, piecewise-quadratic
// unaries), on any sorted breakpoint store:
//
//     x = argmin_x  sum_e w_e |x_{e+1} - x_e| + sum_i (x_i - y_i)^2 / 2 + sum_i c_i |x_i - d_i| .
//
// The derivative h of the message is non-decreasing, piecewise linear and may
// jump.  With unit quadratic weights every linear piece has an integer slope
// s - k (s = i + 1 unaries added so far; k the step at which the piece was a
// flat end), so a breakpoint holds its position lam, the tag k of the piece to
// its right and the jump of h at lam (>= 0).  The pieces beyond either end
// have slope 1 once the current unary is added; the left end's value is the
// previous clip level w^- plus the unary's left part, the right end's
// likewise.  The back breakpoint's right piece is the right end: its tag is
// kept at 0 (a canonical value, so equal sets compare equal entry by entry).
//
// Adding the unary g_i = z - y_i + c_i sign(z - d_i) inserts a breakpoint at
// d_i with jump 2 c_i; the clip to [-w_i, w_i] scans each end, pops the
// breakpoints it passes and pushes the crossing point.  A crossing at a jump
// replaces that breakpoint with the part of its jump inside the clip range
// (the update of FindMin's increment in Sec. 4.2), so every stored jump stays
// >= 0.
//
// A store provides: size, ovf (set when a push finds it full; the run is then
// discarded), get(j) / put(j, e) on logical positions, pop_front / pop_back,
// push_front / push_back and insert(q, e) keeping the order.
#pragma once
#include "chain_core.h"

namespace tvc {

// Every rounded operation of the DP is the one written: no multiply-add
// contraction (FMAs are explicit), so each step rounds the same in every
// kernel that inlines it and in every build, which the bit-for-bit comparison
// of segment states and the segmented = sequential results rely on.
#pragma clang fp contract(off)


// Slope tag and value jump of a TV-l1 breakpoint.
template <typename T>
struct TagJ {
    T k, j;
};
template <typename T>
__device__ __forceinline__ bool operator==(const TagJ<T> &a, const TagJ<T> &b) {
    return a.k == b.k && a.j == b.j;
}

template <typename T>
struct L1E {
    T l, k, j;  // position, tag of the piece to the right, jump at l
};

// The set in a plain per-lane array in HBM (the fallback), starting in its
// middle: at most one front push per node, and at most three pushes per node.
template <typename T>
struct L1ArrayStore {
    T *lam;
    TagJ<T> *tj;
    int64_t head, size, cap;
    bool ovf;
    __device__ __forceinline__ void init(T *l, TagJ<T> *t, int64_t capacity, int64_t front_room) {
        lam = l;
        tj = t;
        cap = capacity;
        head = front_room;
        size = 0;
        ovf = false;
    }
    __device__ __forceinline__ L1E<T> get(int64_t j) const {
        const TagJ<T> t = tj[head + j];
        return L1E<T>{lam[head + j], t.k, t.j};
    }
    __device__ __forceinline__ void put(int64_t j, const L1E<T> &e) const {
        lam[head + j] = e.l;
        tj[head + j] = TagJ<T>{e.k, e.j};
    }
    __device__ __forceinline__ void pop_front(int64_t k) {
        head += k;
        size -= k;
    }
    __device__ __forceinline__ void pop_back(int64_t k) { size -= k; }
    __device__ __forceinline__ void push_front(const L1E<T> &e) {
        if (head <= 0) {
            ovf = true;
            return;
        }
        --head;
        ++size;
        put(0, e);
    }
    __device__ __forceinline__ void push_back(const L1E<T> &e) {
        if (head + size >= cap) {
            ovf = true;
            return;
        }
        ++size;
        put(size - 1, e);
    }
    __device__ __forceinline__ void insert(int64_t q, const L1E<T> &e) {
        if (head + size >= cap) {
            ovf = true;
            return;
        }
        for (int64_t j = size; j > q; --j) put(j, get(j - 1));
        ++size;
        put(q, e);
    }
};

// The point where h crosses level v from below, scanning from the left:
// h(z) <= v <= h(z+), with h(z) = z + base on the left end piece.  Returns z
// and sets p (breakpoints passed), jump (the crossing is the jump of
// breakpoint p; vj is then h just right of it) and the tag of the piece the
// crossing lies in.
template <typename T, class St>
__device__ __forceinline__ T l1_cross_left(const St &S, T s, T base, T v, int &p, bool &jump, T &vj, T &tagc) {
    const int t = (int)S.size;
    jump = false;
    vj = (T)0;
    if (t == 0) {
        p = 0;
        tagc = s - (T)1;
        return v - base;  // slope 1
    }
    L1E<T> e = S.get(0);
    T vl = e.l + base;  // h just left of the first breakpoint
    if (vl >= v) {
        p = 0;
        tagc = s - (T)1;
        return e.l - (vl - v);
    }
    int j = 0;
    for (;;) {
        const T vr = vl + e.j;
        if (vr >= v) {
            p = j;
            jump = true;
            vj = vr;
            tagc = e.k;
            return e.l;
        }
        if (j + 1 == t) {  // right end piece, slope 1
            p = t;
            tagc = s - (T)1;
            return e.l + (v - vr);
        }
        const L1E<T> nx = S.get(j + 1);
        const T sl = s - e.k;
        const T vn = vr + sl * (nx.l - e.l);  // h just left of the next breakpoint
        if (vn >= v) {
            p = j + 1;
            tagc = e.k;
            return clampv(e.l + (v - vr) * recip(sl), e.l, nx.l);
        }
        vl = vn;
        e = nx;
        ++j;
    }
}

// One forward step at node i (s = i + 1); lop / hip are the clip levels of the
// previous edge, lo / hi those of the leaving edge.  An empty store (the first
// node of a chain, or the start of a run from an assumed zero message) has no
// previous clip: lop = hip = 0 there.  At the root only lm (the zero of h) is
// computed.
template <typename T, class St>
__device__ __forceinline__ void l1_step(St &S, T s, T yi, T di, T ci, T lop, T hip, T lo, T hi, bool root, T &lm,
                                        T &lp) {
    if (S.size == 0) {
        lop = (T)0;
        hip = (T)0;
    }
    // (a) add the unary: the data breakpoint at d_i with jump 2 c_i
    if (ci > (T)0) {
        const int t = (int)S.size;
        int q = 0;
        while (q < t && S.get(q).l <= di) ++q;
        // the new breakpoint splits a piece and inherits its tag; the end pieces
        // have slope 1 (tag s - 1); beyond the back, the old back's right piece
        // becomes interior (slope 1) and the new breakpoint is the back (tag 0)
        T g;
        if (q == t) {
            if (t > 0) {
                L1E<T> b = S.get(t - 1);
                b.k = s - (T)1;
                S.put(t - 1, b);
            }
            g = (T)0;
        } else {
            g = (q == 0) ? s - (T)1 : S.get(q - 1).k;
        }
        S.insert(q, L1E<T>{di, g, (T)2 * ci});
        if (S.ovf) {  // the run is discarded; keep every access in bounds
            lm = lp = (T)0;
            return;
        }
    }
    const T basel = lop - yi - ci;  // left end: h(z) = z + basel
    const T baser = hip - yi + ci;  // right end: h(z) = z + baser
    int p;
    bool jump;
    T vj, tagc;
    lm = l1_cross_left<T>(S, s, basel, root ? (T)0 : lo, p, jump, vj, tagc);
    if (root) return;
    // (b) left clip: flat at lo left of lm; a crossed jump keeps its part above lo
    const int t0 = (int)S.size;
    const bool all = !jump && p == t0;  // lm lies on the right end piece
    if (jump) {
        const T jm = vj - lo;
        S.pop_front(p + 1);
        S.push_front(L1E<T>{lm, (p + 1 == t0) ? (T)0 : tagc, jm < (T)0 ? (T)0 : jm});
    } else {
        S.pop_front(p);
        S.push_front(L1E<T>{lm, all ? (T)0 : tagc, (T)0});
    }
    if (S.ovf) {
        lp = lm;
        return;
    }
    // (c) right clip: flat at hi right of lp; never passes the front entry
    const int t = (int)S.size;
    int j = t - 1;
    L1E<T> e = S.get(j);
    T ur = e.l + baser;  // h just right of the back breakpoint (right end piece)
    if (ur <= hi) {
        lp = e.l + (hi - ur);  // slope 1
        e.k = s - (T)1;         // its right piece is now interior, slope 1
        S.put(j, e);
        S.push_back(L1E<T>{lp, (T)0, (T)0});
    } else {
        for (;;) {
            const T ul = ur - e.j;
            if (ul <= hi || j == 0) {  // crossing at the jump of lam_j
                lp = e.l;
                const T jm = hi - ul;
                S.pop_back(t - j);
                S.push_back(L1E<T>{e.l, (T)0, jm < (T)0 ? (T)0 : jm});
                break;
            }
            const L1E<T> q = S.get(j - 1);
            const T sl = s - q.k;
            const T uq = ul - sl * (e.l - q.l);  // h just right of lam_{j-1}
            if (uq <= hi) {  // inside the piece (lam_{j-1}, lam_j)
                lp = clampv(e.l - (ul - hi) * recip(sl), q.l, e.l);
                S.pop_back(t - j);
                S.push_back(L1E<T>{lp, (T)0, (T)0});
                break;
            }
            ur = uq;
            e = q;
            --j;
        }
    }
    lp = lp < lm ? lm : lp;
}

// ---------------------------------------------------------------------------
// The same step on a set held in registers.  Sets of TV-l1 messages are small
// (salt-and-pepper chains, w = 0.3 to 0.8: two breakpoints in 97% of the
// steps, the largest set of a 64-lane wave at most 3 in 87%, at most 5 in
// 99.9%), so the loops over a ring in LDS cost latency and divergence (5 us a
// node) where a fixed number of positions needs neither: every scan below
// visits M + 1 or M + 2 positions, selects by comparisons, and moves entries by
// selects.  Each value is computed by l1_step's operations in l1_step's order,
// so both give the same bits.
// ---------------------------------------------------------------------------
constexpr int kL1Regs = 8;  // largest set held; a step on at most M entries leaves at most M + 3
template <typename T>
struct L1Regs {
    T l[kL1Regs], j[kL1Regs];  // entries past the size: +inf, 0
    int k[kL1Regs];            // slope tags (integers)
    int t;
};

// One step on a set of at most M entries (M + 3 <= kL1Regs).
template <typename T, int M>
__device__ __forceinline__ void l1_step_regs(L1Regs<T> &S, int s, T yi, T di, T ci, T lop, T hip, T lo, T hi, bool root,
                                             T &lm_out, T &lp_out) {
    static_assert(M + 3 <= kL1Regs, "the step's result fits");
    constexpr int N = M + 3;  // positions 1 .. M + 2; the set after the insertion is 1 .. t
    const T inf = (T)__builtin_huge_val();
    T l[N], J[N];
    int k[N];
    if (S.t == 0) {
        lop = (T)0;
        hip = (T)0;
    }
    // (a) the data breakpoint goes after every entry <= d
    const bool ins = ci > (T)0;
    const int t0 = S.t;
    int q = 0;
    bool le[M + 2];
    le[0] = true;
    le[M + 1] = !ins;
#pragma unroll
    for (int i = 1; i <= M; ++i) {
        const bool b = i <= t0 && S.l[i - 1] <= di;
        q = b ? i : q;
        le[i] = b || !ins;
    }
    const bool is_end = ins && q == t0;
    const T cj = (T)2 * ci;
    l[0] = l[N - 1] = inf;
    J[0] = J[N - 1] = (T)0;
    k[0] = k[N - 1] = 0;
#pragma unroll
    for (int i = 1; i <= M + 1; ++i) {
        const T pl = i <= M ? S.l[i <= M ? i - 1 : 0] : inf, pj = i <= M ? S.j[i <= M ? i - 1 : 0] : (T)0;
        const int pk = i <= M ? S.k[i <= M ? i - 1 : 0] : 0;
        const T bl = i >= 2 ? S.l[i >= 2 ? i - 2 : 0] : inf, bj = i >= 2 ? S.j[i >= 2 ? i - 2 : 0] : (T)0;
        const int bk = i >= 2 ? S.k[i >= 2 ? i - 2 : 0] : s - 1;
        const T ml = le[i - 1] ? di : bl, mj = le[i - 1] ? cj : bj;
        const int dk = is_end ? 0 : bk;  // the split piece's tag
        const int mk = le[i - 1] ? dk : bk;
        l[i] = le[i] ? pl : ml;
        J[i] = le[i] ? pj : mj;
        k[i] = le[i] ? pk : mk;
        k[i] = (is_end && i == t0) ? s - 1 : k[i];  // the old back's right piece is now interior
    }
    const int t = t0 + (ins ? 1 : 0);
    const T basel = lop - yi - ci, baser = hip - yi + ci, v = root ? (T)0 : lo;
    // left crossing: E the last entry with h(l+) < v, G the one after it
    T El = (T)0, Ev = (T)0, Gl = inf, Gv = inf;
    int Ek = 0, Gk = 0, p = 0;
    bool jump = false, prev = true;
    const T vl1 = l[1] + basel;
    T vl = vl1;
#pragma unroll
    for (int i = 1; i <= M + 1; ++i) {
        const T vr = vl + J[i];
        const bool br = vr < v, g = prev && !br;
        El = br ? l[i] : El;
        Ev = br ? vr : Ev;
        Ek = br ? k[i] : Ek;
        p = br ? i : p;
        Gl = g ? l[i] : Gl;
        Gv = g ? vr : Gv;
        Gk = g ? k[i] : Gk;
        jump = g ? vl < v : jump;
        prev = br;
        if (i <= M) vl = vr + (T)(s - k[i]) * (l[i + 1] - l[i]);
    }
    const bool p0 = p == 0, pe = p == t;
    const T sl = pe ? (T)1 : (T)(s - Ek);
    const T lin = clampv(El + (v - Ev) * recip(sl), El, Gl);
    T lm = p0 ? l[1] - (vl1 - v) : lin;
    lm = t == 0 ? v - basel : lm;
    lm = jump ? Gl : lm;
    // (b) the new front, in the place of the first f entries: flat at lo left of it
    const int f = p + (jump ? 1 : 0);
    const T jm = Gv - lo, JF = jump ? (jm < (T)0 ? (T)0 : jm) : (T)0;
    const int kj = p + 1 == t ? 0 : Gk, kn = pe ? 0 : (p0 ? s - 1 : Ek), kF = jump ? kj : kn;
    // the front at position 1, the entries after f from position 2 on
    const bool up = f == 0;
    const int sh = up ? 0 : f - 1;
#pragma unroll
    for (int i = N - 1; i >= 2; --i) {
        l[i] = up ? l[i - 1] : l[i];
        J[i] = up ? J[i - 1] : J[i];
        k[i] = up ? k[i - 1] : k[i];
    }
#pragma unroll
    for (int b = 1; b <= M; b *= 2) {
        const bool on = (sh & b) != 0;
#pragma unroll
        for (int i = 2; i < N; ++i) {
            l[i] = on ? (i + b < N ? l[i + b < N ? i + b : 0] : inf) : l[i];
            J[i] = on ? (i + b < N ? J[i + b < N ? i + b : 0] : (T)0) : J[i];
            k[i] = on ? (i + b < N ? k[i + b < N ? i + b : 0] : 0) : k[i];
        }
    }
    l[1] = lm;
    J[1] = JF;
    k[1] = kF;
    const int t1 = t - f + 1;
    // (c) right crossing, from the back: U the last entry with h(l+) <= hi, V the one after it
    T Ul = (T)0, Uu = (T)0, Vl = (T)0, Vu = (T)0;
    int Uk = 0, R = 0;
    bool found = false, Vc = false;
    T ul = (T)0, lnext = (T)0;
#pragma unroll
    for (int i = N - 1; i >= 1; --i) {
        const T top = l[i] + baser, in = ul - (T)(s - k[i]) * (lnext - l[i]);
        const T ur = i == t1 ? top : in;
        ul = ur - J[i];
        lnext = l[i];
        const bool on = i <= t1 && !found, cR = ur <= hi, u = on && cR, w = on && !cR;
        Ul = u ? l[i] : Ul;
        Uu = u ? ur : Uu;
        Uk = u ? k[i] : Uk;
        R = u ? i : R;
        Vl = w ? l[i] : Vl;
        Vu = w ? ul : Vu;
        Vc = w ? (i == 1 || ul <= hi) : Vc;
        found = found || u;
    }
    const bool end = found && R == t1, jr = !end && Vc;
    const T mid = clampv(Vl - (Vu - hi) * recip((T)(s - Uk)), Ul, Vl);
    T lp = end ? Ul + (hi - Uu) : mid;
    lp = jr ? Vl : lp;
    const T jb = hi - Vu, JB = jr ? (jb < (T)0 ? (T)0 : jb) : (T)0;
    const int r = R + 1;  // the new back: flat at hi right of it
#pragma unroll
    for (int i = 1; i <= N; ++i) {
        const int m = i < N ? i : 0;
        const int ki = (end && i == t1) ? s - 1 : k[m];
        const bool in = i < r && i < N, at = i == r;
        S.l[i - 1] = in ? l[m] : (at ? lp : inf);
        S.j[i - 1] = in ? J[m] : (at ? JB : (T)0);
        S.k[i - 1] = in ? ki : 0;
    }
    S.t = r;
    lm_out = lm;
    lp_out = lp < lm ? lm : lp;
}

#pragma clang fp contract(fast)
}  // namespace tvc
