// tree_dp.hip -- Algorithm 2 on a batch of trees with the Sec. 4.2 unaries
//
//     x = argmin_x  sum_i ( a_i x_i^2 / 2 - b_i x_i + c_i |x_i - d_i| ) + sum_{i != root} f_i(x_parent(i) - x_i),
//     f_i(z) = wm_i z (z < 0), wp_i z (z >= 0),
//
// (the chain is the tree with parent(i) = i + 1).  Sixteen lanes per tree, a
// breakpoint each (k_tree_row); trees it leaves, one lane each (k_tree_dp).  The
// derivative of each message is kept as in Sec. 4.2: its left end (al, bl),
// right end (ar, br) and the multiset of breakpoints (lambda, da, db) sorted
// by lambda (right of lambda the linear piece changes by (da, db)).  A node's
// message is its unary plus the sum of its children's clipped messages, i.e.
// the union of their breakpoint sets with the ends added (the "Extension to
// trees" of Sec. 4.2); clipping it to [wm_i, wp_i] pops the breakpoints past
// each crossing and pushes the crossing point, updating a crossed
// breakpoint's increment in place at a jump.  All arithmetic is FP64.
//
// Trees are numbered in depth-first post-order (every subtree is a contiguous
// range ending at its root), so the clipped messages of a node's children are
// the top entries of a stack of pending messages: each tree has an arena in
// the workspace holding that stack (at most 3 breakpoints per node of the
// finished subtrees) and a merge buffer.
#include <hip/hip_runtime.h>

#include "kernels.h"
#include "chain_core.h"

namespace tvc {

struct TreeBatch {
    int64_t num_trees;
    const int64_t *offsets;  // [num_trees + 1] node ranges
    const int64_t *parent;   // [N] global parent index, -1 at each tree's root
};

// A breakpoint: lambda and the changes (da, db) of the linear piece to its
// right.  Each record is one 32-byte block, so a lane's access to it is one
// pair of 16-byte loads from a single cache line.
struct alignas(32) TBp {
    double l, a, b, pad;
};
// A pending message: its run [start, start + count) inside the region that
// starts at reg, the node it is for, and its clip levels (flat ends).
struct alignas(16) THdr {
    int64_t start, count, reg, parent;
    double lo, hi;
};
// lambda^-, lambda^+ of a node's edge (root: x_root twice).
struct alignas(16) TLam {
    double lo, hi;
};

struct TreeWs {
    TBp *ent;   // arena [6 N + 16 T] (entries of tree t from 6 off[t] + 16 t)
    THdr *hdr;  // pending-message stack [N]
    TLam *lam;  // [N]
    int *bad;   // set if a tree is not numbered in post-order
};

__device__ __forceinline__ TBp tb_get(const TreeWs &W, int64_t i) { return W.ent[i]; }
__device__ __forceinline__ void tb_put(const TreeWs &W, int64_t i, const TBp &e) { W.ent[i] = e; }

// Moves cnt breakpoints from src to dst (overlap allowed), eight at a time with
// every load of a group issued before its stores, so a group costs one memory
// latency rather than eight.
constexpr int kMoveGroup = 8;
__device__ __forceinline__ void arena_move_n(const TreeWs &W, int64_t dst, int64_t src, int64_t cnt) {
    if (cnt <= 0 || dst == src) return;
    TBp r[kMoveGroup];
    if (dst > src) {  // from the top down
        for (int64_t hi = cnt; hi > 0; hi -= kMoveGroup) {
            const int64_t lo = hi > kMoveGroup ? hi - kMoveGroup : 0;
#pragma unroll
            for (int g = 0; g < kMoveGroup; ++g)
                if (lo + g < hi) r[g] = tb_get(W, src + lo + g);
#pragma unroll
            for (int g = 0; g < kMoveGroup; ++g)
                if (lo + g < hi) tb_put(W, dst + lo + g, r[g]);
        }
    } else {  // from the bottom up
        for (int64_t lo = 0; lo < cnt; lo += kMoveGroup) {
            const int64_t hi = lo + kMoveGroup < cnt ? lo + kMoveGroup : cnt;
#pragma unroll
            for (int g = 0; g < kMoveGroup; ++g)
                if (lo + g < hi) r[g] = tb_get(W, src + lo + g);
#pragma unroll
            for (int g = 0; g < kMoveGroup; ++g)
                if (lo + g < hi) tb_put(W, dst + lo + g, r[g]);
        }
    }
}

// h(z) <= v <= h(z+) scanning from the left over entries [s, s + t) of the
// arena; returns z, the entries passed, the piece left of z and whether z is
// the jump of entry s + passed.  The next entry is loaded one step ahead.
__device__ double tree_cross_left(const TreeWs &W, int64_t s, int64_t t, double A, double B, double v,
                                  int64_t *passed, double *pa, double *pb, bool *jump) {
    int64_t j = 0;
    double z;
    *jump = false;
    TBp e{0.0, 0.0, 0.0}, nx{0.0, 0.0, 0.0};
    if (t > 0) e = tb_get(W, s);
    double lprev = 0.0;
    for (;;) {
        if (j == t) {
            z = (v - B) / A;
            break;
        }
        if (j + 1 < t) nx = tb_get(W, s + j + 1);
        const double l = e.l;
        const double vl = A * l + B;
        if (vl >= v) {
            z = (v - B) / A;
            z = z > l ? l : z;
            if (j > 0 && z < lprev) z = lprev;
            break;
        }
        const double vr = vl + e.a * l + e.b;
        if (vr >= v) {
            z = l;
            *jump = true;
            break;
        }
        A += e.a;
        B += e.b;
        lprev = l;
        e = nx;
        ++j;
    }
    *passed = j;
    *pa = A;
    *pb = B;
    return z;
}

__device__ double tree_cross_right(const TreeWs &W, int64_t s, int64_t t, double A, double B, double v,
                                   int64_t *passed, double *pa, double *pb, bool *jump) {
    int64_t j = t - 1, k = 0;
    double z;
    *jump = false;
    TBp e{0.0, 0.0, 0.0}, nx{0.0, 0.0, 0.0};
    if (j >= 0) e = tb_get(W, s + j);
    double lnext = 0.0;
    for (;;) {
        if (j < 0) {
            z = (v - B) / A;
            break;
        }
        if (j > 0) nx = tb_get(W, s + j - 1);
        const double l = e.l;
        const double vr = A * l + B;
        if (vr <= v) {
            z = (v - B) / A;
            z = z < l ? l : z;
            if (j + 1 < t && z > lnext) z = lnext;
            break;
        }
        const double vl = vr - (e.a * l + e.b);
        if (vl <= v) {
            z = l;
            *jump = true;
            break;
        }
        A -= e.a;
        B -= e.b;
        lnext = l;
        e = nx;
        --j;
        ++k;
    }
    *passed = k;
    *pa = A;
    *pb = B;
    return z;
}

// tree_cross_left / tree_cross_right on a run of at most kRankMerge entries:
// the run is loaded at once and scanned in registers with the same
// arithmetic, in the same order, so the results are the same bits; the
// crossed entry's increments come back in ja, jb when z is its jump.
template <int N>
__device__ __forceinline__ double tree_cross_left_short(const TreeWs &W, int64_t s, int64_t t, double A, double B,
                                                        double v, int64_t *passed, double *pa, double *pb,
                                                        bool *jump, double *ja, double *jb) {
    TBp E[N];
#pragma unroll
    for (int j = 0; j < N; ++j)
        if (j < t) E[j] = tb_get(W, s + j);
    bool done = false;
    double z = 0.0, lprev = 0.0;
    int64_t k = t;
    *jump = false;
    *ja = 0.0;
    *jb = 0.0;
#pragma unroll
    for (int j = 0; j < N; ++j) {
        if (!done && j < t) {
            const double l = E[j].l;
            const double vl = A * l + B;
            if (vl >= v) {
                z = (v - B) / A;
                z = z > l ? l : z;
                if (j > 0 && z < lprev) z = lprev;
                k = j;
                done = true;
            } else {
                const double vr = vl + E[j].a * l + E[j].b;
                if (vr >= v) {
                    z = l;
                    *jump = true;
                    *ja = E[j].a;
                    *jb = E[j].b;
                    k = j;
                    done = true;
                } else {
                    A += E[j].a;
                    B += E[j].b;
                    lprev = l;
                }
            }
        }
    }
    if (!done) z = (v - B) / A;
    *passed = k;
    *pa = A;
    *pb = B;
    return z;
}

template <int N>
__device__ __forceinline__ double tree_cross_right_short(const TreeWs &W, int64_t s, int64_t t, double A, double B,
                                                         double v, int64_t *passed, double *pa, double *pb,
                                                         bool *jump, double *ja, double *jb) {
    TBp E[N];  // E[m]: entry t - 1 - m of the run
#pragma unroll
    for (int m = 0; m < N; ++m)
        if (m < t) E[m] = tb_get(W, s + t - 1 - m);
    bool done = false;
    double z = 0.0, lnext = 0.0;
    int64_t k = t;
    *jump = false;
    *ja = 0.0;
    *jb = 0.0;
#pragma unroll
    for (int m = 0; m < N; ++m) {
        if (!done && m < t) {
            const double l = E[m].l;
            const double vr = A * l + B;
            if (vr <= v) {
                z = (v - B) / A;
                z = z < l ? l : z;
                if (m > 0 && z > lnext) z = lnext;
                k = m;
                done = true;
            } else {
                const double vl = vr - (E[m].a * l + E[m].b);
                if (vl <= v) {
                    z = l;
                    *jump = true;
                    *ja = E[m].a;
                    *jb = E[m].b;
                    k = m;
                    done = true;
                } else {
                    A -= E[m].a;
                    B -= E[m].b;
                    lnext = l;
                }
            }
        }
    }
    if (!done) z = (v - B) / A;
    *passed = k;
    *pa = A;
    *pb = B;
    return z;
}

// A node's inputs in FP64 and its parent.
struct TIn {
    double a, b, c, d, lo, hi;
    int64_t p;
};

// Runs of at most this many breakpoints are merged by rank: both are loaded
// at once and every entry goes straight to its place (an entry of the first
// run after the second run's entries with a smaller lambda, one of the second
// run after the first run's entries with a lambda at most its own, as the
// sequential merge orders them), so a merge costs one memory latency rather
// than one per entry.  The same bound selects the unary's insertion point
// from parallel loads.
constexpr int kRankMerge = 8;

// Merge runs [cs, cs + ct) and [s, s + t) (1 <= ct, t <= kRankMerge) into
// [dst, dst + ct + t); every load precedes every store, so dst may overlap
// both runs.
__device__ __forceinline__ void tree_rank_merge(const TreeWs &W, int64_t cs, int64_t ct, int64_t s, int64_t t,
                                                int64_t dst) {
    TBp U[kRankMerge], V[kRankMerge];
#pragma unroll
    for (int k = 0; k < kRankMerge; ++k)
        if (k < ct) U[k] = tb_get(W, cs + k);
#pragma unroll
    for (int m = 0; m < kRankMerge; ++m)
        if (m < t) V[m] = tb_get(W, s + m);
    int64_t pu[kRankMerge], pv[kRankMerge];
#pragma unroll
    for (int k = 0; k < kRankMerge; ++k) {
        int64_t pos = k;
#pragma unroll
        for (int m = 0; m < kRankMerge; ++m) pos += (k < ct && m < t && V[m].l < U[k].l) ? 1 : 0;
        pu[k] = pos;
    }
#pragma unroll
    for (int m = 0; m < kRankMerge; ++m) {
        int64_t pos = m;
#pragma unroll
        for (int k = 0; k < kRankMerge; ++k) pos += (k < ct && m < t && U[k].l <= V[m].l) ? 1 : 0;
        pv[m] = pos;
    }
#pragma unroll
    for (int k = 0; k < kRankMerge; ++k)
        if (k < ct) tb_put(W, dst + pu[k], U[k]);
#pragma unroll
    for (int m = 0; m < kRankMerge; ++m)
        if (m < t) tb_put(W, dst + pv[m], V[m]);
}

// The working message of a node is the run [s, s + t) of its region [r, s + t)
// (the front may float inside the region, so front pops and pushes move
// nothing); the region ends at top = s + t, and the regions of pending
// messages are stacked contiguously below it.
// Lanes (trees) per 64-wide wave.  Each lane's work is a chain of dependent
// memory accesses, so waves that are partly empty trade issue slots for more
// waves per SIMD to hide that latency.
constexpr int kTreeLanes = 64;

// ---------------------------------------------------------------------------
// Sixteen lanes (a DPP row) per tree.  Messages are small (random trees of 256
// nodes with l1 terms: at most 8 breakpoints before the clip in 99% of the
// nodes, at most 14 in all but a few in a hundred thousand and in the roots that
// take every pending subtree), so a node's whole message sits one breakpoint
// per lane:
//  - the children's runs and the unary's breakpoint are loaded side by side and
//    sorted once by rank (a lane counts the breakpoints before its own);
//  - a scan gives every lane the linear piece A z + B right of its breakpoint;
//  - every lane forms the crossings on its piece, and masks pick the lanes
//    whose crossing is the new front and the new back.
// Nothing walks, where a lane per tree ran its own serial walk through memory
// and a wave every lane's path: 16,384 trees x 256 nodes took 5.7 ms (22 us a
// node on 256 waves), 65,536 trees 9.0 ms.  Larger messages, up to kTreeWide, are
// cut where they lie (tree_cut, tree_wide) a few times per tree.  A tree with more
// of them, or with one beyond that, goes on in the lane-per-tree kernel from the node
// that it has reached: there a step on a deep sorted message reads the few
// breakpoints that it drops (16,384 paths of 256 nodes with smooth data, w = 30:
// 1.1 ms by lanes, 19 ms with every message cut here).  One with an invalid
// numbering is done again there from the start.
// ---------------------------------------------------------------------------
constexpr int kTreeRow = 16;
constexpr int kTreeMost = kTreeRow - 2;  // a lane past the last breakpoint and one before the first
// A message of this many breakpoints takes about as long in tree_cut (twice,
// a dozen passes of t / 16 loads) as in the lane kernel's merge and scans.
constexpr int kTreeWide = 128;
// How many of them a tree may have: each counts by what it costs a lane less than here.
// With one child's message and no l1 term a lane reads only what it drops: the first one
// ends the row's work.  With one child and an l1 term a lane shifts half of a sorted run:
// ten of them do.  Several children's messages a lane merges, which takes as long as here
// without l1 terms (six) and longer with them (they count the other way).  us, lanes alone /
// every wide message cut here / this rule: 16,384 x 256 smooth paths, w = 3 1170 / 8300 /
// 1210, with l1 terms, w = 30 4110 / 6810 / 4450; caterpillars, w = 30 3050 / 3710 / 3130,
// with l1 terms 5090 / 4190 / 4360; random trees with l1 terms, w = 30 14800 / 4630 / 8670.
// What a row spends before it hands over stays: paths of 60 smooth nodes, w = 30, 247 us by
// lanes, 360 by this rule.
constexpr int kTreeWideMost = 60, kTreeWidePath = 61, kTreeWidePathL1 = 6, kTreeWideMerge = 10,
              kTreeWideMergeL1 = 20;
// The lane kernel's orders, in the lambda pair of a tree's last node: the node to go on
// from and the pending messages there, or kTreeDone.
constexpr int64_t kTreeDone = -1;
__device__ __forceinline__ void tree_order(const TreeWs &W, int64_t last, int64_t node, int64_t pending) {
    W.lam[last] = TLam{__longlong_as_double(node), __longlong_as_double(pending)};
}

// Each lane of a row another lane's value (DPP control; lanes without a source read 0).
template <int CTRL> __device__ __forceinline__ double row_mov(double v) {
    const long long b = __double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)b, CTRL, 0xf, 0xf, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ double row_next(double v) { return row_mov<0x12F>(v); }  // row_ror:15
__device__ __forceinline__ double row_prev(double v) { return row_mov<0x121>(v); }  // row_ror:1
__device__ __forceinline__ unsigned row_bits(bool p, int lane) {
    return (unsigned)(__ballot(p) >> (lane & 48)) & 0xffffu;
}
// Inclusive prefix sum, and the sum over the row.
__device__ __forceinline__ double row_scan(double v) {
    v += row_mov<0x111>(v);  // row_shr:1, 2, 4, 8
    v += row_mov<0x112>(v);
    v += row_mov<0x114>(v);
    v += row_mov<0x118>(v);
    return v;
}
__device__ __forceinline__ double row_sum(double v) { return row_mov<0x15F>(row_scan(v)); }  // row_newbcast:15
// Breakpoints before this lane's (ties in lane order): a permutation of the row.
template <int D> __device__ __forceinline__ int row_before(double l, int j) {
    const double o = row_mov<0x120 + D>(l);  // row_ror:D
    return (j >= D ? o <= l : o < l) ? 1 : 0;
}
__device__ __forceinline__ int row_rank(double l, int j) {
    return row_before<1>(l, j) + row_before<2>(l, j) + row_before<3>(l, j) + row_before<4>(l, j) +
           row_before<5>(l, j) + row_before<6>(l, j) + row_before<7>(l, j) + row_before<8>(l, j) +
           row_before<9>(l, j) + row_before<10>(l, j) + row_before<11>(l, j) + row_before<12>(l, j) +
           row_before<13>(l, j) + row_before<14>(l, j) + row_before<15>(l, j);
}
// This lane's value to lane `to` of its row.
__device__ __forceinline__ double row_send(double v, int lane, int to) {
    const int addr = ((lane & 48) + to) * 4;
    const long long b = __double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_ds_permute(addr, (int)(unsigned)b);
    const unsigned hi = (unsigned)__builtin_amdgcn_ds_permute(addr, (int)(b >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Where A z + B plus the increments of the t breakpoints at s (in any order) and
// of a jump at d crosses zero: z, the piece left of it (A, B) and right of it
// (A2, B2, another one at a jump), and the bounds between which the
// breakpoints right (l > left) and left (l < right) of it lie.  The bracket of
// the zero shrinks from pivot to pivot; the sums of the breakpoints left of it
// are kept.
struct TCut {
    double z, A, B, A2, B2, left, right;
};
__device__ TCut tree_cut(const TreeWs &W, int64_t s, int t, double A, double B, double d, double jump, int lane) {
    const double inf = __builtin_huge_val();
    const int j = lane & 15, n = t + (jump > 0.0 ? 1 : 0);
    auto get = [&](int k) { return k < t ? tb_get(W, s + k) : TBp{d, 0.0, jump, 0.0}; };
    double lo = -inf, hi = inf;
    for (int it = 0; it <= n; ++it) {  // every pivot leaves the bracket
        // a pivot: a breakpoint inside it, of the middle one of the lanes that hold one
        double q = inf;
        for (int k = j; k < n; k += kTreeRow) {
            const double l = get(k).l;
            q = l > lo && l < hi ? l : q;
        }
        unsigned m = row_bits(q < inf, lane);
        if (!m) break;
        for (int half = __popc(m) / 2; half > 0; --half) m &= m - 1;
        q = __shfl(q, (lane & 48) + __ffs(m) - 1, 64);
        double a1 = 0.0, b1 = 0.0, a2 = 0.0, b2 = 0.0;
        for (int k = j; k < n; k += kTreeRow) {
            const TBp e = get(k);
            const bool in = e.l > lo && e.l < q, at = e.l == q;
            a1 += in ? e.a : 0.0;
            b1 += in ? e.b : 0.0;
            a2 += at ? e.a : 0.0;
            b2 += at ? e.b : 0.0;
        }
        a1 = A + row_sum(a1);
        b1 = B + row_sum(b1);
        a2 = a1 + row_sum(a2);
        b2 = b1 + row_sum(b2);
        if (a1 * q + b1 >= 0.0) {
            hi = q;
        } else if (a2 * q + b2 >= 0.0) {
            return TCut{q, a1, b1, a2, b2, q, q};
        } else {
            lo = q;
            A = a2;
            B = b2;
        }
    }
    double z = -B / A;
    z = z > hi ? hi : z;
    z = z < lo ? lo : z;
    return TCut{z, A, B, A, B, lo, hi};
}

// The clip of a message too large for a row: cut at both levels, the
// breakpoints between them moved together in place (the next sort orders
// them).  Returns the new count.
__device__ int tree_wide(const TreeWs &W, int64_t s, int t, double A, double B, double d, double jump, double lo,
                         double hi, int lane, TLam *z) {
    const int j = lane & 15, n = t + (jump > 0.0 ? 1 : 0);
    const TCut p = tree_cut(W, s, t, A, B - lo, d, jump, lane);
    TCut r = tree_cut(W, s, t, A, B - hi, d, jump, lane);
    r.z = r.z < p.z ? p.z : r.z;
    *z = TLam{p.z, r.z};
    int m = 0;
    for (int k0 = 0; k0 < n; k0 += kTreeRow) {
        const int k = k0 + j;
        const TBp e = k < t ? tb_get(W, s + k) : TBp{d, 0.0, jump, 0.0};
        const bool keep = k < n && e.l > p.left && e.l < r.right;
        const unsigned kept = row_bits(keep, lane);
        if (keep) tb_put(W, s + m + __popc(kept & ((1u << j) - 1)), e);
        m += __popc(kept);
        __threadfence_block();
    }
    const bool one = p.left == r.right && p.left == p.z;  // both levels in one jump
    if (j == 0) {
        if (one) {
            tb_put(W, s + m, TBp{p.z, 0.0, hi - lo, 0.0});
        } else {
            tb_put(W, s + m, TBp{p.z, p.A2, p.B2, 0.0});
            tb_put(W, s + m + 1, TBp{r.z, -r.A, -r.B, 0.0});
        }
    }
    return m + (one ? 1 : 2);
}

// The pending stack as it was before messages of t breakpoints in all were taken from it.
__device__ __forceinline__ void tree_untake(const TreeWs &W, int64_t n0, int64_t t, int64_t *top, int64_t *sp) {
    for (const int64_t end = *top + t; *top < end; ++*sp) *top += W.hdr[n0 + *sp].count;
}

// Sorts the t breakpoints at s by rank (ties in memory order), by way of the free
// entries at tmp.
__device__ void tree_sort(const TreeWs &W, int64_t s, int t, int64_t tmp, int lane) {
    const int j = lane & 15;
    for (int k = j; k < t; k += kTreeRow) {
        const TBp e = tb_get(W, s + k);
        int r = 0;
#pragma unroll 8
        for (int m = 0; m < t; ++m) {
            const double l = W.ent[s + m].l;
            r += (l < e.l || (l == e.l && m < k)) ? 1 : 0;
        }
        tb_put(W, tmp + r, e);
    }
    __threadfence_block();
    for (int k = j; k < t; k += kTreeRow) tb_put(W, s + k, tb_get(W, tmp + k));
    __threadfence_block();
}

template <typename T>
__global__ __launch_bounds__(64, 4) void k_tree_row(TreeBatch tb, TreeWs W, const T *__restrict__ a,
                                                 const T *__restrict__ b, const T *__restrict__ c,
                                                 const T *__restrict__ d, const T *__restrict__ wm,
                                                 const T *__restrict__ wp, T *__restrict__ x) {
    const double inf = __builtin_huge_val();
    const int lane = threadIdx.x, j = lane & 15;
    const bool pre = j == 15;  // stands before the first breakpoint
    const int64_t tr = (int64_t)blockIdx.x * 4 + (lane >> 4);
    if (tr >= tb.num_trees) return;  // whole rows
    const int64_t n0 = tb.offsets[tr], n1 = tb.offsets[tr + 1];
    if (n1 <= n0) return;
    int64_t top = 6 * n0 + 16 * tr, sp = 0;  // end of the pending runs in this tree's arena; pending messages
    const int64_t aend = top + 6 * (n1 - n0) + 16;
    THdr h0{0, 0, 0, -1, 0.0, 0.0}, h1 = h0;  // the last two of them
    int64_t t64 = 0;  // breakpoints of a node's children
    int wide = 0;  // what the messages cut where they lie have cost so far
    auto load_in = [&](int64_t i) {
        TIn q;
        q.a = a ? (double)a[i] : 1.0;
        q.b = (double)b[i];
        q.c = c ? (double)c[i] : 0.0;
        q.d = d ? (double)d[i] : 0.0;
        q.lo = (double)wm[i];
        q.hi = (double)wp[i];
        q.p = tb.parent[i];
        return q;
    };
    TIn nx = load_in(n0);
    int64_t i = n0;  // stops at the node to go on from in the lane kernel
    for (; i < n1; ++i) {
        const TIn in = nx;
        if (i + 1 < n1) nx = load_in(i + 1);
        // (a) the children's runs, side by side: the top headers whose node is i
        // (their regions are contiguous and end at the old top)
        double bl = -in.b - in.c;
        int64_t src = -1;
        t64 = 0;
        while (sp > 0 && h0.parent == i) {
            const int64_t hc = top - h0.start;  // its count
            if (j >= t64 && j < t64 + hc) src = h0.start + (j - t64);
            t64 += hc;
            bl += h0.lo;
            top = h0.start;
            --sp;
            h0 = h1;
            if (sp > 1) h1 = W.hdr[n0 + sp - 2];
        }
        const bool data = in.c > 0.0, root = in.p < 0;
        const double lo = root ? 0.0 : in.lo, hi = in.hi;
        if ((!root && (in.p <= i || in.p >= n1)) || t64 > (root ? (int64_t)1 << 30 : kTreeWide)) break;
        int t = (int)t64, count;
        const bool big = t + (data ? 1 : 0) > kTreeMost;
        if (big) {
            const double jump = data ? 2.0 * in.c : 0.0;
            TLam z;
            if (root) {  // the zero of h
                z.lo = z.hi = tree_cut(W, top, t, in.a, bl, in.d, jump, lane).z;
                count = 0;
            } else {
                const bool one_run = W.hdr[n0 + sp].count == t64;
                wide += one_run ? (data ? kTreeWidePathL1 : kTreeWidePath) : (data ? -kTreeWideMergeL1 : kTreeWideMerge);
                wide = wide > 0 ? wide : 0;
                if (wide > kTreeWideMost || top + t + 3 > aend) break;
                count = tree_wide(W, top, t, in.a, bl, in.d, jump, lo, hi, lane, &z);
            }
            if (j == 0) W.lam[i] = z;
        } else {
            TBp e{inf, 0.0, 0.0, 0.0};
            if (src >= 0) e = tb_get(W, src);
            // (b) the unary's breakpoint after them
            if (data && j == t) e = TBp{in.d, 0.0, 2.0 * in.c, 0.0};
            if (data) ++t;
            if (t > 1) {
                const int r = row_rank(e.l, j);
                const double sl = row_send(e.l, lane, r), sa = row_send(e.a, lane, r), sb = row_send(e.b, lane, r);
                e.l = sl;
                e.a = sa;
                e.b = sb;
            }
            // the piece right of each breakpoint; the lane before the first has the left end's
            double A = row_scan(e.a) + in.a, B = row_scan(e.b) + bl;
            A = pre ? in.a : A;
            B = pre ? bl : B;
            const bool entry = j < t;
            const double ln = row_next(e.l), vr = A * e.l + B, ve = A * ln + B;
            // (c) clip to [wm_i, wp_i] (root: the zero of h)
            const int p = __ffs(~row_bits(entry && vr < lo, lane)) - 1;  // breakpoints left of lambda^-
            const bool jl = (row_bits(ve < lo, lane) >> ((p + 15) & 15)) & 1;  // at breakpoint p's jump
            const int F = jl ? p : (p + 15) & 15;
            double zl = (lo - B) / A;
            zl = zl > ln ? ln : zl;
            zl = (!pre && zl < e.l) ? e.l : zl;
            const double lm = jl ? e.l : zl;  // at lane F
            const int r0 = __ffs(~row_bits(entry && vr <= hi, lane)) - 1, r = r0 < p ? p : r0;  // left of lambda^+
            const bool one = jl && r == p;                                                       // both in one jump
            const bool jr = (row_bits(ve <= hi, lane) >> ((r + 15) & 15)) & 1;
            const double lf = j == F ? lm : e.l;  // the positions with the new front
            const double Ap = row_prev(A), Bp = row_prev(B), lp0 = row_prev(lf);
            double zr = (hi - Bp) / Ap;
            zr = zr > e.l ? e.l : zr;
            zr = zr < lp0 ? lp0 : zr;
            const double lp = jr ? e.l : zr;  // at lane r
            if (j == F) {
                e.l = lm;
                e.a = one ? 0.0 : A;
                e.b = one ? hi - lo : B - lo;
            } else if (j == r) {
                e.l = lp;
                e.a = -Ap;
                e.b = hi - Bp;
            }
            count = root ? 0 : (one ? 1 : ((r - F) & 15) + 1);
            if (top + count > aend) break;
            const int m = (j - F) & 15;
            if (m < count) tb_put(W, top + m, e);
            if (j == F) W.lam[i].lo = lm;
            if (j == (one || root ? F : r)) W.lam[i].hi = e.l;
        }
        // push the clipped message for the parent
        if (!root) {
            h1 = h0;
            h0 = THdr{top, count, big ? -1 : top, in.p, lo, hi};  // (region -1: not sorted)
            if (j == 0) W.hdr[n0 + sp] = h0;
            ++sp;
            top += count;
        }
        __threadfence_block();
    }
    if (i < n1 || sp != 0) {
        if (i < n1) tree_untake(W, n0, t64, &top, &sp);
        // the pending messages as the lane kernel keeps them: sorted, each its own region;
        // where that cannot be (no room to sort, an invalid numbering) it starts again
        bool again = i == n1;
        for (int64_t q = 0; q < sp && !again; ++q) {
            const THdr hd = W.hdr[n0 + q];
            if (hd.reg >= 0) continue;
            again = top + hd.count > aend;
            if (again) break;
            tree_sort(W, hd.start, (int)hd.count, top, lane);
            if (j == 0) W.hdr[n0 + q].reg = hd.start;
        }
        if (j == 0) tree_order(W, n1 - 1, again ? n0 : i, again ? 0 : sp);
        return;
    }
    // backward pass, sixteen nodes at a time from the last: parents have higher
    // numbers, so a node waits for lanes below its own or for earlier rounds
    for (int64_t hi = n1 - 1; hi >= n0; hi -= kTreeRow) {
        const int64_t i = hi - j;
        const bool in = i >= n0;
        const int64_t p = in ? tb.parent[i] : -1;
        const TLam z = in ? W.lam[i] : TLam{0.0, 0.0};
        bool ready = !in || p < 0 || p > hi;
        double v = z.lo;
        if (in && p > hi) {
            v = (double)x[p];
            v = v < z.lo ? z.lo : (v > z.hi ? z.hi : v);
        }
        v = (double)(T)v;
        const int from = (lane & 48) + (ready ? j : (int)(hi - p));
        while (row_bits(!ready, lane)) {
            const double u = __shfl(v, from, 64);
            const bool go = __shfl((int)ready, from, 64) != 0;
            if (!ready && go) {
                v = (double)(T)(u < z.lo ? z.lo : (u > z.hi ? z.hi : u));
                ready = true;
            }
        }
        if (in) x[i] = (T)v;
        __threadfence_block();
    }
    if (j == 0) tree_order(W, n1 - 1, kTreeDone, 0);
}

// A lane per tree, for the trees that k_tree_row left, from the node it left them at.
template <typename T>
__global__ __launch_bounds__(64) void k_tree_dp(TreeBatch tb, TreeWs W, const T *__restrict__ a,
                                                const T *__restrict__ b, const T *__restrict__ c,
                                                const T *__restrict__ d, const T *__restrict__ wm,
                                                const T *__restrict__ wp, T *__restrict__ x, int lanes) {
    if ((int)threadIdx.x >= lanes) return;
    const int64_t tr = (int64_t)blockIdx.x * lanes + threadIdx.x;
    if (tr >= tb.num_trees) return;
    const int64_t n0 = tb.offsets[tr], n1 = tb.offsets[tr + 1];
    if (n1 <= n0) return;
    const TLam order = W.lam[n1 - 1];
    const int64_t from = __double_as_longlong(order.lo);
    if (from == kTreeDone) return;
    const int64_t abase = 6 * n0 + 16 * tr;     // this tree's arena
    const int64_t aend = abase + 6 * (n1 - n0) + 16;
    int64_t top = abase;                          // end of the pending stack's regions
    int64_t sp = n0 + __double_as_longlong(order.hi);  // header stack pointer
    if (sp > n0) top = W.hdr[sp - 1].start + W.hdr[sp - 1].count;
    bool ok = true;
    // a node's inputs are loaded while the node before it is processed
    auto load_in = [&](int64_t i) {
        TIn q;
        q.a = a ? (double)a[i] : 1.0;
        q.b = (double)b[i];
        q.c = c ? (double)c[i] : 0.0;
        q.d = d ? (double)d[i] : 0.0;
        q.lo = (double)wm[i];
        q.hi = (double)wp[i];
        q.p = tb.parent[i];
        return q;
    };
    TIn nx = load_in(from);
    for (int64_t i = n0; i < n1 && ok; ++i) {
        if (i < from) continue;  // (the lanes' nodes stay abreast)
        const TIn in = nx;
        if (i + 1 < n1) nx = load_in(i + 1);
        // (a) the children's messages: the top headers whose node is i, their
        // regions stacked right below the working one; the first is adopted in
        // place, each further one merged with it via the buffer at top
        double al = 0.0, bl = 0.0, ar = 0.0, br = 0.0;
        int64_t r = top, s = top, t = 0;
        while (sp > n0) {
            const THdr hd = W.hdr[sp - 1];
            if (hd.parent != i) break;
            --sp;
            const int64_t cs = hd.start, ct = hd.count, cr = hd.reg;
            if (cr < abase || cs < cr || cs + ct != r || top + ct + t > aend) {
                ok = false;
                break;
            }
            bl += hd.lo;
            br += hd.hi;
            if (t == 0) {
                r = cr;
                s = cs;
                t = ct;
                continue;
            }
            if (ct <= kRankMerge && t <= kRankMerge) {
                tree_rank_merge(W, cs, ct, s, t, cr);
                r = cr;
                s = cr;
                t += ct;
                top = s + t;
                continue;
            }
            // merge run [cs, cs + ct) with run [s, s + t) into [top, top + ct + t)
            int64_t u = cs, v = s, w = top;
            const int64_t ue = cs + ct, ve = s + t;
            TBp eu{0.0, 0.0, 0.0}, ev{0.0, 0.0, 0.0};
            if (u < ue) eu = tb_get(W, u);
            if (v < ve) ev = tb_get(W, v);
            while (u < ue && v < ve) {
                if (eu.l <= ev.l) {
                    tb_put(W, w++, eu);
                    if (++u < ue) eu = tb_get(W, u);
                } else {
                    tb_put(W, w++, ev);
                    if (++v < ve) ev = tb_get(W, v);
                }
            }
            arena_move_n(W, w, u, ue - u);
            w += ue - u;
            arena_move_n(W, w, v, ve - v);
            arena_move_n(W, cr, top, ct + t);  // back to the bottom of the merged regions
            r = cr;
            s = cr;
            t += ct;
            top = s + t;
        }
        if (!ok) break;
        top = s + t;
        // (b) add the unary
        const double ai = in.a, bi = in.b, ci = in.c, di = in.d;
        al += ai;
        bl += -bi - ci;
        ar += ai;
        br += -bi + ci;
        if (ci > 0.0) {
            // insertion point: after every breakpoint <= d_i; the shorter side moves
            int64_t q = t;
            if (t <= kRankMerge) {
                double l[kRankMerge];
#pragma unroll
                for (int j = 0; j < kRankMerge; ++j) l[j] = j < t ? W.ent[s + j].l : 0.0;
                q = 0;
#pragma unroll
                for (int j = 0; j < kRankMerge; ++j) q += (j < t && l[j] <= di) ? 1 : 0;
            } else {
                while (q > 0 && W.ent[s + q - 1].l > di) --q;
            }
            if (s > r && q < t - q) {
                arena_move_n(W, s - 1, s, q);
                --s;
            } else {
                if (top + 1 > aend) {
                    ok = false;
                    break;
                }
                arena_move_n(W, s + q + 1, s + q, t - q);
            }
            tb_put(W, s + q, TBp{di, 0.0, 2.0 * ci, 0.0});
            ++t;
            top = s + t;
        }
        const int64_t p = in.p;
        int64_t k;
        double pa, pb;
        bool jump;
        if (p < 0) {  // root: the zero of h
            const double xr = tree_cross_left(W, s, t, al, bl, 0.0, &k, &pa, &pb, &jump);
            W.lam[i] = TLam{xr, xr};
            top = r;  // nothing stays pending for this root
            continue;
        }
        if (p <= i || p >= n1) {
            ok = false;
            break;
        }
        // (c) clip to [wm_i, wp_i]
        const double lo = in.lo, hi = in.hi;
        if (top + 2 > aend) {
            ok = false;
            break;
        }
        double ja, jb;
        double lm;
        if (t <= kRankMerge) {
            lm = tree_cross_left_short<kRankMerge>(W, s, t, al, bl, lo, &k, &pa, &pb, &jump, &ja, &jb);
        } else {
            lm = tree_cross_left(W, s, t, al, bl, lo, &k, &pa, &pb, &jump);
            if (jump) {
                const TBp e = tb_get(W, s + k);
                ja = e.a;
                jb = e.b;
            }
        }
        double nda = pa, ndb = pb - lo;
        if (jump) {
            nda += ja;
            ndb += jb;
        }
        const int64_t drop = k + (jump ? 1 : 0);
        if (drop == 0) {  // a new front: room in the region, else shift right by one
            if (s > r) {
                --s;
            } else {
                arena_move_n(W, s + 1, s, t);
            }
            ++t;
        } else {  // the new front takes the last dropped slot
            s += drop - 1;
            t -= drop - 1;
        }
        tb_put(W, s, TBp{lm, nda, ndb});
        double lp;
        if (t <= kRankMerge) {
            lp = tree_cross_right_short<kRankMerge>(W, s, t, ar, br, hi, &k, &pa, &pb, &jump, &ja, &jb);
        } else {
            lp = tree_cross_right(W, s, t, ar, br, hi, &k, &pa, &pb, &jump);
            if (jump) {
                const TBp e = tb_get(W, s + t - 1 - k);
                ja = e.a;
                jb = e.b;
            }
        }
        nda = -pa;
        ndb = hi - pb;
        if (jump) {
            nda += ja;
            ndb += jb;
        }
        t -= k + (jump ? 1 : 0);
        tb_put(W, s + t, TBp{lp, nda, ndb});
        ++t;
        top = s + t;
        W.lam[i] = TLam{lm, lp < lm ? lm : lp};
        // push the clipped message for the parent
        W.hdr[sp] = THdr{s, t, r, p, lo, hi};
        ++sp;
    }
    if (!ok || sp != n0) {  // not a post-order numbering (or a tree left children pending)
        *W.bad = 1;
        return;
    }
    // backward pass: parents (higher indices) before children
    for (int64_t i = n1 - 1; i >= n0; --i) {
        const int64_t p = tb.parent[i];
        double v;
        const TLam L = W.lam[i];
        if (p < 0) {
            v = L.lo;
        } else {
            v = (double)x[p];
            v = v < L.lo ? L.lo : (v > L.hi ? L.hi : v);
        }
        x[i] = (T)v;
    }
}

// Workspace: arena of 6 N + 16 T breakpoint records, the header stack and the
// lambda pairs (one record per node each), flag.
static size_t tree_layout(void *p, int64_t T, int64_t N, TreeWs *out) {
    auto al = [](size_t v) { return (v + 255) & ~(size_t)255; };
    const size_t A = (size_t)(6 * N + 16 * T);
    size_t off = 0;
    const size_t o_e = off;  off += al(sizeof(TBp) * A);
    const size_t o_h = off;  off += al(sizeof(THdr) * (size_t)N);
    const size_t o_l = off;  off += al(sizeof(TLam) * (size_t)N);
    const size_t o_bd = off; off += al(sizeof(int));
    if (p && out) {
        char *c = (char *)p;
        out->ent = (TBp *)(c + o_e);
        out->hdr = (THdr *)(c + o_h);
        out->lam = (TLam *)(c + o_l);
        out->bad = (int *)(c + o_bd);
    }
    return off;
}

size_t tree_dp_ws_bytes(int64_t num_trees, int64_t num_nodes) {
    return tree_layout(nullptr, num_trees, num_nodes, nullptr);
}

template <typename T>
hipError_t launch_tree_dp_lanes(int64_t num_trees, int64_t num_nodes, const int64_t *offsets, const int64_t *parent,
                                const T *a, const T *b, const T *c, const T *d, const T *wm, const T *wp, T *x,
                                void *workspace, int *bad_host, hipStream_t stream, int lanes) {
    TreeWs W;
    tree_layout(workspace, num_trees, num_nodes, &W);
    hipError_t e = hipMemsetAsync(W.bad, 0, sizeof(int), stream);
    if (e != hipSuccess) return e;
    const TreeBatch tb{num_trees, offsets, parent};
    hipLaunchKernelGGL((k_tree_row<T>), dim3((unsigned)((num_trees + 3) / 4)), dim3(64), 0, stream, tb, W, a, b, c, d, wm,
                       wp, x);
    hipLaunchKernelGGL((k_tree_dp<T>), dim3((unsigned)((num_trees + lanes - 1) / lanes)), dim3(64), 0, stream, tb, W,
                       a, b, c, d, wm, wp, x, lanes);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    e = hipMemcpyAsync(bad_host, W.bad, sizeof(int), hipMemcpyDeviceToHost, stream);
    if (e != hipSuccess) return e;
    return hipStreamSynchronize(stream);
}

template <typename T>
hipError_t launch_tree_dp(int64_t num_trees, int64_t num_nodes, const int64_t *offsets, const int64_t *parent,
                          const T *a, const T *b, const T *c, const T *d, const T *wm, const T *wp, T *x,
                          void *workspace, int *bad_host, hipStream_t stream) {
    return launch_tree_dp_lanes<T>(num_trees, num_nodes, offsets, parent, a, b, c, d, wm, wp, x, workspace, bad_host,
                                   stream, kTreeLanes);
}

template hipError_t launch_tree_dp<float>(int64_t, int64_t, const int64_t *, const int64_t *, const float *,
                                          const float *, const float *, const float *, const float *, const float *,
                                          float *, void *, int *, hipStream_t);
template hipError_t launch_tree_dp<double>(int64_t, int64_t, const int64_t *, const int64_t *, const double *,
                                           const double *, const double *, const double *, const double *,
                                           const double *, double *, void *, int *, hipStream_t);

}  // namespace tvc
