// kernels.h -- internal interface between the C-ABI layer and the kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

// A source that instantiates many kernel templates is compiled several times
// by the build, once per part (TVC_PART = 1 .. n), each part instantiating
// one subset; TVC_PART = 0 (the default, a single compilation) instantiates
// everything.
#ifndef TVC_PART
#define TVC_PART 0
#endif
#define TVC_IN_PART(k) (TVC_PART == 0 || TVC_PART == (k))

namespace tvc {

// Breakpoint slots of the per-lane LDS ring.  The deepest deque seen on the
// piecewise-constant / shapes workloads is ~15 breakpoints; chains that go
// deeper are solved with their deque in HBM.
#ifndef TVC_RING_SLOTS
#define TVC_RING_SLOTS 16
#endif
constexpr int kRingSlots = TVC_RING_SLOTS;
// Nodes per register tile: loads run this many nodes ahead of their use.
constexpr int kTile = 8;

struct ChainBatch {
    int64_t num_chains;
    int64_t n;               // uniform length (maximum length with offsets)
    int64_t es, cs;          // element / chain strides (uniform batches)
    const int64_t *offsets;  // CSR starts (device) or nullptr
};

constexpr int64_t kGrpMaxLen = 6144;  // the lambda pairs of an FP64 chain fit LDS (137 KB with the rest)
constexpr int64_t kGrpMaxNodes = int64_t(9) << 18;

// Segmentation of a launch: segment length L (S = ceil(n / L) segments per
// chain), halo H run before each segment, checkpoint spacing CK, and the
// number K of breakpoint slots of the LDS ring (16, 32; 64 or 128 for 8-byte entries).
// wg: the workgroup-per-chain kernel instead, with a geometry of its own.
struct SegPlan {
    int64_t L;
    int64_t H;
    int64_t CK;
    int K;
    int wg = 0;
};

// Segment length, halo and block size of a launch; lds_lam: the lambda pairs of
// a chain stay in LDS (else they go to the workspace's stream); lds: bytes of
// dynamic LDS (the deep chains' deques take all of it).
struct GrpGeom {
    int L, H, threads, lds_lam, lds;
};
// LDS of a block without the lambda pairs.
constexpr size_t grp_lds_bytes(size_t threads, size_t elem, size_t tag) {
    return (2 * elem + 2 * tag + 2) * threads + 256;
}

// Geometry of a workgroup-per-chain launch: 32-node segments with a 64-node
// halo, in at most 64 groups; twice as long (the halo costs less, the chain's
// latency more) while there are more than four waves per SIMD.  us per prox /
// per 2D iteration, FP32, w = 0.3: 512 x 512 at L = 32 66 / 119, 64 77 / 153,
// 128 100 / 222; 1024 x 1024 143 / 279, 103 / 261, 116 / 343.  Halos of 48 to
// 96 are within 5% of it, 32 leaves more segments to run again.  16-node segments
// up to 256 nodes, where a chain's groups are a wave for each SIMD of a CU, while
// the launch has under two waves a SIMD (us, L = 32 / 16 at w = 0.1 and 0.5: 250 x 250 29.5 /
// 25.5 and 75 / 76, 317 x 203 33.7 / 28.5 and 66 / 60, 400 x 200 33.8 / 28.9 and 70 / 65;
// FP64 500 x 200 55 / 47 and 95 / 104); with five or six waves a chain only under one a
// SIMD (203 x 317 29.6 / 28.0 and 77 / 79, 2D 203 x 317 69 / 62 at lambda = 0.05; FP64
// 260 x 300 55 / 56 and 97 / 104, 2D 330 x 330 115 / 146); not on longer ones, whose later
// passes add up (64 x 1000 56 / 75), and up to 128 nodes, where 32-node segments fit one
// wave, only on half of the SIMDs (2D 128 x 128 60 / 52; 512 x 128 42 / 44).
inline GrpGeom grp_geom(int64_t C, int64_t n) {
    int L = 32;
    auto threads = [&](int l) { return (int)((n + l - 1) / l * 16 + 63) / 64 * 64; };
    if (n <= 384 && C * (threads(16) / 64) <= (n <= 128 ? 512 : (n <= 256 ? 1792 : 1024))) L = 16;
    while (L < 128 && C * (threads(L) / 64) > 4096) L *= 2;
    if (threads(L) > 1024) L = (int)((n + 63) / 64 + 15) / 16 * 16;
    return GrpGeom{L, 64, threads(L), 0, 0};
}

// Whether the workgroup-per-chain kernel can solve a launch of this size (its
// lambda pairs in LDS; more than 1024 chains keep a whole deque there, 2n + 4 FP64
// entries up to n = 4096) and may win: what an autotuner tries.
inline bool grp_plan_ok(int64_t num_chains, int64_t n, bool iter2d) {
    const int64_t most = (n < 256 ? kGrpMaxNodes / 4 : kGrpMaxNodes) * (iter2d ? 2 : 1);
    return num_chains > 0 && n <= (num_chains > 1024 ? 4096 : kGrpMaxLen) && num_chains * n <= most;
}

// Whether a launch takes it by default.  With its deque spread over 16 lanes a node
// step has a fifth of the latency, but a wave advances 4 chains or segments instead
// of 64: it wins while its waves fit the chip at once, about four a SIMD, and the
// lane-per-segment kernels leave SIMDs idle.  Counted in waves (C chains of as many as
// grp_geom gives n nodes) the line is the same for every length; lanes' time over the
// groups', prox at w = 0.05 / 0.3:
//  FP32  4096 waves: n = 32 1.26 / 1.34, 64 1.17 / 1.30, 192 1.54 / 1.45, 1024 1.39 /
//        1.67, 4096 1.44 / 1.37; 5000: 192 0.95 / 0.87, 512 1.03 / 1.04, 4096 1.15 / 1.20;
//        6144: 128 0.83 / 0.96, 1024 0.87 / 1.04, 5120 0.83 / 0.84.  Below 24 nodes a lane
//        has as few steps: n = 8 2048 waves 1.13 / 1.15, 3072 0.93 / 0.94.
//  FP64  a group's step takes twice as long: n = 8 512 waves 1.44 / 1.36, 1024 0.95 / 0.96;
//        16 2048 1.07, 3072 0.86; 64 3072 1.15 / 1.24, 4096 0.94 / 1.00; 256 4096 1.88 /
//        1.63.  A second turn of blocks (the lambda pairs of longer chains fill LDS) costs
//        as much as the lanes: 204 x 5120 1.37 / 1.14, 307 x 5120 0.66 / 0.66, 768 x 2048
//        1.31 / 1.30, 1024 x 2048 1.02 / 0.87; so do 128-node segments of chains that the
//        lanes walk in fewer steps: 3072 x 320 0.86 / 0.91.
//  2D    (us an iteration, lambda = 0.04 / 0.1 / 0.2, groups and lanes): more segments
//        start from a state that is not the true one, and each costs the lanes a repair.
//        FP32 1700 x 1700 (6800 waves) 312 / 404 / 961 and 323 / 429 / 1664, 2048 x 2048
//        (8192) 370 / 490 / 1218 and 328 / 433 / 2060, 2200 x 2100 (11,000) 544 / 622 /
//        1552 and 339 / 442 / 2271; batches of 8000 waves of 200-node chains 333 and 268.
//        FP64 1250 x 1250 (3750) 433 / 532 / 1071 and 435 / 528 / 1601, 1500 x 1500 535 /
//        667 / 1539 and 435 / 548 / 2015, 1024 x 2048 483 / 602 / 1262 and 429 / 537 / 1767.
// nodes: of all chains (fewer than num_chains * n where their lengths differ).
inline bool grp_wins(int64_t num_chains, int64_t n, size_t elem, bool iter2d, int64_t nodes) {
    const GrpGeom gm = grp_geom(num_chains, n);
    const int64_t per = gm.threads / 64;
    const double mean = (double)nodes / (double)(num_chains * n) * (double)per;  // waves of a chain of mean length
    const double waves = (double)num_chains * (mean > 1.0 ? mean : 1.0);
    if (elem == 4) {
        if (iter2d) return waves <= (n < 64 ? 4096 : (n < 256 ? 4608 : 7168));
        return waves <= (n < 24 ? 2048 : (n < 64 ? 4096 : 4608));
    }
    if (iter2d) return waves <= (n < 128 ? 3072 : 4096) && nodes <= int64_t(6) << 18;
    if (waves > (n < 16 ? 768 : (n < 32 ? 2048 : (n < 128 ? 3072 : 4096)))) return false;
    if (gm.L == 128 && n < 768) return false;
    const int64_t pairs = n + (n / per + 16 > gm.L ? n / per + 16 : gm.L), deque = num_chains > 1024 ? 2 * n + 6 : 0;
    const size_t state = grp_lds_bytes(gm.threads, 8, 8) + 16 * (size_t)pairs, dq = 16 * (size_t)deque;
    const int64_t fit = (int64_t)(159 * 1024 / (state > dq ? state : dq)), at_once = fit < 16 / per ? fit : 16 / per;
    return num_chains <= 256 * at_once;
}

// Which launch a plan is for: the best segmentation depends on the problem's
// data source, so tuned plans are cached per kind and shape.
enum PlanKind {
    kPlanChain = 0,
    kPlan2dCol = 1,
    kPlan2dRow = 2,
    kPlanBatchCol = 3,
    kPlanBatchRow = 4,
    kPlanDp = 5,
    kPlanL1 = 6,
    kPlan2dRowL1 = 7,
    kPlan2dColL1 = 8,  // the TV-l1 solve's column (ROF dual) launch: deeper deques than ROF's
    kPlanKinds = 9
};

// Process-wide tuning: target lanes per launch, shortest segment, halo.
struct SegTuning {
    int64_t target_lanes;
    int64_t min_segment;
    int64_t halo;
    int64_t ring_slots;
};
SegTuning &seg_tuning();
// The plan used for a launch of num_chains chains of length <= n: the tuned
// plan of this kind, shape and working precision (elem bytes; 8 for TV-l1 sets,
// which are FP64 on either data) if one was chosen (tv_*_autotune), else the
// process-wide tuning.
// nodes: of all chains, num_chains * n if 0.
SegPlan seg_plan(int64_t num_chains, int64_t n, int kind, size_t elem, int64_t nodes = 0);
SegPlan seg_default_plan(int64_t num_chains, int64_t n);
void seg_set_tuned(int kind, int64_t num_chains, int64_t n, const SegPlan &p, size_t elem);
void seg_clear_tuned();
// Tag of a TV-l1 breakpoint (slope tag and jump; defined in l1_core.h).
template <typename T> struct TagJ;

// Candidate plans for the autotuner (the default plan first); every workspace
// query reserves room for the largest of them, so a tuned plan always fits.
// G is the tag type of the deque entries (T when a_i = 1, FP64 otherwise).
template <typename T, typename G = T>
int seg_candidates(int64_t num_chains, int64_t n, SegPlan *out, int max_out, bool iter2d = false);
template <typename T, typename G = T>
size_t seg_bytes_max(int64_t num_chains, int64_t n, int kind);

template <typename T>
size_t chain_prox_ws_bytes(const ChainBatch &b, const SegPlan &plan);
// Workspace bytes of one launch of num_chains chains of length <= n under plan.
template <typename T, typename G = T>
size_t seg_ws_bytes_plan(int64_t num_chains, int64_t n, const SegPlan &plan);

template <typename T>
hipError_t launch_chain_prox(const ChainBatch &b, const T *y, const T *w, T w_scalar, T *x, void *workspace,
                             const SegPlan &plan, hipStream_t stream);

// Up to kMaxChainBatches uniform batches in one launch (see tv_chain_prox_multi).
constexpr int kMaxChainBatches = 8;
template <typename T>
hipError_t launch_chain_prox_multi(int nb, const ChainBatch *bs, const T *const *y, const T *const *w,
                                   const double *w_scalar, T *const *x, void *workspace, const SegPlan &plan,
                                   hipStream_t stream);

// General unaries and asymmetric weights (see tv_chain_dp): workspace bytes
// with seg_bytes for the segmented kernels, and the launch.
template <typename T>
size_t chain_dp_ws_bytes(int64_t num_chains, int64_t n, size_t seg_bytes);
template <typename T>
hipError_t launch_chain_dp(const ChainBatch &b, const T *a, const T *bv, const T *wm, const T *wp, T *x,
                           void *workspace, const SegPlan &plan, hipStream_t stream);

// TV-l1 chain prox (see tv_chain_prox_l1): workspace bytes and the launch.
template <typename T>
size_t chain_l1_ws_bytes(int64_t num_chains, int64_t n);
template <typename T>
hipError_t launch_chain_l1(const ChainBatch &b, const T *y, const T *d, const T *w, T w_scalar, const T *c,
                           T c_scalar, T *x, void *workspace, hipStream_t stream);

// Algorithm 2 on a batch of trees (see tv_tree_dp); the launch reads the
// post-order check back into *bad_host and synchronizes the stream.
size_t tree_dp_ws_bytes(int64_t num_trees, int64_t num_nodes);
template <typename T>
hipError_t launch_tree_dp(int64_t num_trees, int64_t num_nodes, const int64_t *offsets, const int64_t *parent,
                          const T *a, const T *b, const T *c, const T *d, const T *wm, const T *wp, T *x,
                          void *workspace, int *bad_host, hipStream_t stream);

template <typename T>
hipError_t launch_chain_adjoint(const ChainBatch &b, const T *x, const T *g, T *gy, T *gw,
                                int w_per_edge, hipStream_t stream);

}  // namespace tvc
