"""The chain prox with its deque spread over the lanes of a group (a workgroup per
chain): small launches take it, and so do the chains that the lane-per-segment
kernels hand on (a deque deeper than the ring, a segment whose repair did not
meet the first pass).  Both ways give the bits of the sequential run."""
import numpy as np
import pytest
import torch

import oracle
from paper_1502_07770_amd import binding, synth

pytestmark = pytest.mark.gpu
TOL = {torch.float32: 1e-4, torch.float64: 1e-12}  # of the data range, as for every chain prox


@pytest.fixture
def tuning():
    saved = binding.get_tuning()
    yield binding.set_tuning
    binding.set_tuning(**saved)


def _data(kind, C, n, seed):
    """(y, w): ordinary chains; square-root ramps whose deques hold from a few to
    hundreds of breakpoints; constant data with zero weights (two breakpoints more
    per node, the most there can be)."""
    if kind == "piecewise":
        return synth.piecewise_constant(C, n, seed=seed), synth.edge_weights((C, n), lo=0.05, hi=0.8, seed=seed + 1)
    if kind == "ramp":
        y = np.sqrt(np.arange(n)[None, :] + 3.0 * np.arange(C)[:, None])
        return y, np.repeat(np.array([(0.5, 3.0, 10.0, 100.0)[c % 4] for c in range(C)])[:, None], n, axis=1)
    y, w = np.ones((C, n)), np.zeros((C, n))
    w[:, n // 2:] = 0.25
    y[:, n // 2:] += 0.1 * synth.normal((C, n - n // 2), seed=seed)
    return y, w


SHAPES = [(3, 1), (2, 2), (5, 15), (4, 16), (3, 17), (7, 31), (2, 33), (3, 96), (2, 97), (9, 513), (2, 2048),
          (2, 2049), (1, 6144), (1, 6145), (1100, 130)]


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("kind", ["piecewise", "ramp", "flat"])
def test_group_kernel_equals_lane_kernels(tuning, kind, dtype):
    for C, n in SHAPES:
        if kind != "piecewise" and n > 2049:
            continue  # one lane's walk over hundreds of breakpoints a node
        y, w = _data(kind, C, n, seed=C + n)
        yt, wt = torch.tensor(y, dtype=dtype, device="cuda"), torch.tensor(w, dtype=dtype, device="cuda")
        tuning(target_lanes=1 << 17, min_segment=128, halo=128, ring_slots=16)  # the default: a workgroup per chain
        rows = binding.chain_prox(yt, wt, dim=1)
        cols = binding.chain_prox(yt.t().contiguous(), wt.t().contiguous(), dim=0).t()
        tuning(target_lanes=1, min_segment=1, ring_slots=32)  # one lane per chain
        ref = binding.chain_prox(yt, wt, dim=1)
        assert torch.equal(rows, ref), (kind, C, n)
        assert torch.equal(cols, ref), (kind, C, n)
        if C * n < 20000:
            yv, wv = yt.double().cpu().numpy(), wt.double().cpu().numpy()
            err = np.abs(ref.double().cpu().numpy() - oracle.chain_prox(yv, w=wv)).max()
            assert err <= TOL[dtype] * max(np.ptp(yv), 1.0), (kind, C, n, err)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("n", [300, 4100, 20000])
def test_handed_on_chains_equal_the_sequential_run(tuning, n, dtype):
    """Without a halo and with 16 ring slots most chains are handed on: their lambda pairs
    stay in LDS at 300 nodes and go through memory at 20,000."""
    y = np.concatenate([synth.piecewise_constant(40, n, seed=n), np.sqrt(np.arange(n)[None, :] + np.arange(3)[:, None])])
    w = np.full((43, n), 0.7)
    w[40], w[41], w[42] = 1.0, 5.0, 60.0
    yt, wt = torch.tensor(y, dtype=dtype, device="cuda"), torch.tensor(w, dtype=dtype, device="cuda")
    tuning(target_lanes=1 << 30, min_segment=32, halo=0, ring_slots=16)
    got = binding.chain_prox(yt, wt, dim=1)
    tuning(target_lanes=1, min_segment=1, ring_slots=32)
    assert torch.equal(got, binding.chain_prox(yt, wt, dim=1))


def test_short_weights_and_many_chains(tuning):
    """A scalar weight of zero, one chain of one node in a batch of batches, and more chains
    than blocks with a deque of their own in memory."""
    for dtype in (torch.float32, torch.float64):
        y = torch.rand(2500, 40, dtype=dtype, device="cuda")
        z = torch.rand(1, 5, dtype=dtype, device="cuda")
        a = binding.chain_prox_multi([(y, 1), (z, 0), (y, 0)], [0.0, 0.3, 2.0])
        tuning(target_lanes=1, min_segment=1, ring_slots=32)
        b = binding.chain_prox_multi([(y, 1), (z, 0), (y, 0)], [0.0, 0.3, 2.0])
        assert all(torch.equal(u, v) for u, v in zip(a, b))
        binding.reset_tuning()


@pytest.mark.parametrize("dtype,shape", [(torch.float32, (2048, 2048)), (torch.float32, (2200, 2150)),
                                         (torch.float64, (1100, 4096)), (torch.float64, (1027, 4097)),
                                         (torch.float64, (1024, 4600))])
def test_2d_solves_of_millions_of_nodes(tuning, dtype, shape):
    """The 2D iterations take the group kernel up to 4.7M nodes, the deques of more
    than 1024 chains in LDS (FP64: up to 4096 nodes): the bits of the lane kernels."""
    f = torch.tensor(synth.shapes_image(*shape, sigma=0.1, seed=5), dtype=dtype, device="cuda")
    got = []
    for t in (dict(target_lanes=1 << 17, min_segment=128, halo=128, ring_slots=16),
              dict(target_lanes=1 << 16, min_segment=128, halo=64, ring_slots=32)):
        tuning(**t)
        x, info = binding.Tv2dSolver(*shape, dtype=dtype).solve(f, 0.2, max_iter=3, gap_every=3)
        got.append((x, info["gap_norm"]))
    assert torch.equal(got[0][0], got[1][0]) and got[0][1] == got[1][1]


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_batched_gap_at_the_edges_of_its_row_blocks(dtype):
    """The gap's dual pass sums 64 rows a wave, 1024 a step of the block, columns
    of images of different heights side by side: the single-image gap exactly."""
    shapes = [(1, 40), (63, 3), (64, 65), (65, 7), (128, 1), (1, 1), (1023, 5), (1024, 70), (1025, 33), (2049, 2)]
    imgs = [torch.tensor(synth.shapes_image(*s, sigma=0.1, seed=j), dtype=dtype, device="cuda")
            for j, s in enumerate(shapes)]
    xs, infos = binding.tv2d_batched(imgs, [0.1] * len(imgs), max_iter=6, gap_every=3)
    for f, xb, ib in zip(imgs, xs, infos):
        x1, i1 = binding.tv2d(f, 0.1, max_iter=6, gap_every=3)
        assert torch.equal(xb, x1)
        for k in ("gap_norm", "primal", "dual"):
            assert ib[k] == i1[k], (tuple(f.shape), k)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_segment_lengths_and_wide_segments(tuning, dtype):
    """At the edges of the rule for 16-node segments, and on ramps whose deques
    outgrow 16 lanes in some segments (run by a wave) or 31 breakpoints at a
    segment's end (the whole chain by waves): the bits of one lane per chain."""
    for C, n in [(3, 64), (2, 80), (40, 384), (40, 385), (213, 384), (214, 384), (256, 128), (257, 128), (255, 129)]:
        y, w = _data("piecewise", C, n, seed=n)
        ramp = np.sqrt(np.arange(n)[None, :] + 2.0 * np.arange(C)[:, None])
        ramp[:, ::7] += 0.3 * synth.normal((C, (n + 6) // 7), seed=C)
        for yy, ww in ((y, w), (ramp, np.full((C, n), 1.5)), (ramp, np.full((C, n), 4.0))):
            yt, wt = torch.tensor(yy, dtype=dtype, device="cuda"), torch.tensor(ww, dtype=dtype, device="cuda")
            tuning(target_lanes=1 << 17, min_segment=128, halo=128, ring_slots=16)
            got = binding.chain_prox(yt, wt, dim=1)
            tuning(target_lanes=1, min_segment=1, ring_slots=32)
            assert torch.equal(got, binding.chain_prox(yt, wt, dim=1)), (C, n, ww[0, 0])


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_weighted_data_and_asymmetric_edges_equal_lane_kernels(tuning, dtype):
    """General quadratic unaries and asymmetric edges by groups of lanes: tile,
    anchor-group and segment remainders, deques past 16 lanes, both layouts."""
    shapes = [(3, 1), (2, 2), (5, 7), (5, 8), (4, 9), (4, 17), (3, 33), (40, 385), (2, 511), (9, 520), (1, 2049),
              (1, 6144), (1, 6145), (1100, 270)]
    for C, n in shapes:
        y, w = _data("piecewise", C, n, seed=C + n)
        a = np.exp(synth.normal((C, n), seed=n))
        ramp = np.sqrt(np.arange(n)[None, :] + 2.0 * np.arange(C)[:, None])
        for b, wm, wp, aa in ((a * y, -w, 0.5 * w, a), (ramp, np.full((C, n), -3.0), np.full((C, n), 2.0), None),
                              (a * y, 0.25 * w, w, a)):
            t = [None if v is None else torch.tensor(v, dtype=dtype, device="cuda") for v in (aa, b, wm, wp)]
            tuning(target_lanes=1 << 17, min_segment=128, halo=128, ring_slots=16)
            got = binding.chain_dp(t[1], t[2], t[3], a=t[0], dim=1)
            c = [None if v is None else v.t().contiguous() for v in t]
            cols = binding.chain_dp(c[1], c[2], c[3], a=c[0], dim=0).t()
            tuning(target_lanes=1, min_segment=1, ring_slots=32)
            ref = binding.chain_dp(t[1], t[2], t[3], a=t[0], dim=1)
            assert torch.equal(got, ref) and torch.equal(cols, ref), (C, n)


def _one_lane(tuning, y, w, dtype):
    """Each chain on one lane with the largest ring (FP32 128 slots, FP64 32): chains whose deque
    the ring holds stay there whole.  Returns x and whether the ring held every chain."""
    yv, wv = y.double().cpu().numpy(), w.double().cpu().numpy()
    _, st = oracle.chain_prox(yv, w=wv, counts=True)
    tuning(target_lanes=1, min_segment=1, halo=128, ring_slots=128)
    return binding.chain_prox(y, w, dim=1), st[:, 2] + 2 < (128 if dtype == torch.float32 else 32)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("C,n,L,halo", [(3, 70000, 32, 48), (3, 70000, 32, 0), (40, 5000, 64, 32), (300, 600, 32, 32),
                                        (2000, 400, 32, 16), (1, 33, 32, 0), (5, 97, 32, 0)])
def test_segments_redone_by_lanes_and_by_groups(tuning, C, n, L, halo, dtype):
    """Short halos leave a few or most segments repaired from a wrong state: redone by the
    chain's lane or the chain solved whole by a workgroup, the bits of one lane per chain."""
    for seed, wv in enumerate((0.2, 0.6, 1.5)):
        y = synth.piecewise_constant(C, n, seed=n + seed)
        w = wv * synth.edge_weights((C, n), lo=0.5, hi=1.0, seed=seed)
        yt, wt = torch.tensor(y, dtype=dtype, device="cuda"), torch.tensor(w, dtype=dtype, device="cuda")
        ref, held = _one_lane(tuning, yt, wt, dtype)
        assert held.all()
        tuning(target_lanes=1 << 30, min_segment=L, halo=halo, ring_slots=32)
        assert torch.equal(binding.chain_prox(yt, wt, dim=1), ref), wv


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("C,n", [(3000, 300), (1100, 1000), (40, 5000), (6, 9000)])
def test_deep_chains_side_by_side(tuning, C, n, dtype):
    """Ramps of 16 to some 300 breakpoints among shallow chains, several to a block of the
    list: by a wave where a part is wide, by a lane each in the block's LDS where all is.
    The bits of one lane per chain where its ring holds the deque, else the oracle's values."""
    y = synth.piecewise_constant(C, n, seed=n)
    w = np.full((C, n), 0.4)
    ramp = np.arange(C) % 3 > 0
    y[ramp] = np.sqrt(np.arange(n)[None, :] + 3.0 * np.arange(ramp.sum())[:, None])
    y[1::6] += 0.05 * synth.normal(y[1::6].shape, seed=C)
    w[ramp] = np.array([(0.5, 2.0, 10.0, 100.0)[c % 4] for c in range(ramp.sum())])[:, None]
    yt, wt = torch.tensor(y, dtype=dtype, device="cuda"), torch.tensor(w, dtype=dtype, device="cuda")
    ref, held = _one_lane(tuning, yt, wt, dtype)
    assert 0 < held.sum() < C
    tuning(target_lanes=1 << 30, min_segment=128, halo=64, ring_slots=16)
    got = binding.chain_prox(yt, wt, dim=1)
    assert torch.equal(got[torch.tensor(held, device="cuda")], ref[torch.tensor(held, device="cuda")])
    pick = np.concatenate([np.nonzero(~held)[0][:40], np.nonzero(held)[0][:10]])
    yv, wv = yt.double().cpu().numpy()[pick], wt.double().cpu().numpy()[pick]
    err = np.abs(got.double().cpu().numpy()[pick] - oracle.chain_prox(yv, w=wv)).max(axis=1)
    assert (err <= TOL[dtype] * np.maximum(np.ptp(yv, axis=1), 1.0)).all()


def test_deques_that_outgrow_the_blocks_lds(tuning):
    """1500 constant nodes with zero weights hold 3000 breakpoints (FP64), more than the LDS of
    a block of the list: one lane in HBM, the bits of the small launch's walk there."""
    n = 1500
    y, w = np.ones((5, n)), np.zeros((5, n))
    w[:, n - 60:] = 0.25
    y[:, n - 60:] += 0.1 * synth.normal((5, 60), seed=3)
    y[1] += np.linspace(0.0, 1.0, n)
    yt, wt = torch.tensor(y, device="cuda"), torch.tensor(w, device="cuda")
    small = binding.chain_prox(yt, wt, dim=1)
    tuning(target_lanes=1 << 30, min_segment=128, halo=64, ring_slots=16)
    got = binding.chain_prox(yt, wt, dim=1)
    assert torch.equal(got, small)
    assert np.abs(got.cpu().numpy() - oracle.chain_prox(y, w=w)).max() <= TOL[torch.float64]


def test_sizes_of_lds_from_several_threads():
    """Launches of one kernel with little and with most of the LDS, on streams of four threads."""
    import threading
    ys = [torch.rand(40, n, dtype=torch.float64, device="cuda") for n in (100, 6000, 500, 5000)]
    refs = [binding.chain_prox(y, 0.3, dim=1) for y in ys]
    torch.cuda.synchronize()
    errors = []

    def work(k):
        try:
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                for _ in range(50):
                    x = binding.chain_prox(ys[k], 0.3, dim=1)
                s.synchronize()
                if not torch.equal(x, refs[k]):
                    errors.append(k)
        except Exception as e:  # noqa: BLE001
            errors.append(e)
    ts = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not errors, errors


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_both_sides_of_the_rule_give_the_same_bits(tuning, dtype):
    """Chains of 2 to 400 nodes around the numbers at which the default changes kernels and
    segment lengths, by rows and by columns."""
    for C, n in [(768, 2), (769, 2), (2048, 23), (2049, 23), (3072, 33), (4097, 60), (4608, 100), (4609, 100), (448, 256),
                 (449, 256), (204, 384), (205, 384), (1100, 300), (4700, 130)]:
        y, w = _data("piecewise", C, n, seed=C + n)
        yt, wt = torch.tensor(y, dtype=dtype, device="cuda"), torch.tensor(w, dtype=dtype, device="cuda")
        tuning(target_lanes=1 << 17, min_segment=128, halo=128, ring_slots=16)  # the default
        rows = binding.chain_prox(yt, wt, dim=1)
        cols = binding.chain_prox(yt.t().contiguous(), wt.t().contiguous(), dim=0).t()
        ref, held = _one_lane(tuning, yt, wt, dtype)
        assert held.all()
        assert torch.equal(rows, ref) and torch.equal(cols, ref), (C, n)
