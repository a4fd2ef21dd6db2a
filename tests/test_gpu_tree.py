"""GPU parity of Algorithm 2 on batches of trees (tv_tree_dp) against the
oracle's forest DP (pinned in tests/test_oracle_tree.py to brute force, a KKT
certificate, the chain case and relabelling).  The GPU computes in FP64 for
either dtype; bars per tree relative to s = max(range of x, range of b / a, 1):
1e-11 with FP64 inputs, 1e-5 with FP32 inputs (the oracle sees the same
rounded inputs)."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_1502_07770_amd import binding, synth

pytestmark = pytest.mark.gpu


def _tree_data(N, seed, l1=True, unit_a=False):
    rng = np.random.default_rng(seed)
    a = np.ones(N) if unit_a else rng.uniform(0.3, 2.0, N)
    b = a * (rng.normal(size=N) * 0.5 + np.repeat(rng.uniform(0, 1, N // 16 + 1), 16)[:N])
    c = rng.uniform(0, 1.0, N) * (rng.random(N) < 0.7) if l1 else np.zeros(N)
    d = np.round(rng.normal(size=N) * 2) / 2
    wp = rng.uniform(0, 0.8, N)
    wm = -rng.uniform(0, 0.8, N)
    return a, b, c, d, wm, wp


def _check(par, off, arrays, xg, trees, tol):
    a, b, c, d, wm, wp = arrays
    for t in trees:
        lo, hi = off[t], off[t + 1]
        p = par[lo:hi].copy()
        p[p >= 0] -= lo
        xo = oracle.tree_pq(p, *(v[lo:hi] for v in (a, b, c, d, wm, wp)))[0]
        s = max(np.ptp(xo), np.ptp(b[lo:hi] / a[lo:hi]), 1.0)
        assert np.abs(xg[lo:hi] - xo).max() <= tol * s, t


@pytest.mark.parametrize("dtype,tol", [(torch.float64, 1e-11), (torch.float32, 1e-5)])
@pytest.mark.parametrize("l1", [True, False])
def test_random_forests_match_oracle(dtype, tol, l1):
    par, off = synth.post_order_forest(300, 150, seed=5)
    arrays = _tree_data(par.size, seed=6, l1=l1)
    dev = [torch.tensor(v, dtype=dtype, device="cuda") for v in arrays]
    arrays = [v.double().cpu().numpy() for v in dev]
    x = binding.tree_dp(torch.tensor(par, device="cuda"), torch.tensor(off, device="cuda"), dev[1], dev[4], dev[5],
                        a=dev[0], c=dev[2] if l1 else None, d=dev[3] if l1 else None)
    _check(par, off, arrays, x.double().cpu().numpy(), range(300), tol)


def test_chain_is_the_chain_dp():
    """parent(i) = i + 1: the general chain DP's result."""
    rng = np.random.default_rng(7)
    C, n = 40, 600
    a, b, _, _, wm, wp = _tree_data(C * n, seed=8, l1=False)
    par = np.arange(1, C * n + 1, dtype=np.int64)
    par[n - 1::n] = -1
    off = np.arange(C + 1, dtype=np.int64) * n
    dev = [torch.tensor(v, device="cuda") for v in (a, b, wm, wp)]
    x = binding.tree_dp(torch.tensor(par, device="cuda"), torch.tensor(off, device="cuda"), dev[1], dev[2], dev[3],
                        a=dev[0]).cpu().numpy().reshape(C, n)
    ref = binding.chain_dp(*(v.reshape(C, n) for v in dev[1:]), a=dev[0].reshape(C, n)).cpu().numpy()
    assert np.abs(x - ref).max() <= 1e-10


def test_single_nodes_and_forest_ranges():
    """Trees of one node (x = argmin of the unary) and ranges holding several
    trees (several roots)."""
    par = np.array([-1, 2, -1, 4, 5, -1, -1], dtype=np.int64)   # ranges [0,1) [1,3) [3,7)
    off = np.array([0, 1, 3, 7], dtype=np.int64)
    arrays = _tree_data(7, seed=9)
    dev = [torch.tensor(v, device="cuda") for v in arrays]
    x = binding.tree_dp(torch.tensor(par, device="cuda"), torch.tensor(off, device="cuda"), dev[1], dev[4], dev[5],
                        a=dev[0], c=dev[2], d=dev[3]).cpu().numpy()
    _check(par, off, arrays, x, range(3), 1e-11)


def test_not_post_order_is_rejected():
    """0 is a child of 2, but 1 (a child of 3) lies between them: the subtree
    {0, 2} is not a contiguous range, so the numbering is rejected."""
    par = np.array([2, 3, 3, -1], dtype=np.int64)
    off = np.array([0, 4], dtype=np.int64)
    dev = [torch.ones(4, dtype=torch.float64, device="cuda") for _ in range(3)]
    with pytest.raises(binding.TvChainError) as e:
        binding.tree_dp(torch.tensor(par, device="cuda"), torch.tensor(off, device="cuda"), *dev)
    assert e.value.status == binding.TV_ERR_INVALID_ARG
    bad_parent = np.array([-1, 0], dtype=np.int64)     # parent below the child
    with pytest.raises(binding.TvChainError):
        binding.tree_dp(torch.tensor(bad_parent, device="cuda"), torch.tensor([0, 2], device="cuda"),
                        *(torch.ones(2, dtype=torch.float64, device="cuda") for _ in range(3)))


def test_full_size_sample_fp32():
    """65,536 trees of 256 nodes (the benchmark's batch); 300 trees checked."""
    par, off = synth.post_order_forest(65536, 256, seed=1)
    arrays = _tree_data(par.size, seed=2)
    dev = [torch.tensor(v, dtype=torch.float32, device="cuda") for v in arrays]
    x = binding.tree_dp(torch.tensor(par, device="cuda"), torch.tensor(off, device="cuda"), dev[1], dev[4], dev[5],
                        a=dev[0], c=dev[2], d=dev[3]).double().cpu().numpy()
    arrays = [v.double().cpu().numpy() for v in dev]
    rng = np.random.default_rng(3)
    _check(par, off, arrays, x, rng.choice(65536, 300, replace=False), 1e-5)


def _stars_and_chains():
    """Trees around the sizes at which a message outgrows a row of lanes or goes to the lane
    kernel: k leaves under a root, k leaves under an inner node (k up to 300), chains with
    large weights (deques of hundreds) and an inner node over two such chains."""
    trees = []
    for k in (1, 4, 5, 6, 7, 13, 14, 15, 16, 40, 41, 42, 43, 130, 300):
        trees.append([k] * k + [-1])
        trees.append([k] * k + [k + 1, -1])
    for n in (2, 17, 200):
        trees.append([j + 1 for j in range(n - 1)] + [-1])
        trees.append([j + 1 for j in range(n - 1)] + [2 * n] + [n + j + 1 for j in range(n - 1)] + [2 * n, 2 * n + 1, -1])
    par, off = [], [0]
    for t in trees:
        par += [p + off[-1] if p >= 0 else -1 for p in t]
        off.append(off[-1] + len(t))
    return np.array(par, dtype=np.int64), np.array(off, dtype=np.int64)


@pytest.mark.parametrize("dtype,tol", [(torch.float64, 1e-11), (torch.float32, 1e-5)])
@pytest.mark.parametrize("kind", ["random", "ties", "wide weights", "no l1"])
def test_message_sizes_match_oracle(dtype, tol, kind):
    """The oracle on trees of every message size, with equal breakpoints (integer data), with
    weights so large that nothing is clipped, and without l1 terms."""
    par, off = _stars_and_chains()
    N = par.size
    a, b, c, d, wm, wp = _tree_data(N, seed=21, l1=kind != "no l1")
    if kind == "ties":
        rng = np.random.default_rng(22)
        a, b = np.ones(N), rng.integers(-2, 3, N).astype(float)
        c, d = rng.integers(0, 2, N).astype(float), rng.integers(-1, 2, N).astype(float)
        wm, wp = -rng.integers(0, 3, N).astype(float), rng.integers(0, 3, N).astype(float)
    if kind == "wide weights":
        wm, wp = 40.0 * wm - 20.0, 40.0 * wp + 20.0
    dev = [torch.tensor(v, dtype=dtype, device="cuda") for v in (a, b, c, d, wm, wp)]
    x = binding.tree_dp(torch.tensor(par, device="cuda"), torch.tensor(off, device="cuda"), dev[1], dev[4], dev[5],
                        a=dev[0], c=dev[2] if kind != "no l1" else None, d=dev[3] if kind != "no l1" else None)
    _check(par, off, [v.double().cpu().numpy() for v in dev], x.double().cpu().numpy(), range(off.size - 1), tol)


def _deep_trees():
    """Trees that change to the lane kernel on the way, at different nodes: paths of smooth
    data, the same below inner nodes with leaves, and several of them under one node, with
    subtrees pending on both sides of the change."""
    trees = []
    for n in (20, 61, 150, 400):
        path = [j + 1 for j in range(n - 1)] + [-1]
        cater = [min(j + 1 + (j % 2), n - 1) for j in range(n - 1)] + [-1]
        q = n // 4
        joined = [n - 1 if j % q == q - 1 else min(j + 1, n - 1) for j in range(n - 1)] + [-1]
        late = [n - 1] * 3 + [j + 1 for j in range(3, n - 1)] + [-1]  # leaves pending below a path
        trees += [path, cater, joined, late, cater, path]
    par, off = [], [0]
    for t in trees:
        par += [p + off[-1] if p >= 0 else -1 for p in t]
        off.append(off[-1] + len(t))
    return np.array(par, dtype=np.int64), np.array(off, dtype=np.int64)


@pytest.mark.parametrize("dtype,tol", [(torch.float64, 1e-11), (torch.float32, 1e-5)])
@pytest.mark.parametrize("l1", [0.0, 0.1, 1.0])
@pytest.mark.parametrize("w", [2.0, 30.0])
def test_trees_handed_over_match_oracle(dtype, tol, l1, w):
    """l1: the share of the nodes with an l1 term, whose messages are cut where they lie and
    are sorted before the lane kernel takes them."""
    par, off = _deep_trees()
    N = par.size
    rng = np.random.default_rng(int(w) + 3)
    a = np.ones(N)
    b = np.concatenate([np.sqrt(np.arange(m) + k) for k, m in enumerate(np.diff(off))])
    c = rng.uniform(0.2, 1.0, N) * (rng.random(N) < l1)
    d = b + rng.normal(size=N)
    dev = [torch.tensor(v, dtype=dtype, device="cuda") for v in (a, b, c, d, np.full(N, -w), np.full(N, 0.7 * w))]
    x = binding.tree_dp(torch.tensor(par, device="cuda"), torch.tensor(off, device="cuda"), dev[1], dev[4], dev[5],
                        c=dev[2] if l1 else None, d=dev[3] if l1 else None)
    _check(par, off, [v.double().cpu().numpy() for v in dev], x.double().cpu().numpy(), range(off.size - 1), tol)


def test_numbering_is_checked_after_the_change_of_kernels():
    """A path that is handed over, then a subtree that is not a contiguous range."""
    n = 60
    par = np.array([j + 1 for j in range(n)] + [n + 3, n + 4, n + 4, n + 4, -1], dtype=np.int64)
    b = torch.tensor(np.sqrt(np.arange(par.size)), device="cuda")
    w = torch.full_like(b, 30.0)
    off = torch.tensor([0, par.size], device="cuda")
    with pytest.raises(binding.TvChainError) as e:
        binding.tree_dp(torch.tensor(par, device="cuda"), off, b, -w, w)
    assert e.value.status == binding.TV_ERR_INVALID_ARG
    par[n + 1:n + 4] = (n + 2, n + 3, n + 4)  # the same as a path: accepted
    par[n] = n + 1
    x = binding.tree_dp(torch.tensor(par, device="cuda"), off, b, -w, w).cpu().numpy()
    o = oracle.tree_pq(par, np.ones(par.size), b.cpu().numpy(), np.zeros(par.size), np.zeros(par.size),
                       -w.cpu().numpy(), w.cpu().numpy())[0]
    assert np.abs(x - o).max() <= 1e-11 * max(np.ptp(o), np.ptp(b.cpu().numpy()))
