"""GPU parity of the workgroup-per-instance kernels (quartic family) against the CPU oracle, at
the sizes where their tiles, panels and blocks of rows end: multiples of 16 and 64 and their
neighbours. The bars are those of tests/parity.py.
"""
import numpy as np
import pytest

import oracle
from paper_2106_14995_amd import workloads as W
from parity import check_parity, oracle_ref

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tron():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2106_14995_amd import tron as T
    T.lib()
    return T


def result(r):
    import torch
    torch.cuda.synchronize()
    return {k: v.cpu().numpy() for k, v in zip(("x", "f", "status", "iters"), r)}


def batch(count, n):
    """count instances; the first has a third of its variables fixed, and the second starts
    outside its box."""
    bt = W.qp4_batch(count, n, config_id=300 + n)
    bt.hi[:n:3] = bt.lo[:n:3]
    bt.x0[n:2 * n] = 3.0
    return bt


@pytest.mark.parametrize("n", [65, 79, 80, 81, 96, 97, 111, 112, 113, 127, 128, 129, 143, 144, 145, 160, 161, 191, 192, 193, 255, 256, 257, 273, 320, 383, 449, 511, 512])
def test_edges(tron, n):
    bt = batch(3, n)
    h = tron.Batch(bt.family, n, batch=bt.batch)
    check_parity(bt, result(h.solve(*tron.to_device(bt))), oracle_ref(bt), convex=True)
    h.close()


@pytest.mark.parametrize("n", [130, 200, 321])
def test_workspace_strides_agree(tron, n):
    """A handle's workspace slots hold rows of whole lines, the allocation-free call's do not:
    the same bits either way, alone and among others."""
    bt = batch(4, n)
    d = tron.to_device(bt)
    h = tron.Batch(bt.family, n, batch=4)
    a, b = result(h.solve(*d)), result(tron.solve_noalloc(bt.family, n, 4, *d))
    h.close()
    one = bt.subset([2])
    h = tron.Batch(bt.family, n, batch=1)
    c = result(h.solve(*tron.to_device(one)))
    h.close()
    for k in a:
        assert np.array_equal(a[k], b[k]), k
        m = n if k == "x" else 1
        assert np.array_equal(a[k][2 * m:3 * m], c[k]), k


@pytest.mark.parametrize("n", [9, 15, 16, 17, 31, 33, 47, 48, 49, 63, 64, 72, 100])
def test_kernels_agree(tron, n):
    """A few instances run on another kernel or register build than many: the same bits, and
    the oracle's result within the bars."""
    bt = W.qp4_batch(2100 if n < 48 else 260, n, config_id=400 + n)
    h = tron.Batch(bt.family, n, batch=bt.batch)
    a = result(h.solve(*tron.to_device(bt)))
    h.close()
    idx = list(range(0, bt.batch, 131))
    few = bt.subset(idx)
    h = tron.Batch(bt.family, n, batch=few.batch)
    b = result(h.solve(*tron.to_device(few)))
    h.close()
    for k in b:
        m = n if k == "x" else 1
        assert np.array_equal(a[k].reshape(-1, m)[idx].ravel(), b[k]), k
    check_parity(few, b, oracle_ref(few), convex=True)


@pytest.mark.parametrize("n", [72, 128, 144, 193, 257, 400])
def test_shift_retries(tron, n):
    """Half-rank Q: the first factorisations meet non-positive pivots and are repeated."""
    bt = W.qp4_half_rank_batch(3, n, config_id=95)
    st = oracle.solve(bt)["stats"]
    assert np.all(st[:, 3] > st[:, 6]), "no shifted retry in the oracle"
    h = tron.Batch(bt.family, n, batch=3)
    check_parity(bt, result(h.solve(*tron.to_device(bt))), oracle_ref(bt), convex=True)
    h.close()


@pytest.mark.parametrize("nmax,count", [(24, 40), (64, 40), (128, 60), (128, 300)])
def test_bucket_of_many_sizes(tron, nmax, count):
    """One bucket for every size (edge 128): with n > 64 among them the small ones run on a
    workgroup too, in a matrix array of their own stride; same bits as in the default plan."""
    sizes = W.loguniform_sizes(count, 9, nmax, config_id=97)
    sizes[:4] = [9, 16, 17, nmax]
    bt = W.qp4_batch(count, sizes, config_id=97)
    got = []
    for spec in (None, tron.plan_spec(edges=[128], pool_waves=0)):
        h = tron.Batch(bt.family, sizes, spec=spec)
        got.append(result(h.solve(*tron.to_device(bt))))
        h.close()
    for k in got[0]:
        assert np.array_equal(got[0][k], got[1][k]), k
    check_parity(bt, got[1], oracle_ref(bt), convex=True)


def test_more_workgroups_than_one_launch_holds(tron):
    """8,388,651 instances in one bucket on workgroups of 512 threads: more than 2^32 threads. All
    but the first repeat 50 problems of n = 9, and so do their results."""
    import torch
    reps = (1 << 23) // 50 + 1
    one, few = W.qp4_batch(1, 128, config_id=98), W.qp4_batch(50, 9, config_id=99)
    d1, d = tron.to_device(one), tron.to_device(few)
    sizes = np.full(1 + 50 * reps, 9, np.int32)
    sizes[0] = 128
    assert 512 * sizes.size >= 1 << 32
    h = tron.Batch(W.QP4, sizes, spec=tron.plan_spec(edges=[128], pool_waves=0))
    x, f, status, iters = h.solve(*[torch.cat([a, b.repeat(reps)]) for a, b in zip(d1, d)])
    torch.cuda.synchronize()
    h.close()
    h = tron.Batch(W.QP4, 9, batch=50)
    rx, rf, rs, ri = h.solve(*d)
    torch.cuda.synchronize()
    h.close()
    assert bool((x[128:].view(reps, -1) == rx).all())
    for a, b in ((f, rf), (status, rs), (iters, ri)):
        assert bool((a[1:].view(reps, -1) == b).all())
    h = tron.Batch(W.QP4, 128, batch=1)
    assert bool((h.solve(*d1)[0] == x[:128]).all())
    h.close()


@pytest.mark.parametrize("n", [80, 128, 129, 200, 300])
def test_starts_and_bounds(tron, n):
    """Crossed bounds, a NaN start, no bounds and one-sided bounds among ordinary instances."""
    bt = W.qp4_batch(6, n, config_id=310 + n)
    at = lambda b, i: b * n + i
    bt.lo[at(1, n - 1)] = 5.0                                      # l > u, in the last row
    bt.x0[at(2, 70)] = np.nan
    bt.lo[at(3, 0):at(4, 0)], bt.hi[at(3, 0):at(4, 0)] = -np.inf, np.inf
    bt.lo[at(4, 0):at(5, 0):2], bt.hi[at(4, 1):at(5, 0):2] = -np.inf, np.inf
    h = tron.Batch(bt.family, n, batch=6)
    g = result(h.solve(*tron.to_device(bt)))
    h.close()
    ref = oracle_ref(bt)
    assert list(g["status"]) == list(ref["status"]) == [0, 4, 3, 0, 0, 0]
    assert np.array_equal(g["x"][at(1, 0):at(2, 0)], bt.x0[at(1, 0):at(2, 0)])
    check_parity(bt, g, ref, convex=True)


@pytest.mark.parametrize("n", [80, 128, 129, 200, 300])
def test_in_place_and_warm(tron, n):
    """x0 and x in one buffer; a start from a given radius and step length, which is the cold
    start with that radius; a restart from the solution, which takes no iteration."""
    import torch
    bt = batch(3, n)
    h = tron.Batch(bt.family, n, batch=3, opts=tron.options(delta0=0.5))
    cold = result(h.solve(*tron.to_device(bt)))
    params, lo, hi, x = tron.to_device(bt)
    inplace = result(h.solve(params, lo, hi, x, x=x))
    h.set_options(tron.options(warm=True))
    h.set_state(torch.tensor([0.5] * 3 + [1.0] * 3, device="cuda", dtype=torch.float64))
    warm = result(h.solve(*tron.to_device(bt)))
    again = result(h.solve(params, lo, hi, x, x=x))
    h.close()
    for k in cold:
        assert np.array_equal(cold[k], inplace[k]) and np.array_equal(cold[k], warm[k]), k
    assert np.all(again["iters"] == 0) and np.array_equal(again["x"], cold["x"])
