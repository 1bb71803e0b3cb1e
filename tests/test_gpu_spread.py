"""How a batch is spread over the wavefronts does not show in its results: the kernels that hold
several instances per wavefront solve a small batch with few of them in each, the other lanes
repeating one, and a large batch with all lanes their own. Every instance has the same bits
either way, at counts around the steps of that rule and with an incomplete last wavefront.
"""
import numpy as np
import pytest

from paper_2106_14995_amd import workloads as W

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
    return [v.cpu().numpy() for v in r]


def agree(many, few, per):
    for i, (a, b) in enumerate(zip(many, few)):
        m = per if i == 0 else 1
        assert np.array_equal(a.reshape(-1, m)[:b.size // m], b.reshape(-1, m)), i


@pytest.mark.parametrize("plan", [dict(lane_group=1), dict(lane_group=4), dict(lane_group=8), dict(lane_group=1, lane_block=256)])
@pytest.mark.parametrize("n", [3, 6, 8])
def test_quartic(tron, n, plan):
    bt = W.qp4_batch(20000, n, config_id=500 + n)

    def solve(b):
        h = tron.Batch(b.family, n, batch=b.batch, spec=tron.plan_spec(**plan))
        r = result(h.solve(*tron.to_device(b)))
        h.close()
        return r

    many = solve(bt)
    for count in (1, 63, 1023, 1025, 2047, 2050, 8200):
        agree(many, solve(bt.subset(list(range(count)))), n)


def test_branches(tron):
    bt = W.br6_batch(34000, config_id=510)

    def solve(b):
        h = tron.Batch(b.family, 6, batch=b.batch)
        r = result(h.solve(*tron.to_device(b)))
        h.close()
        return r

    many = solve(bt)
    for count in (1, 1025, 5000):
        agree(many, solve(bt.subset(list(range(count)))), 6)


def test_multiplier_loop(tron):
    bt = W.br8l_batch(3000, config_id=520)

    def solve(b):
        h = tron.Batch(b.family, 8, batch=b.batch)
        d = tron.to_device(b)
        r = result(h.al_solve(*d)) + [d[0].cpu().numpy()]
        h.close()
        return r

    many = solve(bt)
    for count in (1, 1023, 1025, 2049):
        few = solve(bt.subset(list(range(count))))
        agree(many[:-1], few[:-1], 8)
        assert np.array_equal(many[-1].reshape(-1, 40)[:count], few[-1].reshape(-1, 40))


@pytest.mark.parametrize("family,n,group", [(W.QP4, 9, 8), (W.QP4, 16, 8), (W.QP4, 9, 16), (W.QP4, 16, 16), (W.HS45M, 16, 8), (W.HS45M, 16, 16)])
def test_groups_to_16(tron, family, n, group):
    bt = W.qp4_batch(2500, n, config_id=530 + n) if family == W.QP4 else W.hs45m_random_start(2500, n, config_id=530 + n)

    def solve(b):
        h = tron.Batch(family, n, batch=b.batch, spec=tron.plan_spec(group16=group))
        r = result(h.solve(*tron.to_device(b)))
        h.close()
        return r

    many = solve(bt)
    for count in (1, 127, 129, 255, 257, 1025):
        agree(many, solve(bt.subset(list(range(count)))), n)


@pytest.mark.parametrize("family,n,group", [(W.HS45M, 3, 1), (W.HS45M, 8, 1), (W.HS45M, 8, 8), (W.BR6, 6, 8), (W.BR6, 6, 4)])
def test_other_families(tron, family, n, group):
    bt = W.br6_batch(9000, config_id=540) if family == W.BR6 else W.hs45m_random_start(9000, n, config_id=540 + n)

    def solve(b):
        h = tron.Batch(family, n, batch=b.batch, spec=tron.plan_spec(lane_group=group))
        r = result(h.solve(*tron.to_device(b)))
        h.close()
        return r

    many = solve(bt)
    for count in (1, 130, 1025, 4096, 4097):
        agree(many, solve(bt.subset(list(range(count)))), n)


@pytest.mark.parametrize("group", [1, 8])
def test_in_place(tron, group):
    """x0 and x in one buffer where idle lanes repeat an instance: uniform batches, and packs of
    one size of a mixed batch that are not full."""
    for sizes in (np.full(300, 8, np.int32), np.full(70, 3, np.int32), W.loguniform_sizes(500, 1, 8, config_id=550)):
        bt = W.qp4_batch(len(sizes), sizes, config_id=550)
        uniform = len(set(sizes)) == 1
        spec = tron.plan_spec(lane_group=group)
        h = tron.Batch(bt.family, int(sizes[0]) if uniform else sizes, batch=len(sizes) if uniform else None, spec=spec)
        apart = result(h.solve(*tron.to_device(bt)))
        params, lo, hi, x = tron.to_device(bt)
        same = result(h.solve(params, lo, hi, x, x=x))
        h.close()
        for a, b in zip(apart, same):
            assert np.array_equal(a, b)


def test_padded_packs(tron):
    """A mixed batch whose size classes do not fill their packs against one that does."""
    sizes = np.repeat(np.arange(1, 13, dtype=np.int32), 128)
    bt = W.qp4_batch(len(sizes), sizes, config_id=560)
    few = bt.subset([b for b in range(bt.batch) if b % 128 < 5 + b // 128])

    def solve(b):
        h = tron.Batch(b.family, b.n)
        r = result(h.solve(*tron.to_device(b)))
        h.close()
        return r

    many, less = solve(bt), solve(few)
    keep = np.array([b % 128 < 5 + b // 128 for b in range(bt.batch)])
    assert np.array_equal(many[0][np.repeat(keep, sizes)], less[0])
    for a, b in zip(many[1:], less[1:]):
        assert np.array_equal(a[keep], b)


def test_admm_branches(tron):
    """Branch solves spread over a wavefront per CU (up to 4,096 branches) and packed: a network
    alone and beside a copy of itself takes the same iterations."""
    import torch
    import oracle
    net = W.network(nbus=1500, nbranch=2200, ngen=300, config_id=570)
    shifted = lambda v: np.concatenate([v, v + net.nbus])
    twice = lambda v: np.concatenate([v, v])
    two = W.Network(2 * net.nbus, shifted(net.br_from), shifted(net.br_to), twice(net.br_adm), twice(net.br_lo),
                    twice(net.br_hi), shifted(net.gen_bus), twice(net.gen_cost), twice(net.gen_lim), twice(net.bus_load))
    assert net.nbranch <= 4096 < two.nbranch

    def run(nw):
        a = tron.Admm(nw)
        a.step(12)
        v = a.get_state()
        torch.cuda.synchronize()
        a.close()
        return v.cpu().numpy()

    a, b = oracle.admm_views(net, run(net)), oracle.admm_views(two, run(two))
    for k in a:
        assert np.array_equal(a[k], b[k][:len(a[k])]), k
