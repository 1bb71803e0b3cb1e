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
