"""Plans of few tiles cut their outputs' K ranges finer than the default kpart,
so that the tiles fill the GPU: the parts cover the same products, an explicit
kpart is taken as it is, and the results agree with the oracle and with the
unrefined plan."""
import numpy as np
import pytest

from oracle.hpsi import HEff
from paper_2309_16724_amd import binding as B
from paper_2309_16724_amd.synth.problem import exact_problem, random_problem

CASES = {"exact8": lambda: exact_problem(8, 8, 0, 0),
         "one_cell": lambda: exact_problem(4, 4, 0, 0),
         "ragged": lambda: random_problem(7, 6, 0, 11, D=130, D_right=270, cap=False)}
# sums of a few thousand products in another order: 1e-13 of the largest element
TOL = 1e-12


@pytest.mark.parametrize("name", sorted(CASES))
def test_fine_parts_cover_the_same_products(name):
    prob = CASES[name]()
    t = B.debug_plan_tiles(prob, 2)
    t0 = B.debug_plan_tiles(prob, 2, kpart=2048)
    assert len(t) >= len(t0)
    if name == "exact8":
        assert len(t) >= 4 * len(t0)
    work = [(2 * a[:, 0] * a[:, 1] * a[:, 3]).sum() for a in (t, t0)]
    assert work[0] == work[1]
    x = np.random.default_rng(4).standard_normal(HEff(prob).size)
    y, _ = B.debug_plan_host_apply(prob, x)
    y0, _ = B.debug_plan_host_apply(prob, x, kpart=2048)
    assert np.abs(y - y0).max() <= TOL * np.abs(y0).max()


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(CASES))
def test_fine_parts_match_oracle(name):
    import torch
    from paper_2309_16724_amd.hpsi import Plan
    assert torch.cuda.is_available()
    prob = CASES[name]()
    he = HEff(prob)
    x = np.random.default_rng(6).standard_normal(he.size)
    ref = he.apply(x)
    for kw in (dict(), dict(kpart=2048), dict(kpart=64)):
        plan = Plan(prob, **kw)
        y = plan.apply(torch.from_numpy(x).cuda()).cpu().numpy()
        plan.free()
        print(name, kw, np.abs(y - ref).max() / np.abs(ref).max(), flush=True)
        assert np.abs(y - ref).max() <= TOL * np.abs(ref).max()
