"""Slice panels of the split plans: operand lines are stored in panels of 32,
the last one of an operand shorter, and a tile's lines may begin anywhere in a
panel (stripe columns that start at a later operator position).  Sector sizes
around the panel edge, one- and two-sided site shifts, all slice counts."""
import numpy as np
import pytest

from paper_2309_16724_amd.synth.problem import random_problem

pytestmark = pytest.mark.gpu

# fixed-point slicing with 8-bit slices: error about 2^-8s relative to the line
# maxima, times the cancellation in H.psi (the bounds of the split plans' tests)
BOUND = {3: 5e-6, 5: 1e-10, 7: 1e-13}


@pytest.mark.parametrize("D,Dr", [(24, 40), (64, 64), (90, 33), (130, 270)])
def test_panels_match_oracle(D, Dr):
    import torch
    from oracle.hpsi import HEff
    from paper_2309_16724_amd.hpsi import Plan
    assert torch.cuda.is_available()
    prob = random_problem(7, 6, 0, 11, D=D, D_right=Dr, cap=False)
    he = HEff(prob)
    x = np.random.default_rng(2).standard_normal(he.size)
    ref = he.apply(x)
    for ns in sorted(BOUND):
        plan = Plan(prob, precision=1, n_slices=ns)
        y = plan.apply(torch.from_numpy(x).cuda()).cpu().numpy()
        plan.free()
        print("D %d %d s %d: %.3e" % (D, Dr, ns, np.abs(y - ref).max() / np.abs(ref).max()), flush=True)
        assert np.abs(y - ref).max() <= BOUND[ns] * np.abs(ref).max()
