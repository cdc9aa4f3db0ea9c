"""Transposed copies (U before a renormalization, operators applied as
adjoints) are made in 32 x 32 pieces, element by element for blocks of fewer
than 16 rows or columns: an H.psi whose sectors lie on both sides of those
sizes, and whose operators are used as adjoints, against the oracle (FP64 sums
in another order: 1e-12 of the largest element)."""
import numpy as np
import pytest

from paper_2309_16724_amd.synth.problem import random_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,Dr", [(120, 120), (210, 100), (100, 420)])
def test_transposed_operators_match_oracle(D, Dr):
    import torch
    from oracle.hpsi import HEff
    from paper_2309_16724_amd.hpsi import Plan
    assert torch.cuda.is_available()
    prob = random_problem(6, 6, 0, 9, D=D, D_right=Dr, cap=False)
    he = HEff(prob)
    x = np.random.default_rng(1).standard_normal(he.size)
    ref = he.apply(x)
    plan = Plan(prob)
    y = plan.apply(torch.from_numpy(x).cuda()).cpu().numpy()
    plan.free()
    print(D, Dr, np.abs(y - ref).max() / np.abs(ref).max(), flush=True)
    assert np.abs(y - ref).max() <= 1e-12 * np.abs(ref).max()
