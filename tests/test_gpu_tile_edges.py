"""Sizes at which the kernels' work is cut differently, against the oracle.

FP64 tiles of H.psi: sector sizes around the edges of the 128 x 128 and 64 x 64
work-group tiles (48, 64, 96, 128), K blocks of 1 to 5 states, whose position
walk crosses a boundary inside one K step, and plans of a few tiles up to
thousands.  Sums of FP64 products in another order: 1e-12 of the largest
element.  Learned preconditioner: row counts around the change from four
column groups to one and around the row groups' edges, widths of one to eight
fragments, at the tolerances of its other tests (2e-5 norm-wise forward, 1e-6
loss and gradient)."""
import numpy as np
import pytest

from paper_2309_16724_amd.synth.problem import exact_problem, random_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,l,D,Dr", [(6, 6, 300, 300), (6, 6, 340, 700), (6, 6, 620, 150), (6, 6, 160, 640)])
def test_f64_tiles_match_oracle(L, l, D, Dr):
    import torch
    from oracle.hpsi import HEff
    from paper_2309_16724_amd import binding as B
    from paper_2309_16724_amd.hpsi import Plan
    assert torch.cuda.is_available()
    prob = random_problem(L, l, 0, 5, D=D, D_right=Dr, cap=False)
    t = B.debug_plan_tiles(prob, 2)
    he = HEff(prob)
    x = np.random.default_rng(3).standard_normal(he.size)
    ref = he.apply(x)
    plan = Plan(prob)
    y = plan.apply(torch.from_numpy(x).cuda()).cpu().numpy()
    plan.free()
    print("D %d %d: kinds %s, rows %s, err %.2e" % (D, Dr, sorted(set(t[:, 6])), sorted(set(t[:, 4])),
                                                    np.abs(y - ref).max() / np.abs(ref).max()), flush=True)
    assert np.abs(y - ref).max() <= 1e-12 * np.abs(ref).max()


@pytest.mark.parametrize("prob", [lambda: exact_problem(6, 6, 0, 0), lambda: exact_problem(8, 6, 0, 0),
                                  lambda: random_problem(8, 8, 0, 4, D=20, cap=False)])
def test_small_k_blocks_match_oracle(prob):
    import torch
    from oracle.hpsi import HEff
    from paper_2309_16724_amd.hpsi import Plan
    prob = prob()
    he = HEff(prob)
    x = np.random.default_rng(8).standard_normal(he.size)
    ref = he.apply(x)
    plan = Plan(prob)
    for _ in range(3):   # the launches alternate between two sets of queue counters
        y = plan.apply(torch.from_numpy(x).cuda()).cpu().numpy()
        assert np.abs(y - ref).max() <= 1e-12 * np.abs(ref).max()
    plan.free()


@pytest.mark.parametrize("n", [15, 16, 17, 63, 65, 8191, 8192, 8193, 16400])
def test_learned_preconditioner_row_counts(n):
    import torch
    from oracle import mlp as omlp
    from paper_2309_16724_amd.precond import MLP
    from paper_2309_16724_amd.synth.mlp_inputs import mlp_batch, mlp_params
    W = 256
    p = mlp_params(2, W, 3)
    x, a, b = mlp_batch(n, 2, 4)
    net = MLP(W, seed=0)
    net.set_params(p)
    dev = [torch.from_numpy(np.ascontiguousarray(v)).cuda() for v in (x, a, b)]
    g = net.forward(dev[0]).cpu().numpy()
    ref, _ = omlp.forward(p.astype(np.float64), x, W)
    loss, gr = net.loss_grad(*dev)
    gr = gr.cpu().numpy()
    lref, gref = omlp.grad(p.astype(np.float64), x, a, b, W)
    net.free()
    assert np.linalg.norm(g - ref) <= 2e-5 * np.linalg.norm(ref)
    assert abs(loss - lref) <= 1e-6 * lref
    assert np.linalg.norm(gr - gref) <= 1e-6 * np.linalg.norm(gref)
