"""A row's output of the learned preconditioner does not depend on the rows
beside it: calls of few rows split the columns of the hidden layers over the
wavefronts (up to 32768 rows), larger ones do not, and both add a row's terms in
the same order.  Bitwise, so no tolerance; the large call is compared with the
oracle (2e-5 norm-wise, as in the other tests of the forward pass)."""
import numpy as np
import pytest

from oracle import mlp as omlp
from paper_2309_16724_amd.synth.mlp_inputs import mlp_batch, mlp_params

pytestmark = pytest.mark.gpu

MANY = 32769    # the smallest call without the split


@pytest.mark.parametrize("width", [32, 64, 128, 256])
def test_forward_rows_are_independent(width):
    import torch
    from paper_2309_16724_amd.precond import MLP
    assert torch.cuda.is_available()
    p = mlp_params(2, width, 21)
    x = mlp_batch(MANY, 2, 22)[0]
    net = MLP(width, seed=0)
    net.set_params(p)
    xd = torch.from_numpy(x).cuda()
    g = net.forward(xd).cpu().numpy()
    ref, _ = omlp.forward(p.astype(np.float64), x, width)
    assert np.linalg.norm(g - ref) <= 2e-5 * np.linalg.norm(ref)
    for n in (1, 15, 16, 17, 4096, MANY - 2, MANY - 1):
        assert np.array_equal(net.forward(xd[:n].contiguous()).cpu().numpy(), g[:n]), n
    net.free()


@pytest.mark.parametrize("width", [64, 256])
def test_step_elements_are_independent(width):
    import torch
    from paper_2309_16724_amd.precond import MLP
    net = MLP(width, seed=0)
    net.set_params(mlp_params(2, width, 23))
    rng = np.random.default_rng(24)
    d = torch.from_numpy(rng.standard_normal(MANY) * 3.0).cuda()
    r = torch.from_numpy(rng.standard_normal(MANY) * 1e-4).cuda()

    def step(n):
        return net.step(d[:n].contiguous(), r[:n].contiguous(), [0, n], [-9.0], [7.5], [2e-3]).cpu().numpy()

    t = step(MANY)
    for n in (33, MANY - 1):
        assert np.array_equal(step(n), t[:n]), n
    net.free()
