"""Learned preconditioner at the edges of its kernels' work split."""
import numpy as np
import pytest

from paper_2309_16724_amd.synth.mlp_inputs import mlp_batch, mlp_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width", [32, 256])
@pytest.mark.parametrize("n", [1, 17, 300])
def test_infinite_gradient_is_no_nan(width, n):
    """Rows that fill up the last block of sixteen add nothing: with positive
    parameters and an infinite feature in the last row, every dW2 is a sum of
    finite and infinite positive terms (exact, no tolerance)."""
    import torch
    from paper_2309_16724_amd.precond import MLP
    assert torch.cuda.is_available()
    p = np.abs(mlp_params(2, width, 31)) + np.float32(0.01)
    x, a, b = mlp_batch(n, 2, 32)
    x = np.abs(x)
    a, b = np.ones_like(a), np.zeros_like(b)
    x[-1, 0] = np.inf
    net = MLP(width, seed=0)
    net.set_params(p)
    grad = net.loss_grad(*[torch.from_numpy(v).cuda() for v in (x, a, b)])[1].cpu().numpy()
    net.free()
    w2 = grad[3 * width:3 * width + width * width]
    assert np.all(w2 == np.inf), w2[:8]


@pytest.mark.parametrize("width", [32, 64, 128, 256])
@pytest.mark.parametrize("n", [100, 257, 4097, 32767, 32768, 32769, 40000])
def test_gradient_at_the_edges_of_the_row_splits(width, n):
    """Forward and backward passes on both sides of the change from four column
    groups to one (32768 rows) and of the row splits' lengths, all widths.  FP32
    storage and layer sums, FP64 backward sums: 2e-5 norm-wise forward, 1e-6 loss
    and gradient, as in the other tests of these kernels."""
    import torch
    from oracle import mlp as omlp
    from paper_2309_16724_amd.precond import MLP
    p = mlp_params(2, width, 33)
    x, a, b = mlp_batch(n, 2, 34)
    net = MLP(width, seed=0)
    net.set_params(p)
    dev = [torch.from_numpy(v).cuda() for v in (x, a, b)]
    g = net.forward(dev[0]).cpu().numpy()
    loss, grad = net.loss_grad(*dev)
    grad = grad.cpu().numpy()
    net.free()
    ref, _ = omlp.forward(p.astype(np.float64), x, width)
    lref, gref = omlp.grad(p.astype(np.float64), x, a, b, width)
    assert np.linalg.norm(g - ref) <= 2e-5 * np.linalg.norm(ref)
    assert abs(loss - lref) <= 1e-6 * lref
    assert np.linalg.norm(grad - gref) <= 1e-6 * np.linalg.norm(gref)


@pytest.mark.parametrize("width", [32, 256])
def test_step_of_many_segments(width):
    """Up to eight segments travel as kernel arguments, more in device memory:
    nine segments, some empty and with ends inside the groups of 16 and 64 rows, of
    which two end beyond 32768 elements.  Against the oracle (1e-5 norm-wise, as
    in the two-segment test) and against one call per segment (bitwise: the same
    sums in the same order)."""
    import torch
    from oracle import mlp as omlp
    from paper_2309_16724_amd.precond import MLP
    p = mlp_params(2, width, 35)
    net = MLP(width, seed=0)
    net.set_params(p)
    rng = np.random.default_rng(36)
    off = np.array([0, 7, 7, 80, 1000, 1003, 20011, 33333, 39999, 40017])
    d, r = rng.standard_normal(off[-1]) * 3.0, rng.standard_normal(off[-1]) * 1e-3
    seg = [slice(a, b) for a, b in zip(off[:-1], off[1:])]
    theta = [float(d[s].min() - 0.4) if s.stop > s.start else -9.0 for s in seg]
    sigma = [float(np.sqrt(np.mean((d[s] - t) ** 2))) if s.stop > s.start else 1.0 for s, t in zip(seg, theta)]
    rnorm = [float(np.linalg.norm(r[s])) if s.stop > s.start else 1.0 for s in seg]
    dd, rd = torch.from_numpy(d).cuda(), torch.from_numpy(r).cuda()
    t = net.step(dd, rd, off, theta, sigma, rnorm).cpu().numpy()
    for k, s in enumerate(seg):
        if s.stop == s.start:
            continue
        ref = omlp.mlp_step(p.astype(np.float64), width, d[s], r[s], theta[k])
        assert np.linalg.norm(t[s] - ref) <= 1e-5 * np.linalg.norm(ref), k
        one = net.step(dd[s].contiguous(), rd[s].contiguous(), [0, s.stop - s.start], theta[k:k + 1], sigma[k:k + 1],
                       rnorm[k:k + 1]).cpu().numpy()
        assert np.array_equal(t[s], one), k
    net.free()
