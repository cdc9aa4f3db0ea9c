"""H.psi plans, density matrices and renormalizations whose sectors reach the
work-group tiles (64 x 64 from 48 states on, 128 x 128 from 64 x 96 on), both
sides, against the oracle.  That the sizes reach both kinds is asserted."""
import ctypes

import numpy as np
import pytest

from oracle.layout import psi_blocks
from oracle.renorm import product_sectors, product_sectors_right, renormalize, renormalize_right
from oracle.truncate import sector_matrices, sector_matrices_right
from paper_2309_16724_amd import binding as B
from paper_2309_16724_amd.synth import catalogue as cat
from paper_2309_16724_amd.synth.problem import random_problem, random_vector

pytestmark = pytest.mark.gpu


def _kinds(sizes):
    return {int(k) for m in sizes for n in sizes for k in B.debug_f64_cells(m, n)[:, 2]}


def _launches(plan, code):
    n = ctypes.c_int64()
    B.check(plan.lib.dmrg_get_profile(plan.handle, code, ctypes.byref(n), None, None), plan.lib)
    return n.value


@pytest.mark.parametrize("D,Dr,codes", [(340, 700, (11, 12, 31, 32)), (620, 150, (11, 12, 31, 32)),
                                        (160, 640, (11, 31, 32))])
def test_batches_use_work_group_tiles(D, Dr, codes):
    """Sixteen copies of a problem give both stages enough outputs for work-group
    tiles (their launches are counted: 1 for 64 x 64, 3 for 128 x 128, then the
    stage; the last shape has no second-stage output between them); each copy, with a vector of its own, against the
    oracle.  FP64 sums in another order: 1e-12 of the largest element."""
    import torch
    from oracle.hpsi import HEff
    from paper_2309_16724_amd.hpsi import Plan
    prob = random_problem(6, 6, 0, 5, D=D, D_right=Dr, cap=False)
    he = HEff(prob)
    x = np.random.default_rng(3).standard_normal((16, he.size))
    plan = Plan([prob] * 16)
    B.check(plan.lib.dmrg_set_profiling(plan.handle, 1), plan.lib)
    y = plan.apply(torch.from_numpy(x.reshape(-1)).cuda()).cpu().numpy().reshape(x.shape)
    counts = {code: _launches(plan, code) for code in codes}
    plan.free()
    assert all(counts.values()), counts
    for k in (0, 5, 15):
        ref = he.apply(x[k])
        assert np.abs(y[k] - ref).max() <= 1e-12 * np.abs(ref).max(), k


@pytest.mark.parametrize("opts", [dict(workspace_bytes=2 << 20), dict(workspace_bytes=8 << 20), dict(kpart=16384)])
def test_plans_of_few_tiles_match_oracle(opts):
    import torch
    from oracle.hpsi import HEff
    from paper_2309_16724_amd.hpsi import Plan
    prob = random_problem(6, 6, 0, 5, D=340, D_right=300, cap=False)
    he = HEff(prob)
    x = np.random.default_rng(4).standard_normal(he.size)
    ref = he.apply(x)
    plan = Plan(prob, **opts)
    y = plan.apply(torch.from_numpy(x).cuda()).cpu().numpy()
    plan.free()
    assert np.abs(y - ref).max() <= 1e-12 * np.abs(ref).max()


@pytest.mark.parametrize("right", [False, True])
@pytest.mark.parametrize("D,sizes,kinds", [(310, {47, 48, 131}, {8, 32}), (420, {64, 65, 178}, {8, 32}),
                                           (630, {96, 97, 267}, {32})])
def test_density_matrices_of_large_sectors(right, D, sizes, kinds):
    """The kept vectors U and the weights against the oracle's rho: rho U = U
    diag(w) and their sum.  Elements of rho are sums of at most a thousand FP64
    products and the eigensolver's backward error is of the order of rows x
    2^-53: 1e-12 of the trace."""
    import torch
    from paper_2309_16724_amd.hpsi import keep_host, truncate
    assert torch.cuda.is_available()
    prob = random_problem(6, 6, 0, 5, D=200 if right else D, D_right=D if right else 200, cap=False)
    dims = {s[2] for s in (prob.right if right else prob.left).sectors}
    assert sizes <= dims and kinds <= _kinds(dims)
    size = psi_blocks(prob.left.sectors, prob.right.sectors, prob.n_elec, prob.two_s)[1]
    psi = random_vector(size, 6)
    keep, u, (kept, trace) = truncate(prob, torch.from_numpy(psi).cuda(), 400, 0.0, right=right)
    mats = (sector_matrices_right if right else sector_matrices)(prob, psi)
    assert abs(trace - 1.0) <= 1e-12 and sum(k[2] for k in keep) == 400
    total = 0.0
    for n, s2, U in keep_host(prob, keep, u, right=right):
        rho = mats[(n, s2)][0] @ mats[(n, s2)][0].T
        w = np.einsum("ij,ij->j", U, rho @ U)
        assert np.abs(rho @ U - U * w).max() <= 1e-12, (n, s2)
        assert np.abs(U.T @ U - np.eye(U.shape[1])).max() <= 1e-12, (n, s2)
        total += w.sum()
    every = np.sort(np.concatenate([np.linalg.eigvalsh(m @ m.T) for m, _ in mats.values()]))
    assert abs(total - every[-400:].sum()) <= 1e-12
    assert abs(kept - total) <= 1e-12


@pytest.mark.parametrize("right", [False, True])
def test_renormalization_of_large_sectors(right):
    """Sums of at most a few hundred FP64 products per stage: 1e-12 of the
    family's largest element, as in the other tests of the renormalization."""
    from paper_2309_16724_amd.hpsi import Renorm
    prob = random_problem(6, 6, 0, 5, D=310, D_right=310, cap=False)
    secs = product_sectors_right(prob.right.sectors) if right else product_sectors(prob.left.sectors)
    rng = np.random.default_rng(7)
    keep = [(n, s2, np.linalg.qr(rng.standard_normal((rows, max(1, 2 * rows // 3))))[0]) for n, s2, rows, _ in secs]
    kinds = _kinds({k[2].shape[1] for k in keep})
    assert {8, 32} <= kinds and max(k[2].shape[1] for k in keep) > 128
    r = Renorm(prob, keep, right=right)
    r.apply()
    got = r.block()
    r.free()
    families = (cat.H, cat.C)
    want = (renormalize_right if right else renormalize)(prob, keep, families=families)
    for fam in families:
        keys = [(row, col) for f, row, col, _, _ in want.records if f == fam]
        scale = max(np.abs(want.block(fam, *k)).max() for k in keys)
        for k in keys:
            assert np.abs(got.block(fam, *k) - want.block(fam, *k)).max() <= 1e-12 * max(1.0, scale), (fam, k)
