"""Performance cases of the two-site DMRG library, through its Python entry points.

A case is one call that a DMRG program makes again and again: H_eff psi of a
plan (`hpsi.Plan.apply`), a Davidson solve on a plan (`Plan.davidson`), the
renormalization of a block (`hpsi.Renorm.apply`), the learned correction of
one Davidson iteration (`precond.MLP.step`) and the gradient of one training
batch (`MLP.loss_grad`).  Problems, plans, truncation matrices and networks
are in hand before the call, as in a program that keeps them over a solve.

The block operators of a random problem are drawn once per shape; another
seed changes the signs of all basis states and the scale of the integrals,
which gives other operators with the same symmetries.
"""
import math

import numpy as np
import torch

from paper_2309_16724_amd import binding as B
from paper_2309_16724_amd.hpsi import Plan, Renorm
from paper_2309_16724_amd.precond import MLP
from paper_2309_16724_amd.synth.mlp_inputs import mlp_batch, mlp_params, param_count
from paper_2309_16724_amd.synth.problem import BlockData, Problem, exact_problem, random_problem, random_vector

DEVICE = "cuda:0"
FLOOR = 1e-2            # the solver's default denominator floor


def _hpsi(n_orb, D, **kw):
    case = {"kind": "hpsi", "blocks": "random", "n_orb": n_orb, "n_elec": n_orb, "two_s": n_orb % 2, "D": D,
            "narrow": False, "precision": "fp64", "n_slices": 0, "graph": False, "workspace_gib": 16}
    case.update(kw)
    return case


def _renorm(n_orb, D, **kw):
    case = {"kind": "renorm", "blocks": "random", "n_orb": n_orb, "n_elec": n_orb, "two_s": n_orb % 2, "D": D,
            "narrow": False, "side": "left", "all_pairs": False}
    case.update(kw)
    return case


def listed():
    return [
        # the first and last bonds of a sweep: few small sectors, launches count
        dict(_hpsi(8, 0, blocks="exact", graph=True), name="hpsi_L8_exact"),
        # a small active space, called without graphs (new plan per bond)
        dict(_hpsi(16, 128), name="hpsi_L16_D128"),
        # the middle bond of a 24-orbital space, graph replays as in a long solve
        dict(_hpsi(24, 512, graph=True), name="hpsi_L24_D512"),
        # the same in split-BF16 arithmetic (five slices meet 1e-10)
        dict(_hpsi(24, 512, graph=True, precision="split", n_slices=5), name="hpsi_L24_D512_split"),
        # the large runs: 54 orbitals, large ragged sectors
        dict(_hpsi(54, 1024, narrow=True), name="hpsi_L54_D1024"),
        dict(_hpsi(54, 768, narrow=True, precision="split", n_slices=5), name="hpsi_L54_D768_split"),
        # independent problems of mixed size and spin in one plan
        dict(_hpsi(0, 512, kind="batch", graph=True, problems=8, first_seed=1000), name="hpsi_batch8"),
        # a solve stopped after 30 iterations (one restart), as sweeps do it
        dict(_hpsi(24, 512, kind="davidson", max_iter=30), name="davidson_L24_D512"),
        # the block updates of both sweep directions
        dict(_renorm(54, 512, narrow=True), name="renorm_left_L54_D512"),
        dict(_renorm(24, 512, side="right"), name="renorm_right_L24_D512"),
        # the learned preconditioner inside a solve of the L=24 problem
        {"name": "mlp_step_224k", "kind": "mlp_step", "n": 224112, "segments": 1, "width": 256},
        # and one batch of its training
        {"name": "mlp_grad_4096", "kind": "mlp_grad", "n": 4096, "width": 256},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_space(rng):
    """(orbitals, 2S, D, narrow) over the range of the listed H psi cases."""
    if rng.random() < 0.25:
        n_orb = rng.randrange(36, 55)
        return n_orb, n_orb % 2, _log_int(rng, 96, 640), True
    n_orb = rng.randrange(10, 33)
    return n_orb, n_orb % 2 + rng.choice((0, 0, 2)), _log_int(rng, 16, 640), False


def draw(rng):
    kind = rng.choice(("hpsi", "hpsi", "hpsi", "split", "split", "batch", "davidson", "renorm", "renorm", "mlp_step",
                       "mlp_grad", "exact"))
    n_orb, two_s, D, narrow = _draw_space(rng)
    space = {"two_s": two_s, "narrow": narrow}
    if kind == "exact":
        n = rng.choice((5, 6, 7, 8))
        return _hpsi(n, 0, blocks="exact", two_s=n % 2 + rng.choice((0, 2)), graph=rng.random() < 0.5)
    if kind == "hpsi":
        return _hpsi(n_orb, D, graph=rng.random() < 0.5, **space)
    if kind == "split":
        return _hpsi(n_orb, D, graph=rng.random() < 0.5, precision="split", n_slices=rng.choice((4, 5, 5, 5, 6)), **space)
    if kind == "batch":
        return _hpsi(0, _log_int(rng, 130, 512), kind="batch", graph=rng.random() < 0.5, problems=rng.randrange(2, 9),
                     first_seed=rng.randrange(1000, 2000))
    if kind == "davidson":
        return _hpsi(n_orb, min(max(D, 64), 512), kind="davidson", max_iter=rng.randrange(5, 31), **space)
    if kind == "renorm":
        side = rng.choice(("left", "right"))
        return _renorm(n_orb, min(D, 512), side=side, all_pairs=side == "left" and not narrow and rng.random() < 0.3,
                       **space)
    if kind == "mlp_step":
        n = _log_int(rng, 1000, 2000000)
        return {"kind": "mlp_step", "n": n, "segments": rng.choice((1, 1, 1, 7)), "width": rng.choice((64, 128, 256, 256))}
    return {"kind": "mlp_grad", "n": _log_int(rng, 100, 65536), "width": rng.choice((32, 64, 128, 256, 256))}


# ------------------------------------------------------------------ inputs
_templates = {}


def _template(*key):
    """The random problem of one shape (the last two shapes are kept)."""
    if key not in _templates:
        while len(_templates) > 1:
            _templates.pop(next(iter(_templates)))
        n_orb, n_elec, two_s, seed, D, narrow, all_pairs = key
        shape = dict(spin_ratio=0.45, sigma_frac=0.03) if narrow else {}
        _templates[key] = random_problem(n_orb, n_elec, two_s, seed, D, all_pairs=all_pairs, **shape)
    return _templates[key]


def _resigned(block, rng):
    """The block in a basis whose states have random signs."""
    sign = [rng.choice((-1.0, 1.0), dim) for (_, _, dim) in block.sectors]
    out = BlockData(block.role, block.n_orb, block.p, block.sectors, all_pairs=getattr(block, "all_pairs", False))
    out.records, out.data = block.records, np.empty_like(block.data)
    for (_, row, col, off, npos) in block.records:
        shape = (npos, len(sign[col]), len(sign[row]))
        size = shape[0] * shape[1] * shape[2]
        np.multiply(block.data[off:off + size].reshape(shape), sign[col][:, None] * sign[row][None, :],
                    out=out.data[off:off + size].reshape(shape))
    return out


def _random(seed, *key):
    base, rng = _template(*key), np.random.default_rng(seed)
    scale = rng.uniform(0.8, 1.2)
    return Problem(base.n_orb, base.n_elec, base.two_s, base.p, scale * base.h, scale * base.eri,
                   _resigned(base.left, rng), _resigned(base.right, rng), "random")


_batches = {}


def _batch_keys(case):
    """Shapes of a batch: 16 to 32 orbitals, D from 128 up to the case's, singlets and triplets."""
    rng = np.random.default_rng(case["first_seed"])
    keys = []
    for k in range(case["problems"]):
        n_orb = int(rng.integers(16, 33))
        D = int(rng.integers(128, case["D"] + 1))
        keys.append((n_orb, n_orb, n_orb % 2 + 2 * int(rng.integers(0, 2)), case["first_seed"] + k, D, False, False))
    return keys


def _batch(case, seed):
    keys = tuple(_batch_keys(case))
    if keys not in _batches:
        _batches.clear()
        _batches[keys] = [random_problem(*key[:5]) for key in keys]
    rng = np.random.default_rng(seed)
    return [Problem(p.n_orb, p.n_elec, p.two_s, p.p, p.h, p.eri, _resigned(p.left, rng), _resigned(p.right, rng),
                    "random") for p in _batches[keys]]


def _problem(case, seed):
    if case["blocks"] == "exact":
        return exact_problem(case["n_orb"], case["n_elec"], case["two_s"], seed)
    return _random(seed, case["n_orb"], case["n_elec"], case["two_s"], 1, case["D"], case["narrow"],
                   case.get("all_pairs", False))


def _keep(prob, right, seed):
    """A quarter of every product sector's states, an orthonormal basis each."""
    rng = np.random.default_rng(seed)
    return [(n, s2, np.linalg.qr(rng.standard_normal((rows, max(1, rows // 4))))[0])
            for (n, s2, rows) in B.renorm_product(prob, right=right)[0]]


def _step_inputs(case, seed):
    """diag, residual, segment offsets and per-segment scalars of a Davidson
    iteration; network parameters of a trained network's size."""
    n, k = case["n"], case["segments"]
    rng = np.random.default_rng(seed)
    off = np.linspace(0, n, k + 1).astype(np.int64)
    diag = rng.standard_normal(n) * 3.0
    r = rng.standard_normal(n) * np.exp(rng.standard_normal(n)) * 1e-4
    theta, sigma, rnorm = [], [], []
    for a, b in zip(off[:-1], off[1:]):
        th = diag[a:b].min() - 0.5
        theta.append(float(th))
        sigma.append(float(np.sqrt(np.mean((diag[a:b] - th) ** 2))))
        rnorm.append(float(np.linalg.norm(r[a:b])))
    return diag, r, off, theta, sigma, rnorm, mlp_params(B.DMRG_MLP_IN, case["width"], seed + 1)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "mlp_step":
        diag, r, off, theta, sigma, rnorm, params = _step_inputs(case, seed)
        net = MLP(case["width"], seed=0)
        net.set_params(params)
        return {"kind": kind, "net": net, "diag": torch.from_numpy(diag).to(DEVICE), "r": torch.from_numpy(r).to(DEVICE),
                "scalars": (off, theta, sigma, rnorm)}
    if kind == "mlp_grad":
        net = MLP(case["width"], seed=0)
        net.set_params(mlp_params(B.DMRG_MLP_IN, case["width"], seed + 1))
        rows = [torch.from_numpy(v).to(DEVICE) for v in mlp_batch(case["n"], B.DMRG_MLP_IN, seed)]
        return {"kind": kind, "net": net, "rows": rows}
    if kind == "renorm":
        prob, right = _problem(case, seed), case["side"] == "right"
        return {"kind": kind, "renorm": Renorm(prob, _keep(prob, right, seed), device=DEVICE, right=right)}
    probs = _batch(case, seed) if kind == "batch" else _problem(case, seed)
    plan = Plan(probs, device=DEVICE, precision=B.DMRG_SPLIT_BF16 if case["precision"] == "split" else B.DMRG_FP64,
                n_slices=case["n_slices"], workspace_bytes=case["workspace_gib"] << 30,
                flags=B.DMRG_PLAN_GRAPH if case["graph"] else 0)
    psi = torch.from_numpy(random_vector(plan.size, seed)).to(DEVICE)
    return {"kind": kind, "plan": plan, "psi": psi, "out": torch.empty_like(psi), "max_iter": case.get("max_iter")}


def run(state):
    kind = state["kind"]
    if kind == "mlp_step":
        return state["net"].step(state["diag"], state["r"], *state["scalars"], floor=FLOOR)
    if kind == "mlp_grad":
        return state["net"].loss_grad(*state["rows"])
    if kind == "renorm":
        return state["renorm"].apply()
    if kind == "davidson":
        energy, psi, _ = state["plan"].davidson(state["psi"], tol=1e-12, max_iter=state["max_iter"], check=False)
        return energy, psi
    return state["plan"].apply(state["psi"], state["out"])


# -------------------------------------------------------------- least work
def work(case):
    kind = case["kind"]
    if kind in ("mlp_step", "mlp_grad"):
        w = case["width"]
        macs = B.DMRG_MLP_IN * w + w * w + w
        if kind == "mlp_step":
            return {"bytes": 24.0 * case["n"], "flops": 2.0 * macs * case["n"]}
        size = 4.0 * param_count(B.DMRG_MLP_IN, w)
        return {"bytes": 16.0 * case["n"] + 2 * size, "flops": 6.0 * macs * case["n"]}
    if kind == "renorm":
        right = case["side"] == "right"
        prob = _problem(case, 0)
        keep = _keep(prob, right, 0)
        _, st = B.debug_renorm_host(prob, keep, execute=False, right=right)
        block = prob.right if right else prob.left
        return {"bytes": 8.0 * (block.data.size + sum(u.size for _, _, u in keep) + st["out_elems"]),
                "flops": st["flops1"] + st["flops2"]}
    # operators and psi read once, H psi written once; 2mnk of the products that the operator table asks for
    st = prepare(case, 0)["plan"].stats()
    probs = _batch(case, 0) if kind == "batch" else [_problem(case, 0)]
    nbytes = 8.0 * (sum(p.left.data.size + p.right.data.size for p in probs) + 2 * st["psi_len"])
    if kind == "davidson":
        # per iteration the basis and its products are read (m_max 24, about 12 columns on average)
        return {"bytes": case["max_iter"] * (nbytes + 8.0 * st["psi_len"] * 4 * 12),
                "flops": case["max_iter"] * st["flops"]}
    return {"bytes": nbytes, "flops": st["flops"]}


# ------------------------------------------------- results in 64 bits
_SITE_N, _SITE_S = (0, 1, 2), (0, 1, 0)
_SITE_FOCK = ({0: 0}, {1: 1, -1: 2}, {0: 3})    # Fock state of a site multiplet by 2M


def _blocks(prob):
    """(left sector, l, 2S_Ll, r, right sector, 2S_rR) of the wavefunction blocks, in storage order."""
    for a, (na, sa, da) in enumerate(prob.left.sectors):
        for l in range(3):
            for s1 in range(abs(sa - _SITE_S[l]), sa + _SITE_S[l] + 1, 2):
                for r in range(3):
                    for b, (nb, sb, db) in enumerate(prob.right.sectors):
                        if na + _SITE_N[l] + _SITE_N[r] + nb != prob.n_elec:
                            continue
                        for s2 in range(abs(sb - _SITE_S[r]), sb + _SITE_S[r] + 1, 2):
                            if abs(s1 - s2) <= prob.two_s <= s1 + s2 and (s1 + s2 + prob.two_s) % 2 == 0:
                                yield a, l, s1, r, b, s2


def _psi_size(prob):
    return sum(prob.left.sectors[a][2] * prob.right.sectors[b][2] for a, _, _, _, b, _ in _blocks(prob))


def _cg(j1, m1, j2, m2, J, M):
    """Clebsch-Gordan coefficient by Racah's formula, all arguments doubled."""
    if m1 + m2 != M or abs(M) > J or not abs(j1 - j2) <= J <= j1 + j2:
        return 0.0
    f = [math.factorial(x // 2) for x in (j1 + j2 - J, j1 - j2 + J, j2 - j1 + J, j1 + m1, j1 - m1, j2 + m2, j2 - m2,
                                          J + M, J - M)]
    total = 0.0
    for k in range((j1 + j2 - J) // 2 + 1):
        d = [k, (j1 + j2 - J) // 2 - k, (j1 - m1) // 2 - k, (j2 + m2) // 2 - k, (J - j2 + m1) // 2 + k,
             (J - j1 - m2) // 2 + k]
        if min(d) >= 0:
            total += (-1) ** k / math.prod(math.factorial(x) for x in d)
    return math.sqrt((J + 1) * math.prod(f) / math.factorial((j1 + j2 + J) // 2 + 1)) * total


def _product_states(prob):
    """((slice of psi, d_L, d_R), coefficient, left basis, left site state, right site state, right basis) of every
    product state |L M_L>|l>|r>|R M_R> in the coupled states at M = S."""
    off = 0
    for a, l, s1, r, b, s2 in _blocks(prob):
        sa, da = prob.left.sectors[a][1:]
        sb, db = prob.right.sectors[b][1:]
        where = (slice(off, off + da * db), da, db)
        off += da * db
        for m1 in range(-s1, s1 + 1, 2):
            c0 = _cg(s1, m1, s2, prob.two_s - m1, prob.two_s, prob.two_s) if abs(prob.two_s - m1) <= s2 else 0.0
            for ml, fl in _SITE_FOCK[l].items():
                for mr, fr in _SITE_FOCK[r].items():
                    ma, mb = m1 - ml, prob.two_s - m1 - mr
                    if c0 == 0.0 or abs(ma) > sa or abs(mb) > sb:
                        continue
                    c = c0 * _cg(sa, ma, _SITE_S[l], ml, s1, m1) * _cg(_SITE_S[r], mr, sb, mb, s2, prob.two_s - m1)
                    yield where, c, prob.left.basis[a][(sa - ma) // 2], fl, fr, prob.right.basis[b][(sb - mb) // 2]


def _fock_hamiltonian(prob, x):
    """H x in the Fock space of all orbitals (orbital j: bits 2j and 2j + 1)."""
    n, states = prob.n_orb, np.arange(x.size)
    parity = np.array([bin(s).count("1") & 1 for s in range(x.size)], dtype=np.int8)

    def excite(i, j, v):                      # E_ij v = sum over spins of a+_i a_j v
        out = np.zeros_like(v)
        for spin in (0, 1):
            p, q = 1 << (2 * i + spin), 1 << (2 * j + spin)
            src = states[(states & q) != 0]
            mid = src ^ q
            ok = (mid & p) == 0
            src, mid = src[ok], mid[ok]
            sign = 1.0 - 2.0 * (parity[mid & (q - 1)] ^ parity[mid & (p - 1)])
            out[mid | p] += sign * v[src]
        return out

    one = prob.h - 0.5 * np.einsum("ijjl->il", prob.eri)
    pairs = [(k, l) for k in range(n) for l in range(n)]
    first = np.stack([excite(k, l, x) for k, l in pairs])
    second = 0.5 * prob.eri.reshape(n * n, n * n) @ first + one.reshape(-1, 1) * x[None, :]
    return sum(excite(i, j, second[q]) for q, (i, j) in enumerate(pairs))


def _exact_hpsi(case, seed):
    prob = _problem(case, seed)
    psi = random_vector(_psi_size(prob), seed)
    dl, dr = 4 ** prob.p, 4 ** (prob.n_orb - prob.p - 2)
    full = np.zeros((dr, 4, 4, dl))
    states = list(_product_states(prob))
    for (where, da, db), c, bl, fl, fr, br in states:
        full[:, fr, fl, :] += c * (br @ psi[where].reshape(db, da) @ bl.T)
    full = _fock_hamiltonian(prob, full.reshape(-1)).reshape(full.shape)
    out = np.zeros_like(psi)
    for (where, da, db), c, bl, fl, fr, br in states:
        out[where] += c * (br.T @ full[:, fr, fl, :] @ bl).reshape(-1)
    return out


def _network(params, width, x):
    """Layers of the network in 64 bits: pre-activations z1, z2 and output g."""
    p, at, parts = params.astype(np.float64), 0, []
    for size in (B.DMRG_MLP_IN * width, width, width * width, width, width, 1):
        parts.append(p[at:at + size])
        at += size
    w1, b1, w2, b2, w3, b3 = parts
    w1, w2 = w1.reshape(-1, width), w2.reshape(width, width)
    z1 = x @ w1 + b1
    z2 = np.maximum(z1, 0.0) @ w2 + b2
    return (w1, w2, w3), z1, z2, np.maximum(z2, 0.0) @ w3 + b3[0]


def _exact_step(case, seed):
    diag, r, off, theta, sigma, rnorm, params = _step_inputs(case, seed)
    out = np.empty_like(r)
    for k in range(case["segments"]):
        for a in range(int(off[k]), int(off[k + 1]), 65536):
            b = min(a + 65536, int(off[k + 1]))
            den = diag[a:b] - theta[k]
            small = np.abs(den) < FLOOR * sigma[k]
            td = -r[a:b] / np.where(small, np.copysign(FLOOR * sigma[k], den), den)
            x = np.stack([np.arcsinh(den / sigma[k]), np.full(b - a, math.log10(rnorm[k]) / 8.0)], axis=1)
            out[a:b] = td * (1.0 + _network(params, case["width"], x)[3])
    return out


def _exact_grad(case, seed):
    x, a, b = (v.astype(np.float64) for v in mlp_batch(case["n"], B.DMRG_MLP_IN, seed))
    (_, w2, w3), z1, z2, g = _network(mlp_params(B.DMRG_MLP_IN, case["width"], seed + 1), case["width"], x)
    e = a * (1.0 + g) - b
    dg = 2.0 * e * a / len(a)
    dz2 = np.where(z2 > 0.0, dg[:, None] * w3, 0.0)
    dz1 = np.where(z1 > 0.0, dz2 @ w2.T, 0.0)
    grad = [x.T @ dz1, dz1.sum(0), np.maximum(z1, 0.0).T @ dz2, dz2.sum(0), dg @ np.maximum(z2, 0.0), dg.sum()]
    return float(np.mean(e * e)), np.concatenate([np.ravel(v) for v in grad])


def exact(case, seed):
    """H psi from the determinant space where the blocks span theirs; the
    network's results.  Truncated random blocks have no such space: their
    products would have to be expanded in all spin projections, which takes
    minutes at these sizes."""
    if case["kind"] == "hpsi" and case["blocks"] == "exact":
        return _exact_hpsi(case, seed)
    if case["kind"] == "mlp_step":
        return _exact_step(case, seed) if case["n"] * case["width"] ** 2 <= 1.5e11 else None
    if case["kind"] == "mlp_grad":
        return _exact_grad(case, seed)
    return None
