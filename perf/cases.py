"""The work that performance is measured on: calls a user of the solver makes,
through its public entry points, with inputs drawn from a seed.

A case is a dict of plain values.  ``listed()`` gives the standing cases,
``draw(rng)`` one more of the same ranges, ``prepare(case, seed)`` what a
program holds before the call, ``run(state)`` one pass, ``work(case)`` the
bytes and operations of a pass that no implementation avoids, and
``exact(case, seed)`` the same outputs from plain FP64 torch and NumPy.

Kinds of call:
  solve    one solve (rdm.solve), per-column or block method, stored basis or
           two passes, with the workspace kept between calls
  batch    solve_batch over instances of different sizes
  grid     scans.entropy_grid: an entropy phase plot, Hamiltonians included
  serve    requests submitted to a running Server and waited for
  product  product_trace, ln Z* from rank-one samples
  ground   ground_state, the low-temperature limit
  apply    one product with H on a block of vectors
Operator families: ``chain`` (random nearest-neighbour XXZ, z-field), ``lr``
(long-range XX + ZZ, x-field), ``lrxxz`` (long-range XXZ, x-field), ``sparse``
(random XXZ on 2N edges), ``tfim`` (ZZ chain, x-field), ``xy`` (power-law XY,
z-field).
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2204_08147_amd as rdm
from paper_2204_08147_amd import scans

OUTPUTS = ("rho", "h_star", "log_z", "entropy", "log_z_t", "log_z_b")


def listed():
    return [
        # the smallest call: one ten-spin chain at one temperature, where
        # launches and host work count
        dict(name="small_chain_fp64", kind="solve", family="chain", n_s=1, n_b=9, n_v=4, k=30, n_beta=1,
             beta=1.0, precision="fp64", mode="auto", method="per_column"),
        # the headline solve: long-range chain, 64 start columns, four
        # temperatures, stored basis
        dict(name="lr20_mixed", kind="solve", family="lr", n_s=2, n_b=18, n_v=16, k=60, n_beta=4, beta=0.5,
             precision="mixed", mode="auto", method="per_column"),
        # the same physics in full FP64, one size down
        dict(name="lr18_fp64", kind="solve", family="lr", n_s=2, n_b=16, n_v=16, k=60, n_beta=4, beta=0.5,
             precision="fp64", mode="auto", method="per_column"),
        # a large XXZ instance whose basis is not stored: two passes
        dict(name="lrxxz23_two_pass", kind="solve", family="lrxxz", n_s=3, n_b=20, n_v=4, k=80, n_beta=1,
             beta=2.0, precision="mixed", mode="two_pass", method="per_column"),
        # the paper's own block Lanczos estimator, odd number of vectors
        dict(name="block19_mixed", kind="solve", family="lr", n_s=2, n_b=17, n_v=7, k=40, n_beta=2, beta=0.5,
             precision="mixed", mode="auto", method="block"),
        # a parameter study: sparse random XXZ instances of many sizes at once
        dict(name="batch_sparse", kind="batch", family="sparse", n_lo=12, n_hi=22, count=16, n_v=8, k=50,
             precision="mixed"),
        # an entropy phase plot at the paper's size
        dict(name="entropy_grid16", kind="grid", family="xy", n_s=2, n_b=14, count=3, n_v=100, k=60, n_beta=8,
             beta=0.1, precision="mixed"),
        # a burst of transverse-field chains at the serving engine
        dict(name="serve_tfim", kind="serve", family="tfim", n_lo=14, n_hi=21, count=12, n_v=8, k=60,
             precision="mixed"),
        # partition function only
        dict(name="product20_mixed", kind="product", family="lr", n_s=2, n_b=18, n_v=16, k=60, n_beta=4,
             beta=0.5, precision="mixed"),
        # the T = 0 limit of a chain
        dict(name="ground16_fp64", kind="ground", family="lrxxz", n_s=2, n_b=14, n_v=4, k=100,
             precision="fp64"),
        # single products of a caller's own Krylov method: sparse operator,
        # odd column count, FP64; and dense operator, 21 spins, FP32
        dict(name="apply_sparse20_fp64", kind="apply", family="sparse", n_s=2, n_b=18, n_cols=13,
             precision="fp64"),
        dict(name="apply_lr21_mixed", kind="apply", family="lr", n_s=2, n_b=19, n_cols=24, precision="mixed"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "solve", "batch", "grid", "serve", "product", "ground", "apply",
                       "apply"])
    prec = rng.choice(["mixed", "fp64"])
    if kind == "solve":
        family = rng.choice(["chain", "lr", "lrxxz", "sparse", "tfim"])
        n = rng.randint(6, 21)
        n_s = rng.randint(1, 3)
        return dict(kind=kind, family=family, n_s=n_s, n_b=n - n_s, n_v=_log_int(rng, 1, 16 if n <= 19 else 6),
                    k=min(rng.randint(15, 60), 1 << (n - 2)), n_beta=rng.randint(1, 5),
                    beta=round(10.0 ** rng.uniform(-1.0, 0.0), 3), precision=prec,
                    mode=rng.choice(["auto", "auto", "two_pass"]),
                    method=rng.choice(["per_column", "per_column", "per_column", "block"]))
    if kind == "batch":
        hi = rng.randint(13, 21)
        return dict(kind=kind, family=rng.choice(["sparse", "chain"]), n_lo=rng.randint(8, 12), n_hi=hi,
                    count=rng.randint(2, 24), n_v=rng.randint(1, 8), k=rng.randint(20, 50), precision=prec)
    if kind == "grid":
        n_b = rng.randint(8, 14)
        return dict(kind=kind, family="xy", n_s=rng.randint(1, 2), n_b=n_b, count=rng.randint(1, 3),
                    n_v=_log_int(rng, 8, 100), k=rng.randint(20, 60), n_beta=rng.randint(1, 8), beta=0.1,
                    precision=prec)
    if kind == "serve":
        return dict(kind=kind, family="tfim", n_lo=rng.randint(8, 14), n_hi=rng.randint(15, 21),
                    count=rng.randint(1, 12), n_v=rng.randint(1, 8), k=rng.randint(20, 60), precision="mixed")
    if kind == "product":
        return dict(kind=kind, family=rng.choice(["lr", "sparse"]), n_s=rng.randint(1, 3), n_b=rng.randint(8, 18),
                    n_v=_log_int(rng, 1, 32), k=rng.randint(20, 60), n_beta=rng.randint(1, 4), beta=0.5,
                    precision=prec)
    if kind == "ground":
        return dict(kind=kind, family="lrxxz", n_s=rng.randint(1, 3), n_b=rng.randint(10, 15),
                    n_v=rng.randint(1, 6), k=rng.randint(90, 120), precision="fp64")
    return dict(kind="apply", family=rng.choice(["chain", "lr", "lrxxz", "sparse", "tfim"]), n_s=2,
                n_b=rng.randint(8, 20), n_cols=_log_int(rng, 1, 40), precision=prec)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _instance(family, n_s, n_b, seed, betas, n_v, k):
    """One seeded instance: couplings (i, j, jx, jy, jz) with i < j, fields."""
    n = n_s + n_b
    rng = np.random.default_rng(seed)
    hx, hz, cps = np.zeros(n), np.zeros(n), []
    if family == "chain":
        for i in range(n - 1):
            jxy, jz = (1.0, 1.0) if i == n_s - 1 else rng.uniform(-1.0, 1.0, size=2)
            cps.append((i, i + 1, float(jxy), float(jxy), float(jz)))
        hz[:] = 0.25
    elif family == "lr":
        hx[:] = rng.uniform(0.25, 0.75)
        cps = [(i, j, float(j - i) ** -1.5, 0.0, float(j - i) ** -1.5) for i in range(n) for j in range(i + 1, n)]
    elif family == "lrxxz":
        hx[:] = rng.uniform(0.4, 0.6)
        for i in range(n):
            for j in range(i + 1, n):
                c = float(j - i) ** -1.2
                cps.append((i, j, c, c, 0.8 * c))
    elif family == "sparse":
        pairs = [(i, j) for i in range(n) for j in range(i + 1, n)]
        for p in sorted(rng.choice(len(pairs), size=min(2 * n, len(pairs)), replace=False).tolist()):
            jxy, jz = rng.uniform(-1.0, 1.0, size=2)
            cps.append((*pairs[p], float(jxy), float(jxy), float(jz)))
    elif family == "tfim":
        hx[:] = 0.5 * rng.uniform(0.2, 2.0)
        cps = [(i, i + 1, 0.0, 0.0, 1.0) for i in range(n - 1)]
    else:
        raise ValueError(family)
    return SimpleNamespace(n_s=n_s, n_b=n_b, couplings=cps, hx=hx, hz=hz, betas=np.asarray(betas, float), n_v=n_v,
                           k=k, seed=int(rng.integers(1, 2 ** 62)))


def _xy(case, h, seed):
    """Isotropic power-law XY chain, z-field of strength h."""
    n = case["n_s"] + case["n_b"]
    cps = [(i, j, float(j - i) ** -1.5, float(j - i) ** -1.5, 0.0) for i in range(n) for j in range(i + 1, n)]
    return SimpleNamespace(n_s=case["n_s"], n_b=case["n_b"], couplings=cps, hx=np.zeros(n), hz=np.full(n, h / 2.0),
                           betas=_betas(case), n_v=case["n_v"], k=case["k"], seed=seed)


def _betas(case):
    return case["beta"] * 2.0 ** np.arange(case["n_beta"])


def _instances(case, seed):
    """The instances of a case, in order."""
    kind = case["kind"]
    if kind in ("solve", "product"):
        return [_instance(case["family"], case["n_s"], case["n_b"], seed, _betas(case), case["n_v"], case["k"])]
    if kind == "ground":
        return [_instance(case["family"], case["n_s"], case["n_b"], seed, [1.0], case["n_v"], case["k"])]
    if kind == "apply":
        return [_instance(case["family"], case["n_s"], case["n_b"], seed, [1.0], 1, 1)]
    rng = np.random.default_rng(seed)
    if kind == "grid":
        fields = np.sort(rng.uniform(0.0, 2.0, size=case["count"]))
        return [_xy(case, float(h), int(rng.integers(1, 2 ** 62))) for h in fields]
    out = []
    for t in range(case["count"]):
        # sizes and system sizes are the case's own; couplings and temperatures are drawn
        n = case["n_lo"] + (t * (case["n_hi"] - case["n_lo"])) // max(case["count"] - 1, 1)
        n_s = 1 + t % (3 if kind == "batch" else 2)
        beta = 10.0 ** rng.uniform(-1.0, 1.0)
        out.append(_instance(case["family"], n_s, n - n_s, int(rng.integers(1, 2 ** 62)), [beta], case["n_v"],
                             min(case["k"], 1 << (n - n_s))))
    return out


def _block(case, seed):
    """The (dim, n_cols) block of vectors of an apply case, in its precision."""
    gen = torch.Generator(device="cuda" if torch.cuda.is_available() else "cpu").manual_seed(seed)
    dtype = torch.float64 if case["precision"] == "fp64" else torch.float32
    dim = 1 << (case["n_s"] + case["n_b"])
    x = torch.randn(dim, case["n_cols"], generator=gen, dtype=dtype, device=gen.device)
    return x / math.sqrt(dim)


def prepare(case, seed):
    insts = _instances(case, seed)
    st = SimpleNamespace(case=case, insts=insts)
    if case["kind"] == "grid":
        st.fields = [2.0 * i.hz[0] for i in insts]
        st.by_field = {f: i for f, i in zip(st.fields, insts)}
        return st
    st.hs = [rdm.Hamiltonian.from_instance(i) for i in insts]
    if case["kind"] == "solve":
        st.opts = dict(precision=case["precision"], mode=case["mode"], method=case["method"])
        nbytes = rdm.workspace_size(st.hs[0], case["n_beta"], case["n_v"], case["k"], **st.opts)
        st.ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    elif case["kind"] == "batch":
        st.items = [dict(h=h, betas=i.betas, n_v=i.n_v, k=i.k, seed=i.seed) for h, i in zip(st.hs, insts)]
    elif case["kind"] == "serve":
        st.server = rdm.Server(hbm_budget=16 << 30, precision=case["precision"])
    elif case["kind"] == "apply":
        st.x = rdm.to_panels(_block(case, seed), case["precision"])
        st.y = torch.empty_like(st.x)
    return st


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def _pick(res, keys=OUTPUTS):
    return {key: res[key] for key in keys}


def _joined(results):
    """The outputs of several solves, end to end per kind of output."""
    return {key: np.concatenate([np.ravel(r[key]) for r in results]) for key in OUTPUTS}


def run(state):
    case, kind = state.case, state.case["kind"]
    if kind == "grid":
        return scans.entropy_grid(lambda f: state.by_field[f], state.fields, precision=case["precision"])
    h, inst = state.hs[0], state.insts[0]
    if kind == "solve":
        return _pick(rdm.solve(h, inst.betas, inst.n_v, inst.k, inst.seed, workspace=state.ws, **state.opts))
    if kind == "batch":
        return _joined(rdm.solve_batch(state.items, precision=case["precision"]))
    if kind == "serve":
        tickets = [state.server.submit(hh, i.betas, i.n_v, i.k, i.seed) for hh, i in zip(state.hs, state.insts)]
        return _joined([state.server.wait(t) for t in tickets])
    if kind == "product":
        return rdm.product_trace(h, inst.betas, inst.n_v, inst.k, inst.seed, precision=case["precision"])
    if kind == "ground":
        return _pick(rdm.ground_state(h, inst.n_v, inst.k, inst.seed, precision=case["precision"]),
                     ("rho", "e_total", "e_bath", "entropy"))
    rdm.apply(h, state.x, state.y, precision=case["precision"], n_cols=case["n_cols"])
    return state.y


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def _flops_per_element(inst, part):
    """Operations per element of one product: through the hop terms (a
    multiply and an add each) or through the Walsh-Hadamard form (two
    transforms, a diagonal each way, the same again for YY), whichever is less."""
    lo = inst.n_s if part else 0
    n = inst.n_s + inst.n_b - lo
    pairs = [c for c in inst.couplings if c[0] >= lo]
    hops = sum(c[2] != 0.0 or c[3] != 0.0 for c in pairs) + int(np.count_nonzero(inst.hx[lo:]))
    yy = any(c[3] != 0.0 for c in pairs)
    return min(2 * hops + 2, (4 if yy else 2) * n + (6 if yy else 4))


def work(case):
    """A Lanczos step reads the current vectors and writes the next ones; the
    recombination reads every basis vector once (not for the block variant and
    the quadrature-only estimators).  apply: vectors in, vectors out."""
    s = 8 if case["precision"] == "fp64" else 4
    kind = case["kind"]
    byts = flops = 0
    for i in _instances(case, 0):
        if kind == "apply":
            el = (1 << (i.n_s + i.n_b)) * case["n_cols"]
            byts += 2 * el * s
            flops += el * _flops_per_element(i, 0)
            continue
        cols = i.n_v if kind in ("product", "ground") else (1 << i.n_s) * i.n_v
        el_t, el_b = (1 << (i.n_s + i.n_b)) * cols, (1 << i.n_b) * i.n_v
        reads = 2 if kind == "product" or case.get("method") == "block" else 3
        byts += i.k * s * (reads * el_t + 2 * el_b)
        flops += i.k * (el_t * (_flops_per_element(i, 0) + 8) + el_b * (_flops_per_element(i, 1) + 8))
        if reads == 3:
            nb = 1 if kind == "ground" else len(i.betas)
            flops += el_t * (2 * i.k * nb + nb * (1 << i.n_s))
    return {"bytes": byts, "flops": flops}


# ---------------------------------------------------------------------------
# the same outputs in plain FP64
# ---------------------------------------------------------------------------
_M64 = (1 << 64) - 1


def _sm64(x):
    """SplitMix64 output from state x, uint64 array (the published rule)."""
    with np.errstate(over="ignore"):
        z = x + np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        return z ^ (z >> np.uint64(31))


def _signs(seed, j, bits):
    """The +-1 entries of random vector j over 2^bits basis states."""
    key = _sm64(np.uint64(seed & _M64) ^ _sm64(np.array([j], dtype=np.uint64)))
    b = np.arange(1 << bits, dtype=np.uint64)
    bit = (_sm64(key ^ (b >> np.uint64(6))) >> (b & np.uint64(63))) & np.uint64(1)
    return 1.0 - 2.0 * bit.astype(np.float64)


class _Operator:
    """H_t (bath = False) or H_b on torch FP64 blocks of rows x columns."""

    def __init__(self, inst, bath, device):
        lo = inst.n_s if bath else 0
        n = inst.n_s + inst.n_b - lo
        self.n = n
        idx = torch.arange(1 << n, device=device)
        sign = [1.0 - 2.0 * ((idx >> (n - 1 - i)) & 1).double() for i in range(n)]
        self.diag = torch.zeros(1 << n, dtype=torch.float64, device=device)
        self.hops = []
        for i, j, jx, jy, jz in inst.couplings:
            if i < lo:
                continue
            a, b = i - lo, j - lo
            zz = sign[a] * sign[b]
            self.diag += jz * zz
            if jx or jy:
                # a scalar when it is the same on every row
                self.hops.append((idx ^ ((1 << (n - 1 - a)) | (1 << (n - 1 - b))), jx - jy * zz if jy else jx))
        for a in range(n):
            self.diag += float(inst.hz[lo + a]) * sign[a]
            if inst.hx[lo + a]:
                self.hops.append((idx ^ (1 << (n - 1 - a)), float(inst.hx[lo + a])))

    def __call__(self, x):
        y = self.diag[:, None] * x
        for perm, c in self.hops:
            y += (c[:, None] if torch.is_tensor(c) else c) * x.index_select(0, perm)
        return y

    def cost(self, cols, steps):
        return (1 << self.n) * cols * steps * (len(self.hops) + 4)


def _lanczos(op, x, k, keep):
    """k steps on every (unit) column: alpha, beta [k, C] and the basis."""
    alpha, beta, basis = [], [], []
    prev, q = torch.zeros_like(x), x
    b = torch.zeros(x.shape[1], dtype=x.dtype, device=x.device)
    big = torch.zeros_like(b)
    for _ in range(k):
        if keep:
            basis.append(q)
        r = op(q) - b * prev
        a = (q * r).sum(0)
        r -= a * q
        b = r.norm(dim=0)
        # an invariant subspace: that column's recurrence ends
        big = torch.maximum(big, torch.maximum(a.abs(), b))
        b = torch.where(b > 1e-12 * big, b, torch.zeros_like(b))
        alpha.append(a)
        beta.append(b)
        prev, q = q, torch.where(b > 0.0, r / b, torch.zeros_like(r))
    return torch.stack(alpha).cpu().numpy(), torch.stack(beta).cpu().numpy(), basis


def _eig(alpha, beta):
    """Eigensystems of every column's tridiagonal matrix."""
    k, c = alpha.shape
    t = np.zeros((c, k, k))
    d = np.arange(k)
    t[:, d, d] = alpha.T
    t[:, d[:-1], d[1:]] = t[:, d[1:], d[:-1]] = beta[:-1].T
    return np.linalg.eigh(t)


def _start(inst, device, kind="sysbath"):
    v = np.stack([_signs(inst.seed, j, inst.n_b) for j in range(inst.n_v)], axis=1) * 2.0 ** (-inst.n_b / 2)
    if kind == "bath":
        return torch.as_tensor(v, device=device)
    d_s, d_b = 1 << inst.n_s, 1 << inst.n_b
    if kind == "product":
        w = np.stack([_signs(inst.seed ^ 0x9E3779B97F4A7C15, j, inst.n_s) for j in range(inst.n_v)], axis=1)
        x = (w[:, None, :] * 2.0 ** (-inst.n_s / 2) * v[None]).reshape(d_s * d_b, inst.n_v)
        return torch.as_tensor(x, device=device)
    x = torch.zeros(d_s, d_b, inst.n_v, d_s, dtype=torch.float64, device=device)
    vt = torch.as_tensor(v, device=device)
    for m in range(d_s):
        x[m, :, :, m] = vt
    return x.reshape(d_s * d_b, inst.n_v * d_s)


def _bath_trace(inst, device, k):
    """Per beta: the mean quadrature of exp(-beta (H_b - E0b)), and E0b."""
    a, b, _ = _lanczos(_Operator(inst, True, device), _start(inst, device, "bath"), k, False)
    th, s = _eig(a, b)
    e0b = th.min()
    return [float((s[:, 0, :] ** 2 * np.exp(-bt * (th - e0b))).sum(1).mean()) for bt in inst.betas], float(e0b)


def _exact_solve(inst, op, device):
    k = min(inst.k, 1 << op.n)
    x = _start(inst, device)
    a, b, basis = _lanczos(op, x, k, True)
    th, s = _eig(a, b)
    e0 = th.min()
    d_s, ln_db = 1 << inst.n_s, inst.n_b * math.log(2.0)
    mbs, e0b = _bath_trace(inst, device, min(inst.k, 1 << inst.n_b))
    out = {key: [] for key in OUTPUTS}
    for bt, mb in zip(inst.betas, mbs):
        y = np.einsum("cjq,cq,cq->jc", s, np.exp(-0.5 * bt * (th - e0)), s[:, 0, :])
        yt = torch.as_tensor(np.ascontiguousarray(y), device=device)
        psi = torch.zeros_like(x)
        for j in range(k):
            psi += yt[j] * basis[j]
        p = psi.reshape(-1, inst.n_v, d_s).permute(1, 2, 0).contiguous()
        m = sum((p[j] @ p[j].T for j in range(inst.n_v)), torch.zeros(d_s, d_s, dtype=x.dtype, device=device))
        m = (m / inst.n_v).cpu().numpy()
        m = 0.5 * (m + m.T)
        mu, u = np.linalg.eigh(m)
        lt = math.log(np.trace(m)) - bt * e0 + ln_db
        lb = math.log(mb) - bt * e0b + ln_db
        he = -np.log(np.maximum(mu, mu.max() * 2.0 ** -52) / mb) / bt + e0 - e0b
        p = mu / mu.sum()
        p = p[p > 0.0]
        out["rho"].append(m / np.trace(m))
        out["h_star"].append((u * he) @ u.T)
        out["log_z"].append(lt - lb)
        out["entropy"].append(-(p * np.log(p)).sum())
        out["log_z_t"].append(lt)
        out["log_z_b"].append(lb)
    return {key: np.array(v) for key, v in out.items()}


def _exact_product(inst, op, device):
    a, b, _ = _lanczos(op, _start(inst, device, "product"), min(inst.k, 1 << op.n), False)
    th, s = _eig(a, b)
    e0, n = th.min(), inst.n_s + inst.n_b
    mbs, e0b = _bath_trace(inst, device, min(inst.k, 1 << inst.n_b))
    lzt, lzb, smp = [], [], []
    for bt, mb in zip(inst.betas, mbs):
        q = (s[:, 0, :] ** 2 * np.exp(-bt * (th - e0))).sum(1)
        smp.append(np.log(q) - bt * e0 + n * math.log(2.0))
        lzt.append(math.log(q.mean()) - bt * e0 + n * math.log(2.0))
        lzb.append(math.log(mb) - bt * e0b + inst.n_b * math.log(2.0))
    lzt, lzb = np.array(lzt), np.array(lzb)
    return {"log_z": lzt - lzb, "log_z_t": lzt, "log_z_b": lzb, "samples": np.array(smp)}


def _ground_vector(op, device, steps=200):
    """Ground state by Lanczos with full reorthogonalisation."""
    gen = torch.Generator(device=device).manual_seed(1)
    steps = min(steps, (1 << op.n) - 1)
    q = torch.randn(1 << op.n, generator=gen, dtype=torch.float64, device=device)
    basis = torch.zeros(steps, 1 << op.n, dtype=torch.float64, device=device)
    basis[0] = q / q.norm()
    alpha, beta = np.zeros(steps), np.zeros(steps)
    for j in range(steps):
        r = op(basis[j][:, None])[:, 0]
        alpha[j] = float(basis[j] @ r)
        for _ in range(2):
            r -= basis[:j + 1].T @ (basis[:j + 1] @ r)
        beta[j] = float(r.norm())
        if j + 1 < steps:
            basis[j + 1] = r / beta[j]
    th, s = _eig(alpha[:, None], beta[:, None])
    return float(th[0, 0]), basis.T @ torch.as_tensor(np.ascontiguousarray(s[0, :, 0]), device=device)


def _exact_ground(inst, op, device):
    e, psi = _ground_vector(op, device)
    eb, _ = _ground_vector(_Operator(inst, True, device), device)
    m = psi.reshape(1 << inst.n_s, -1)
    rho = (m @ m.T).cpu().numpy()
    rho /= np.trace(rho)
    mu = np.linalg.eigvalsh(rho)
    mu = mu[mu > 0.0]
    return {"rho": rho, "e_total": e, "e_bath": eb, "entropy": float(-(mu * np.log(mu)).sum())}


def exact(case, seed):
    kind = case["kind"]
    device = "cuda" if torch.cuda.is_available() else "cpu"
    # elements moved per second by the plain products here, 15 s of them at
    # most, and a stored FP64 basis of at most 40 GB
    limit = 15.0 * (8e10 if device == "cuda" else 2e7)
    insts = _instances(case, seed)
    ops, cost = [], 0.0
    for i in insts:
        # (a rough first look, before the operator's tables are built)
        if (1 << (i.n_s + i.n_b)) * i.n_v * i.k > limit:
            return None
        op = _Operator(i, False, device)
        cols = case["n_cols"] if kind == "apply" else i.n_v if kind == "product" else i.n_v << i.n_s
        steps = 200 if kind == "ground" else i.k
        cost += op.cost(cols, steps)
        ops.append(op)
        stored = 0 if kind in ("apply", "product", "ground") else (8 * cols * steps) << op.n
        if cost > limit or stored > 40e9:
            return None
    if kind == "apply":
        # the entry point's layout: panels of 16 bytes a row, zero padding
        y, w = ops[0](_block(case, seed).double()), 2 if case["precision"] == "fp64" else 4
        y = torch.nn.functional.pad(y, (0, -y.shape[1] % w))
        return y.reshape(y.shape[0], -1, w).permute(1, 0, 2).reshape(-1)
    if kind == "product":
        return _exact_product(insts[0], ops[0], device)
    if kind == "ground":
        return _exact_ground(insts[0], ops[0], device)
    if kind == "solve":
        return _exact_solve(insts[0], ops[0], device)
    res = [_exact_solve(i, o, device) for i, o in zip(insts, ops)]
    return np.array([r["entropy"] for r in res]) if kind == "grid" else _joined(res)
