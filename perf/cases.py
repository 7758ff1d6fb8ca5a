"""The work that programs built on this package have it do, as measurable cases.

Five kinds of call, each through the entry points a program uses:

* ``svd``       ``api.rrsvd_truncate`` on matrices of a decaying spectrum, the
                drop-in replacement of a truncated SVD;
* ``bond``      ``api.tebd_bond_update`` of one bond of a chain;
* ``sweep``     one symmetric Trotter step (three parity sweeps,
                ``api.tebd_sweep``) of a batch of chains from a given state;
* ``evolve``    a whole run of ``api.TEBD`` from a product state, with the
                one-site density matrices a program reads its observables from;
* ``gradient``  ``gradient.CheckpointedTEBD``: forward run, observable, reverse
                run, gate cotangents.

The chains are the package's own models (Ising, XX with random fields,
chain-mapped spin boson) with couplings drawn from the seed.

Outputs.  A singular triplet is defined up to a phase, and the phase that a
call returns follows the rounding of its Jacobi rotations: two correct runs
that round differently return other factors of the same matrix.  So the
factors come back as what a program makes of them and no phase enters: the
matrix U diag(S) V^H itself, and for chains the Schmidt values, the bond
dimensions and the density matrix of every site, from which observables are
read.  Discarded weights of the TEBD cases (1e-10 and below, the difference of
two norms close to 1) come back as the kept weights 1 - w.
"""
import math

import numpy as np
import torch

from paper_1504_00992_amd import _lib, api, gradient, models

EPS = 1e-10   # relative discarded weight of the package's benchmarks and tests
FLOOR = 1e-14
SPECTRUM = 25.0  # s_i = exp(-i / 25), the benchmark's matrices


def listed():
    svd = dict(kind="svd", count=1, m=96, n=80, ragged=False, k=24, p=10, q=2, precision=0)
    chain = dict(chains=1, sites=20, d=2, chi=32, cap=32, dt=0.01, adaptive=2, precision=0)
    return [
        # the smallest standalone call: one matrix in place of one LAPACK call
        dict(svd, name="svd_one"),
        # mixed rectangular matrices of a tensor-network contraction
        dict(svd, name="svd_ragged", count=16, m=640, n=500, ragged=True, k=48),
        # the benchmark's batch: sizes 256 ... 2048, k = 64
        dict(svd, name="svd_batch", count=20, m=2048, n=2048, ragged=True, k=64),
        # the same products in complex FP32
        dict(svd, name="svd_batch_f32", count=8, m=1024, n=1024, k=64, precision=1),
        # mixed-state blocks (100 d^2 at d = 7), k = p = 100
        dict(svd, name="svd_mixed_state", count=2, m=4900, n=4900, k=100, p=100),
        # one bond of a spin chain, the smallest TEBD call
        dict(chain, kind="bond", name="bond_spin"),
        # one step of one Ising chain, N = 20: latency
        dict(chain, kind="sweep", name="step_spin", model="ising", front=False),
        # one step of one XX chain whose bonds have reached chi_max = 64
        dict(chain, kind="sweep", name="step_saturated", model="xx", front=False, sites=40, chi=64,
             cap=64, dt=0.02),
        # one late step of 16 spin-boson chains, N = 100, d = 10
        dict(chain, kind="sweep", name="step_boson", model="boson", front=True, chains=16, sites=100,
             d=10, chi=19, cap=48, dt=0.05),
        # a run with the Accuracy Check as rank rule
        dict(chain, kind="evolve", name="run_accuracy_check", model="boson", chains=4, sites=40, d=8,
             cap=48, dt=0.05, steps=40, adaptive=3),
        # the gradient of <Z_0(T)> in the XX chain with random fields, N = 40
        dict(chain, kind="gradient", name="gradient_xx", model="xx", sites=40, cap=64, dt=0.02,
             steps=20, checkpoint=10),
        # the benchmark's evolution: 16 spin-boson chains, 200 steps
        dict(chain, kind="evolve", name="run_boson", model="boson", chains=16, sites=100, d=10,
             cap=100, dt=0.05, steps=200),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["svd", "svd", "svd", "bond", "sweep", "sweep", "sweep", "evolve", "gradient"])
    if kind == "svd":
        m = _log_int(rng, 48, 4900)
        n = max(40, min(4900, int(m * rng.uniform(0.6, 1.4))))
        # at most the matrix entries of the listed batch
        count = _log_int(rng, 1, max(1, min(20, int(2.4e7 / (m * n)))))
        k = min(_log_int(rng, 8, 128), min(m, n) // 2)
        return dict(kind=kind, count=count, m=m, n=n, ragged=count > 1 and rng.random() < 0.5, k=k,
                    p=rng.choice([5, 10, 10, 10, k]), q=rng.choice([1, 2, 2, 2, 3]),
                    precision=rng.choice([0, 0, 0, 1]))
    if kind == "bond":
        d = rng.randint(2, 8)
        chi = _log_int(rng, 4, min(100, 500 // d))
        return dict(kind=kind, chains=1, sites=rng.randint(4, 24), d=d, chi=chi, cap=chi,
                    dt=rng.uniform(0.01, 0.1), adaptive=rng.choice([0, 2]), precision=0)
    if kind == "sweep":
        model = rng.choice(["ising", "xx", "boson"])
        d = rng.randint(3, 10) if model == "boson" else 2
        front = model == "boson" and rng.random() < 0.6
        cap = _log_int(rng, 16, 100)
        chi = _log_int(rng, 4, min(cap, 24 if front else 128 // d + 8))
        chains = _log_int(rng, 1, 16 if front else 8)
        sites = _log_int(rng, 8, 100 if front else 40)
        return dict(kind=kind, model=model, chains=chains, sites=sites, d=d, chi=chi, cap=cap,
                    front=front, dt=rng.uniform(0.01, 0.06), adaptive=rng.choice([1, 2, 2, 2, 3]),
                    precision=0)
    if kind == "evolve":
        model = rng.choice(["ising", "xx", "boson"])
        d = rng.randint(3, 10) if model == "boson" else 2
        return dict(kind=kind, model=model, chains=_log_int(rng, 1, 16), sites=_log_int(rng, 10, 60),
                    d=d, cap=_log_int(rng, 24, 64), chi=0, dt=rng.uniform(0.02, 0.06),
                    steps=_log_int(rng, 4, 40), adaptive=rng.choice([2, 2, 3]), precision=0)
    return dict(kind=kind, model="xx", chains=1, sites=_log_int(rng, 10, 40), d=2, chi=0,
                cap=_log_int(rng, 16, 64), dt=rng.uniform(0.01, 0.03), steps=_log_int(rng, 3, 20),
                checkpoint=rng.randint(2, 10), adaptive=2, precision=0)


# ---------------------------------------------------------------------------
# Inputs

def _shapes(case):
    out = []
    for i in range(case["count"]):
        m, n = case["m"], case["n"]
        if case["ragged"]:  # m ... m / 8 for the rows, another order for the columns
            m = max(32, int(m * 0.5 ** (3.0 * (i % 7) / 6.0)))
            n = max(32, int(n * 0.5 ** (3.0 * ((3 * i + 1) % 7) / 6.0)))
        out.append((m, n))
    return out


def _factors(case, seed):
    """Gaussian factors and spectrum of every matrix, A = G diag(s) H."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1504 + seed)
    out = []
    for m, n in _shapes(case):
        r = min(m, n, 2 * (case["k"] + case["p"]) + 64)
        g = torch.randn((m, r), dtype=torch.complex128, device="cuda", generator=gen) / math.sqrt(m)
        h = torch.randn((r, n), dtype=torch.complex128, device="cuda", generator=gen) / math.sqrt(n)
        s = torch.exp(-torch.arange(r, dtype=torch.float64, device="cuda") / SPECTRUM)
        out.append((g, s, h))
    return out


def _dims(case):
    d, n = case["d"], case["sites"]
    return [2] + [d] * (n - 1) if case.get("model") == "boson" else [d] * n


def _bond_hams(case, seed):
    rng = np.random.default_rng([1504, seed])
    n, model = case["sites"], case.get("model")
    if model == "ising":
        zz = np.kron(models.PAULI_Z, models.PAULI_Z)
        one = np.kron(models.PAULI_X, np.eye(2))
        two = np.kron(np.eye(2), models.PAULI_X)
        return [-rng.uniform(0.9, 1.1) * zz - 0.5 * rng.uniform(0.9, 1.1) * (one + two)
                for _ in range(n - 1)]
    if model == "xx":
        return models.xx_chain(rng.uniform(0.8, 1.2, n - 1), rng.uniform(-1.0, 1.0, n))[1]
    w, t, t0 = rng.uniform(0.95, 1.05), rng.uniform(0.45, 0.55), rng.uniform(0.45, 0.55)
    return models.spin_boson(n, case["d"], t0=t0, omegas=w, hops=t)[1]


def _gates(dims, hams, tau):
    """exp(-i tau h_b) of every bond on the device; a uniform chain's repeated
    Hamiltonians are exponentiated once."""
    dm = max(dims)
    out = np.zeros((len(hams), dm * dm, dm * dm), dtype=np.complex128)
    seen = {}
    for b, h in enumerate(hams):
        key = h.tobytes()
        if key not in seen:
            seen[key] = models.propagator(h, tau)
        k = h.shape[0]
        out[b, :k, :k] = seen[key]
    return torch.from_numpy(out).cuda()


def _profile(case):
    """Bond dimensions: full (grown from the ends), or the light cone of an
    excitation entering at the left (peak near the start, then 2 and 1)."""
    dims, chi, n = _dims(case), case["chi"], case["sites"]
    cut = [1] * (n + 1)
    left = right = 1
    for k in range(1, n):
        left = min(left * dims[k - 1], chi)
        cut[k] = left
    for k in range(n - 1, 0, -1):
        right = min(right * dims[k], chi)
        cut[k] = min(cut[k], right)
    if case.get("front"):
        for k in range(1, n):
            decay = chi * math.exp(-max(0, k - 4) / 5.0)
            cut[k] = min(cut[k], max(1, int(round(decay))))
    return cut


def _random_state(case, seed):
    """gamma, lam, chi of random chains: Schmidt values falling to 2e-5, the
    weight lambda_a Gamma lambda_b of the tensors graded like the Schmidt
    values on either side, higher local levels less occupied; the bonds of
    dimension 1 ahead of the front hold the vacuum."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(99 + seed)
    dims, chis, cap = _dims(case), _profile(case), case["cap"]
    nc, n, dm = case["chains"], case["sites"], max(dims)
    gamma = torch.zeros((nc, n, dm, cap, cap), dtype=torch.complex128, device="cuda")
    lam = torch.zeros((nc, n - 1, cap), dtype=torch.float64, device="cuda")
    chi = torch.tensor(chis, dtype=torch.int32, device="cuda").repeat(nc, 1).contiguous()
    last = max([k for k in range(n + 1) if chis[k] > 1], default=0)

    def schmidt(c):
        x = torch.exp(-torch.arange(c, dtype=torch.float64, device="cuda") * (10.8 / max(c, 4)))
        return x / x.norm()

    for k in range(n):
        d, cl, cr = dims[k], chis[k], chis[k + 1]
        left, right = schmidt(cl), schmidt(cr)
        if k < n - 1:
            lam[:, k, :cr] = right
        if cl == 1 and cr == 1 and k > last:
            gamma[:, k, 0, 0, 0] = 1.0
        else:
            level = torch.exp((-4.0 if d > 2 else -2.5) * torch.arange(d, dtype=torch.float64, device="cuda"))
            b = torch.randn((nc, d, cl, cr), dtype=torch.complex128, device="cuda", generator=gen)
            grade = level[:, None, None] / torch.sqrt(left[:, None] * right[None, :])
            gamma[:, k, :d, :cl, :cr] = b * grade
    return gamma, lam, chi


def _params(case):
    return _lib.params(case["cap"], 10, 2, EPS, FLOOR, 1504, 0, case["precision"], case["adaptive"])


def _levels(case):
    return [i % 2 for i in range(case["sites"])] if case["model"] == "xx" else [0] * case["sites"]


def prepare(case, seed):
    kind = case["kind"]
    if kind == "svd":
        return dict(case, mats=[((g * s) @ h).contiguous() for g, s, h in _factors(case, seed)])
    dims = _dims(case)
    hams = _bond_hams(case, seed)
    if kind in ("bond", "sweep"):
        mps = api.DeviceMPS(case["chains"], dims, case["cap"])
        start = _random_state(case, seed)
        prm = _params(case)
        st = dict(case, mps=mps, start=start, prm=prm, ws=api.BondWorkspace(mps, prm))
        if kind == "bond":
            st["gate"] = _gates(dims[:2], _generic_pair(case, seed), case["dt"])[0].contiguous()
        else:
            full, half = _gates(dims, hams, case["dt"]), _gates(dims, hams, 0.5 * case["dt"])
            st["gates"] = {1.0: full, 0.5: half}
        return st
    mps = api.DeviceMPS.product_state(case["chains"], dims, _levels(case), case["cap"])
    start = (mps.gamma.clone(), mps.lam.clone(), mps.chi.clone())
    if kind == "evolve":
        drv = api.TEBD(mps, hams, case["dt"], case["cap"], p=10, q=2, trunc_eps=EPS,
                       adaptive=case["adaptive"], precision=case["precision"])
        return dict(case, mps=mps, start=start, drv=drv)
    drv = gradient.CheckpointedTEBD(mps, _gates(dims, hams, 0.5 * case["dt"]),
                                    _gates(dims, hams, case["dt"]), case["cap"], 10, 2, EPS, 1504,
                                    adaptive=case["adaptive"], checkpoint=case["checkpoint"])
    z = torch.tensor([[1.0, 0.0], [0.0, -1.0]], dtype=torch.complex128, device="cuda")
    return dict(case, mps=mps, start=start, drv=drv, z=z)


def _generic_pair(case, seed):
    """A two-site Hamiltonian of dimension d^2 with all matrix elements."""
    rng = np.random.default_rng([7, seed])
    k = case["d"] ** 2
    h = rng.standard_normal((k, k)) + 1j * rng.standard_normal((k, k))
    return [(h + h.conj().T) / math.sqrt(8.0 * k)]


# ---------------------------------------------------------------------------
# One pass

def _reset(st):
    mps, (g, lam, chi) = st["mps"], st["start"]
    mps.gamma.copy_(g)
    mps.lam.copy_(lam)
    mps.chi.copy_(chi)
    return mps


def _density(gamma, lam):
    """One-site density matrices of every chain and site (Vidal form)."""
    nc, n, d, cap, _ = gamma.shape
    one = torch.ones((nc, 1, cap), dtype=lam.dtype, device=lam.device)
    left = torch.cat([one, lam], 1)
    right = torch.cat([lam, one], 1)
    x = gamma * (left[:, :, None, :, None] * right[:, :, None, None, :])
    x = x.reshape(nc * n, d, cap * cap)
    return torch.bmm(x, x.mH).reshape(nc, n, d, d)


def run(st):
    kind = st["kind"]
    if kind == "svd":
        u, s, vh, chi, w, status = api.rrsvd_truncate(st["mats"], st["k"], p=st["p"], q=st["q"],
                                                      trunc_eps=EPS, precision=st["precision"])
        return {"low_rank": [(a * b) @ c for a, b, c in zip(u, s, vh)], "S": s, "chi": chi, "w": w,
                "status": status}
    if kind in ("bond", "sweep"):
        mps, ws, prm = _reset(st), st["ws"], st["prm"]
        if kind == "bond":
            api.tebd_bond_update(mps, 0, (st["sites"] - 1) // 2, st["gate"], prm, ws)
        else:
            for i, (parity, frac) in enumerate(api.trotter_schedule(2)):
                prm.stream_id = i
                api.tebd_sweep(mps, st["gates"][frac], parity, prm, ws)
        return {"density": _density(mps.gamma, mps.lam), "lam": mps.lam, "chi": mps.chi,
                "kept": 1.0 - ws.disc, "status": ws.status}
    mps, drv = _reset(st), st["drv"]
    if kind == "evolve":
        drv.sweeps_done = 0
        for _ in range(st["steps"]):
            drv.step()
        return {"density": _density(mps.gamma, mps.lam), "lam": mps.lam, "chi": mps.chi,
                "kept": 1.0 - drv.ws.disc, "status": drv.ws.status}
    drv.forward(st["steps"])
    gam = mps.gamma[0].clone().requires_grad_(True)
    lam = mps.lam[0].clone().requires_grad_(True)
    loss = gradient.expectation(gam, lam, st["z"], 0)
    loss.backward()
    gh, gf, _, _ = drv.backward(gam.grad[None], lam.grad[None])
    return {"loss": loss.detach(), "gates_half": gh, "gates_full": gf}


# ---------------------------------------------------------------------------
# What a pass cannot do without

def _rrsvd_flops(m, n, k, p, q):
    l = min(k + p, m, n)
    qr = sum(16.0 * r * l * l - 16.0 / 3.0 * l ** 3 for r in [m] * (q + 1) + [n] * (q + 1))
    return (2 * q + 2) * 8.0 * m * n * l + qr + 8.0 * (m + n) * l * min(k, l)


def _bond_flops(dl, dr, cl, cm, cr, p, q):
    m, n = dl * cl, dr * cr
    return (8.0 * m * n * cm + 8.0 * (dl * dr) ** 2 * cl * cr
            + _rrsvd_flops(m, n, min(cm, m, n), p, q))


def work(case):
    kind = case["kind"]
    if kind == "svd":
        k, p, q = case["k"], case["p"], case["q"]
        fl = sum(_rrsvd_flops(m, n, k, p, q) for m, n in _shapes(case))
        by = sum(16.0 * (m * n + k * (m + n)) + 8.0 * k for m, n in _shapes(case))
        return {"bytes": by, "flops": fl}
    dims = _dims(case)
    n = case["sites"]
    if kind in ("bond", "sweep"):
        chis = _profile(case)
        bonds = ([(n - 1) // 2] if kind == "bond"
                 else [b for par in (0, 1, 0) for b in range(par, n - 1, 2)])
        fl = by = 0.0
        for b in bonds:
            fl += _bond_flops(dims[b], dims[b + 1], chis[b], chis[b + 1], chis[b + 2], 10, 2)
            by += 16.0 * (dims[b] * dims[b + 1]) ** 2 / case["chains"]
            by += 2 * 16.0 * (dims[b] * chis[b] * chis[b + 1] + dims[b + 1] * chis[b + 1] * chis[b + 2])
        return {"bytes": by * case["chains"], "flops": fl * case["chains"]}
    # a run grows its bonds from 1: at least the products of dimension-1 bonds
    # at every step, the initial state read and the final one written
    sweeps = 3 * case["steps"] * (3 if kind == "gradient" else 1)
    fl = sum(_bond_flops(dims[b], dims[b + 1], 1, 1, 1, 10, 2) for b in range(n - 1))
    by = 2.0 * 16.0 * sum(dims) + 32.0 * sum((dims[b] * dims[b + 1]) ** 2 for b in range(n - 1))
    return {"bytes": (by * case["chains"]), "flops": 0.5 * sweeps * fl * case["chains"]}


# ---------------------------------------------------------------------------
# The same in plain numpy, 64 bits

def _cut(s, frob2, cap):
    tail = np.maximum(frob2 - np.cumsum(s * s), 0.0)
    rest = np.concatenate([np.cumsum((s * s)[::-1])[::-1][1:], [0.0]])
    w = np.minimum(rest, tail) / frob2 if frob2 > 0 else rest
    ok = np.nonzero(w <= EPS)[0]
    c = int(ok[0]) + 1 if len(ok) and ok[0] + 1 <= cap else min(cap, len(s))
    return c, float(rest[c - 1] / frob2)


def _exact_svd(case, seed):
    values, weights = [], []
    k = case["k"]
    for (g, s, h), (m, n) in zip(_factors(case, seed), _shapes(case)):
        r1 = torch.linalg.qr(g.cpu())[1].numpy()
        r2 = torch.linalg.qr(h.mH.contiguous().cpu())[1].numpy()
        x = np.linalg.svd((r1 * s.cpu().numpy()) @ r2.conj().T, compute_uv=False)
        c, w = _cut(x, float(np.sum(x * x)), k)
        out = np.zeros(k)
        out[:c] = x[:c]
        values.append(out)
        weights.append(w)
    return {"S": values, "w": np.array(weights)}


def _exact_bond(gam, lam, chi, b, gate, cap, n):
    """One two-site update of one chain by a full SVD, in place."""
    cl, cm, cr = chi[b], chi[b + 1], chi[b + 2]
    gl, gr = gam[b], gam[b + 1]
    dl, dr = gl.shape[0], gr.shape[0]
    ll = lam[b - 1][:cl] if b else np.ones(1)
    lr = lam[b + 1][:cr] if b + 1 <= n - 2 else np.ones(1)
    left = ll[None, :, None] * gl[:, :cl, :cm] * lam[b][:cm]
    right = gr[:, :cm, :cr] * lr
    th = np.einsum("iag,jgc->ijac", left, right).reshape(dl * dr, cl * cr)
    a = (gate[:dl * dr, :dl * dr] @ th).reshape(dl, dr, cl, cr)
    a = a.transpose(0, 2, 1, 3).reshape(dl * cl, dr * cr)
    u, s, vh = np.linalg.svd(a, full_matrices=False)
    c, w = _cut(s, float(np.sum(s * s)), cap)
    lam[b] = np.zeros(cap)
    lam[b][:c] = s[:c] / np.linalg.norm(s[:c])
    chi[b + 1] = c
    gam[b] = u[:, :c].reshape(dl, cl, c) / ll[None, :, None]
    gam[b + 1] = vh[:c].reshape(c, dr, cr).transpose(1, 0, 2) / lr
    return w


def exact(case, seed):
    kind = case["kind"]
    if kind == "svd":
        big = sum(max(s) * (2 * (case["k"] + case["p"]) + 64) ** 2 for s in _shapes(case))
        return _exact_svd(case, seed) if big < 4e9 else None
    if kind not in ("bond", "sweep") or case["precision"]:
        return None
    dims, chis, n, cap = _dims(case), _profile(case), case["sites"], case["cap"]
    bonds = [(n - 1) // 2] if kind == "bond" else range(n - 1)
    cost = sum(2 * case["chains"] * (max(dims[b] * chis[b], 8) * max(dims[b + 1] * chis[b + 2], 8)
                                     * min(dims[b] * chis[b], dims[b + 1] * chis[b + 2])) for b in bonds)
    if cost > 5e8:
        return None
    g, l, c = (x.cpu().numpy() for x in _random_state(case, seed))
    hams = _bond_hams(case, seed)
    lam_out, g_out = np.zeros(l.shape), np.zeros(g.shape, dtype=g.dtype)
    kept = np.ones(l.shape[:2])
    if kind == "bond":
        gate = models.propagator(_generic_pair(case, seed)[0], case["dt"])
    else:
        gates = {f: [models.propagator(h, f * case["dt"]) for h in hams] for f in (1.0, 0.5)}
    for ch in range(case["chains"]):
        chi = [int(x) for x in c[ch]]
        gam = [g[ch, k, :dims[k], :chi[k], :chi[k + 1]] for k in range(n)]
        lam = [l[ch, b] for b in range(n - 1)]
        if kind == "bond":
            b = (n - 1) // 2
            kept[ch, b] = 1.0 - _exact_bond(gam, lam, chi, b, gate, cap, n)
        else:
            for par, frac in ((0, 0.5), (1, 1.0), (0, 0.5)):
                for b in range(par, n - 1, 2):
                    kept[ch, b] = 1.0 - _exact_bond(gam, lam, chi, b, gates[frac][b], cap, n)
        lam_out[ch] = lam
        for k in range(n):
            x = gam[k]
            g_out[ch, k, :x.shape[0], :x.shape[1], :x.shape[2]] = x
    density = _density(torch.from_numpy(g_out), torch.from_numpy(lam_out))
    return {"density": density, "lam": lam_out, "kept": kept}
