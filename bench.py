"""Throughput of the batched TEBD bond update with RRSVD on one MI355X.

Headline workload: 16 independent chain-mapped spin-boson chains (Eq. H_1D:
spin-1/2 plus 99 oscillators truncated to d = 10, t_n = 0.5, omega_n = 1),
chi_max = 100, RRSVD with p = 10, q = 2, per-bond discarded weight
<= 1e-10, dt = 0.05, 200 symmetric Trotter steps from |up>|0...0>.  One
"step" of this benchmark is the whole 200-step evolution of all 16 chains
from the product state (600 sweeps, 476,800 bond updates): --warmup W such
evolutions run untimed, then --steps K are timed one by one (the state is
reset to the product state outside the timed region; every repetition
computes the same numbers, its Gaussian test matrices included).

The JSON line also carries:
* roofline   -- the kernel with the largest event time in a profiled
                repetition of the same evolution (HIP events around every
                launch, on the launch's stream); algorithmic flops and bytes
                from the recorded bond dimensions of every problem of every
                sweep, divided by that kernel's summed event time; measured
                HBM bytes per launch from committed rocprofv3 counters while
                the kernel sources match them;
* cpu_baseline -- the FP64 CPU oracle (full-SVD TEBD) on chain 0 of the same
                workload, all 200 steps;
* full_svd   -- the same evolution with the vendor full SVD
                (torch.linalg.svd), batched over every same-shape bond of a
                sweep, truncated on the device, on this GPU;
* tfim, batched_rrsvd, mixed_precision, adjoint -- the other workloads
                (plain TEBD N = 20; 256 standalone RRSVDs; chi_max = 128 with
                complex FP32 sketches; the reverse-mode gradient of the XX
                chain), each with its own roofline and CPU-oracle figure.
"""
import argparse
import hashlib
import json
import os
import re
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_FP64_TFLOPS = 78.6      # MI355X dense FP64 (matrix and vector)
PEAK_FP32_MFMA_TFLOPS = 157.3
PEAK_HBM_GBS = 8000.0
METRIC = "TEBD bond updates/s, RRSVD vs full SVD on 1 GPU at <=1e-10 trunc err"

SB = dict(N=100, d=10, chi_max=100, p=10, q=2, dt=0.05, steps=200, eps=1e-10, seed=1504)
TFIM = dict(N=20, chi_max=32, p=10, q=2, dt=0.01, steps=100, eps=1e-10, seed=1504)


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5,
                    help="timed repetitions of the whole 200-step evolution")
    ap.add_argument("--warmup", type=int, default=1,
                    help="untimed repetitions before the timed ones")
    ap.add_argument("--chains", type=int, default=16)
    ap.add_argument("--copy-probe", action="store_true",
                    help="only copy a 256 MiB device buffer three times (the known-size kernel "
                         "that scales the HBM byte counters) and exit")
    ap.add_argument("--headline-only", action="store_true",
                    help="the headline evolution only (timed, then one profiled repetition)")
    ap.add_argument("--no-profile", action="store_true", help="skip the profiled repetition")
    ap.add_argument("--only", choices=("tfim", "batched", "mixed", "adjoint", "table2"),
                    help="run one secondary workload alone (no headline) and print its entry; "
                         "for profiling that workload by itself")
    for x in ("cpu-baseline", "full-svd", "other-rank", "graph", "tfim", "batched", "mixed",
              "adjoint", "table2", "tedopa", "accuracy", "order4"):
        ap.add_argument(f"--no-{x}", action="store_true")
    # host-only post-processing of rocprofv3 output into the summaries under
    # profiles/ (no GPU): a kernel-trace database, or the FETCH_SIZE and
    # WRITE_SIZE counter CSVs of a run and of the copy probe
    ap.add_argument("--summarize-trace", metavar="RESULTS_DB",
                    help="write a per-kernel summary of a rocprofv3 --kernel-trace database")
    ap.add_argument("--summarize-traffic", nargs=4,
                    metavar=("FETCH_CSV", "WRITE_CSV", "PROBE_FETCH_CSV", "PROBE_WRITE_CSV"),
                    help="write profiles/<workload>_hbm_traffic.txt from counter collections")
    ap.add_argument("--workload", default="spin_boson_16x100")
    ap.add_argument("--command", default="", help="the command the rocprofv3 output came from")
    ap.add_argument("--out", default=None)
    ap.add_argument("--rank", choices=("adaptive", "fixed"), default="adaptive",
                    help="rank of the timed run: two-stage adaptive (k1 from the bond dimension, "
                         "k = chi_max when needed) or fixed k = chi_max")
    a = ap.parse_args()
    if a.headline_only:
        for x in ("cpu_baseline", "full_svd", "other_rank", "graph", "tfim", "batched", "mixed",
                  "adjoint", "table2", "tedopa", "accuracy", "order4"):
            setattr(a, "no_" + x, True)
    return a


def _progress(msg):
    print(f"[bench] {msg}", file=sys.stderr, flush=True)


# ---------------------------------------------------------------------------
# Algorithmic work per kernel (complex arithmetic: one multiply-add = 8 real
# flops; bytes are those the operation must move between HBM and the chip).
def qr_flops(rows, l):
    """Householder factorisation plus explicit thin Q, complex."""
    return 16.0 * rows * l * l - 16.0 / 3.0 * l ** 3


def qr_bytes(rows, l, with_r=False):
    """Read the rows x l sketch, write Q (and the l x l R)."""
    return 16.0 * (2 * rows * l + (l * l if with_r else 0))


# The QRs without pivoting run as k_gram_qr, or as k_gram, k_chol and k_qapply for
# large sketches, counted together under that name with a Householder QR's work.
# A run that has no such kernel took the Householder ones, as sweeps with FP32
# products do in the size classes 0 and 1; their larger sketches have a Gram-based
# QR of their own but for B^H.
GRAM_QR = "k_gram_qr"
GRAM_PARTS = ("k_gram<", "k_chol<", "k_qapply<")
QR_KERNELS = ("k_qr_reg<512, 8, {}>", "k_qr_reg<1024, 12, {}>", "k_qr_lds<1024>", "k_qr_glb<1024>")


class Work:
    """{kernel name: [flops, bytes]} accumulated problem by problem."""

    def __init__(self, lib):
        self.lib = lib
        self.k = {}
        self.unpivoted = {}   # the part of each QR kernel's entry that the Gram-based QR does
        self._cls = {}

    def add(self, name, flops, nbytes):
        e = self.k.setdefault(name, [0.0, 0.0])
        e[0] += flops
        e[1] += nbytes

    def qr_class(self, rows, l):
        key = (rows, l)
        if key not in self._cls:
            self._cls[key] = self.lib.tebd_size_class(0, rows, l)
        return self._cls[key]

    def qr(self, rows, l_class, l, pivot, with_r=False, mixed=False):
        cls = self.qr_class(rows, l_class)
        name = QR_KERNELS[cls].format("true" if pivot else "false")
        self.add(name, qr_flops(rows, l), qr_bytes(rows, l, with_r))
        if pivot or (mixed and cls < 2):
            return
        if with_r or not mixed:
            self.add(GRAM_QR, qr_flops(rows, l), qr_bytes(rows, l, with_r))
        e = self.unpivoted.setdefault(name, [0.0, 0.0])
        e[0] += qr_flops(rows, l)
        e[1] += qr_bytes(rows, l, with_r)

    def rrsvd_pass(self, m, n, l, q, mixed, chi_new, form=True):
        """Kernels of Alg. 1 and steps i-iii for one problem at width l
        (form=False: a first pass whose result the second pass replaces)."""
        lc = l
        sk = "k_sketch_f32<{}>" if mixed else "k_sketch<{}>"
        mn, f = 16.0 * m * n, 8.0 * m * n * l
        self.add("k_omega", 0.0, 16.0 * n * l)
        self.add(sk.format(0), f, mn + 16.0 * (n * l + m * l))
        self.qr(m, lc, l, True)
        for _ in range(q):
            self.add(sk.format(1), f, mn + 16.0 * (m * l + n * l))
            self.qr(n, lc, l, False, mixed=mixed)
            self.add(sk.format(2), f, mn + 16.0 * (n * l + m * l))
            self.qr(m, lc, l, False, mixed=mixed)
        self.add("k_sketch<1>", f, mn + 16.0 * (m * l + n * l))   # B^H = A^H Q (FP64)
        self.qr(n, lc, l, False, with_r=True, mixed=mixed)   # B^H = Q_B R_B, column order
        c = chi_new
        if not form:
            return
        self.add("k_form_uv<1>", 8.0 * (m + n) * l * c,
                 16.0 * (m * l + l * c + m * c) + 16.0 * (n * l + l * c + n * c))


def first_stage_rank(chi_mid, chi_max):
    return min(chi_max, chi_mid + max(4, (chi_mid + 3) // 4))


def sweep_work(work, chi_before, chi_after, status, parity, dims, chi_max, p, q, adaptive,
               mixed=False, bonds=None, gate_bytes=None):
    """Add every problem of one recorded sweep (all chains) to `work`.

    chi_before / chi_after: [chains, N + 1]; status: [chains, N - 1] after the
    sweep (bit 64: the problem ran the second, fixed-rank pass).  The first
    pass runs at l1 = min(k1 + p, m, n) (k1 = chi_max without the adaptive
    rank); the QRs after the first work on the rank it reveals, at most l1,
    so the counts are upper bounds there."""
    n_ch = chi_before.shape[0]
    for c in range(n_ch):
        for b in (range(parity, len(dims) - 1, 2) if bonds is None else bonds):
            cl, cm, cr = int(chi_before[c, b]), int(chi_before[c, b + 1]), int(chi_before[c, b + 2])
            dl, dr = dims[b], dims[b + 1]
            m, n = dl * cl, dr * cr
            cnew = int(chi_after[c, b + 1])
            work.add("k_theta", 8.0 * dl * cl * cm * dr * cr,
                     16.0 * (dl * cl * cm + dr * cm * cr + dl * dr * cl * cr))
            first = c == 0 if gate_bytes is None else gate_bytes
            gbytes = 16.0 * (dl * dr) ** 2 if first else 0.0   # gates shared by the chains
            work.add("k_gate", 8.0 * (dl * dr) ** 2 * cl * cr,
                     gbytes + 16.0 * 2 * dl * dr * cl * cr)
            k1 = first_stage_rank(cm, chi_max) if adaptive else chi_max
            l1 = min(k1 + p, m, n)
            retried = adaptive and int(status[c, b]) & 64
            work.rrsvd_pass(m, n, l1, q, mixed, cnew, form=not retried)
            if retried:
                l2 = min(chi_max + p, m, n)
                work.rrsvd_pass(m, n, l2, q, mixed, cnew)


# ---------------------------------------------------------------------------
# Measured HBM bytes (rocprofv3 FETCH_SIZE / WRITE_SIZE, scaled by a copy of
# known size), keyed by kernel, valid while the kernel sources are unchanged.
CSRC = os.path.join(ROOT, "paper_1504_00992_amd", "csrc")


def code_digest():
    """sha256 over the library's kernel sources with comments and white
    space removed (a comment-only change keeps the digest)."""
    h = hashlib.sha256()
    for f in sorted(os.listdir(CSRC)):
        if not f.endswith((".hip", ".hpp", ".cpp", ".h")):
            continue
        text = open(os.path.join(CSRC, f), encoding="utf-8").read()
        text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
        text = re.sub(r"//[^\n]*", "", text)
        h.update(f.encode())
        h.update(re.sub(r"\s+", "", text).encode())
    return h.hexdigest()


def measured_traffic(kernel, workload):
    """HBM bytes per launch of `kernel` from profiles/<workload>_hbm_traffic.txt,
    or None when absent or taken on other kernel sources."""
    path = os.path.join(ROOT, "profiles", f"{workload}_hbm_traffic.txt")
    try:
        lines = open(path).read().splitlines()
    except OSError:
        return None, None
    fields = dict(l[2:].split(": ", 1) for l in lines if l.startswith("# ") and ": " in l)
    if fields.get("kernel sources sha256") != code_digest():
        return None, os.path.basename(path)
    for l in lines:
        if l.startswith("#") or not l.strip():
            continue
        parts = l.rsplit(None, 4)
        if len(parts) == 5 and parts[0].strip() == kernel:
            return float(parts[4]), os.path.basename(path)
    return None, os.path.basename(path)


ALU_KERNELS = ("k_qr_", "k_svd_pairs", "k_small_svd", "k_jac_", "k_omega", "k_schedule",
               "k_plan", "k_stage2", "k_frob")


def merge_tile_variants(prof):
    """The tile variants of a sketch product (k_sketch<i> on 32 x 32,
    k_sketch_wide<i> on 64 x 64, k_sketch_split<i> on split-depth 16 x 16
    tiles, picked per launch by the autotune cache) do the same work: count
    them as one kernel, k_sketch<i>.  The parts of the large sketches' Gram-based
    QR count as k_gram_qr."""
    out = {}
    for k, (ms, n) in prof.items():
        key = k.replace("k_sketch_wide<", "k_sketch<").replace("k_sketch_split<", "k_sketch<")
        key = GRAM_QR if key.startswith(GRAM_PARTS) else key
        a = out.get(key, (0.0, 0))
        out[key] = (a[0] + ms, a[1] + n)
    return out


def kernel_roofline(prof, work, workload, name=None):
    """Roofline entry of one kernel: `name`, or the one with the largest event time."""
    wide = any(k.startswith(("k_sketch_wide<", "k_sketch_split<")) for k in prof)
    prof = merge_tile_variants(prof)
    kern = {k: v for k, v in prof.items() if k.startswith("k_")}
    if not kern:
        return None
    if name is None:
        name = max(kern, key=lambda k: kern[k][0])
    ms, launches = kern[name]
    e = {"kernel": name, "launches": launches, "event_ms_total": round(ms, 3),
         "avg_launch_us": round(1e3 * ms / launches, 3) if launches else None}
    if wide and name.startswith("k_sketch<"):
        e["note_variants"] = ("launches of the tile variants k_sketch<i>, k_sketch_wide<i> "
                              "and k_sketch_split<i> counted together")
    fl, by = work.k.get(name, (0.0, 0.0))
    if GRAM_QR in prof and name in work.unpivoted:
        fl, by = fl - work.unpivoted[name][0], by - work.unpivoted[name][1]
    f32 = name.startswith("k_sketch_f32")
    if fl > 0 and ms > 0:
        ach = fl / (ms * 1e-3) / 1e12
        alu = name.startswith(ALU_KERNELS)
        peak = PEAK_FP32_MFMA_TFLOPS if f32 else PEAK_FP64_TFLOPS
        e.update({"bound": "alu" if alu else "mfma", "achieved": round(ach, 4), "peak": peak,
                  "unit": "TFLOP/s", "frac": round(ach / peak, 5)})
        e["flops_per_launch"] = round(fl / launches)
        e["algorithmic_bytes_per_launch"] = round(by / launches)
        e["hbm_GBps_algorithmic"] = round(by / (ms * 1e-3) / 1e9, 2)
    else:
        # no fixed flop count (iterative or data movement): rate in bytes
        gbs = by / (ms * 1e-3) / 1e9 if ms > 0 else None
        e.update({"bound": "hbm", "achieved": round(gbs, 3) if gbs else None,
                  "peak": PEAK_HBM_GBS, "unit": "GB/s",
                  "frac": round(gbs / PEAK_HBM_GBS, 5) if gbs else None,
                  "note": "no fixed algorithmic flop count: bytes per event time"})
        e["algorithmic_bytes_per_launch"] = round(by / launches) if launches else None
    t, src = measured_traffic(name, workload)
    e["traffic"] = round(t) if t is not None else None
    if src:
        e["traffic_source"] = f"profiles/{src}" + ("" if t is not None else
                                                   " (taken on other kernel sources: not used)")
    e["measured"] = "HIP events around every launch of a profiled repetition, on its stream"
    return e


def kernel_rooflines(prof, work, workload):
    """The roofline position of every library kernel of a run, by event time
    (achieved, peak and fraction as in the roofline entry; traffic = measured
    HBM bytes per launch where the counters match the kernel sources)."""
    merged = merge_tile_variants(prof)
    out = {}
    for name in sorted((k for k in merged if k.startswith("k_")), key=lambda k: -merged[k][0]):
        e = kernel_roofline(prof, work, workload, name)
        out[name] = {k: e.get(k) for k in ("launches", "avg_launch_us", "bound", "achieved",
                                            "peak", "unit", "frac", "algorithmic_bytes_per_launch",
                                            "traffic")}
    return out


def kernel_table(prof):
    k = {n: v for n, v in prof.items() if n.startswith("k_")}
    return {n: [round(v[0], 3), int(v[1])] for n, v in sorted(k.items(), key=lambda kv: -kv[1][0])}


def phase_table(prof):
    k = {n: v for n, v in prof.items() if not n.startswith("k_")}
    return {n: [round(v[0], 3), int(v[1])] for n, v in sorted(k.items(), key=lambda kv: -kv[1][0])}


# ---------------------------------------------------------------------------
def updates_per_step(n_sites):
    even = n_sites // 2
    odd = (n_sites - 1) // 2
    return 2 * even + odd


class Evolution:
    """A batch of chains evolved by api.TEBD, restartable from its initial
    state (the reset runs outside any timed region)."""

    def __init__(self, torch, api, dims, hb, levels, chains, chi_max, p, q, dt, eps, seed,
                 adaptive=2, precision=0):
        self.torch = torch
        self.mps = api.DeviceMPS.product_state(chains, dims, levels, chi_max)
        self.init = (self.mps.gamma.clone(), self.mps.lam.clone(), self.mps.chi.clone())
        self.drv = api.TEBD(self.mps, hb, dt, chi_max, p=p, q=q, trunc_eps=eps, seed=seed,
                            adaptive=adaptive, precision=precision)
        self.dims = dims

    def reset(self):
        self.mps.gamma.copy_(self.init[0])
        self.mps.lam.copy_(self.init[1])
        self.mps.chi.copy_(self.init[2])
        self.drv.sweeps_done = 0
        self.drv.ws.status.zero_()

    def run(self, steps, record=None):
        """Evolve `steps` steps; with record=list, append (parity, chi before,
        chi after, status) of every sweep (device tensors)."""
        d = self.drv
        for _ in range(steps):
            for parity, gates in d.schedule:
                before = self.mps.chi.clone() if record is not None else None
                d.sweep(parity, gates)
                if record is not None:
                    record.append((parity, before, self.mps.chi.clone(), d.ws.status.clone()))

    def timed(self, steps, reps, warmup):
        torch = self.torch
        for _ in range(warmup):
            self.reset()
            self.run(steps)
        torch.cuda.synchronize()
        times = []
        for _ in range(reps):
            self.reset()
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            self.run(steps)
            torch.cuda.synchronize()
            times.append(time.perf_counter() - t0)
        return times

    def profiled(self, steps, lib):
        """One repetition with per-launch events; returns (prof, history)."""
        torch = self.torch
        self.reset()
        torch.cuda.synchronize()
        hist = []
        lib.tebd_profile_enable(True)
        self.run(steps, record=hist)
        torch.cuda.synchronize()
        prof = lib.tebd_profile_read()
        lib.tebd_profile_enable(False)
        hist = [(p, b.cpu().numpy(), a.cpu().numpy(), s.cpu().numpy()) for p, b, a, s in hist]
        return prof, hist


def history_work(lib, hist, dims, chi_max, p, q, adaptive, mixed=False, times=1):
    """Work of every recorded sweep (times: how often each sweep ran).

    Problems with the same geometry add the same work, so each distinct
    (bond, bond dimensions, second pass) is evaluated once and weighted by
    its count."""
    from collections import Counter
    counts = Counter()
    for parity, before, after, status in hist:
        for c in range(before.shape[0]):
            for b in range(parity, len(dims) - 1, 2):
                counts[(b, int(before[c, b]), int(before[c, b + 1]), int(before[c, b + 2]),
                        int(after[c, b + 1]), int(status[c, b]) & 64, c == 0)] += times
    w = Work(lib)
    for (b, cl, cm, cr, cn, st, first), k in counts.items():
        one = Work(lib)
        one._cls = w._cls
        chi_b = np.zeros((1, len(dims) + 1), dtype=np.int64)
        chi_a = np.zeros((1, len(dims) + 1), dtype=np.int64)
        chi_b[0, b:b + 3] = (cl, cm, cr)
        chi_a[0, b + 1] = cn
        sta = np.zeros((1, len(dims) - 1), dtype=np.int64)
        sta[0, b] = st
        sweep_work(one, chi_b, chi_a, sta, b % 2, dims, chi_max, p, q, adaptive, mixed,
                   bonds=(b,), gate_bytes=first)
        for name, (fl, by) in one.k.items():
            w.add(name, k * fl, k * by)
        for name, (fl, by) in one.unpivoted.items():
            e = w.unpivoted.setdefault(name, [0.0, 0.0])
            e[0] += k * fl
            e[1] += k * by
    return w


# ---------------------------------------------------------------------------
def full_svd_tebd(torch, models, dims, hb, chains, chi_max, dt, steps, eps=1e-10, floor_=1e-14,
                  budget_s=150.0):
    """Torch-only TEBD with the vendor full SVD (torch.linalg.svd) on the GPU.

    Every sweep groups its (chain, bond) problems by shape; each group is one
    batched Theta contraction, gate product and SVD; the truncation rule,
    renormalisation and lambda^-1 reabsorption run on the device with masks.
    The new bond dimensions come back to the host once per sweep (to form the
    next sweep's groups).  Stops after budget_s seconds.  Returns (seconds,
    largest bond dimension, steps done)."""
    import numpy as np
    dev = "cuda"
    N = len(dims)
    dmax = max(dims)
    gam = torch.zeros((chains, N, dmax, chi_max, chi_max), dtype=torch.complex128, device=dev)
    lam = torch.zeros((chains, N + 1, chi_max), dtype=torch.float64, device=dev)
    gam[:, :, 0, 0, 0] = 1.0
    lam[:, :, 0] = 1.0      # lam[:, b + 1] is the bond b; lam[:, 0] and lam[:, N] are edges (1)
    chi = np.ones((chains, N + 1), dtype=np.int64)
    gh = torch.from_numpy(models.gate_stack(dims, hb, 0.5 * dt)).to(dev)
    gf = torch.from_numpy(models.gate_stack(dims, hb, dt)).to(dev)

    def sweep(parity, gates):
        groups = {}
        for c in range(chains):
            for b in range(parity, N - 1, 2):
                key = (dims[b], dims[b + 1], chi[c, b], chi[c, b + 1], chi[c, b + 2])
                groups.setdefault(key, []).append((c, b))
        new_chi = []
        for (dl, dr, cl, cm, cr), items in groups.items():
            ic = torch.tensor([x[0] for x in items], device=dev)
            ib = torch.tensor([x[1] for x in items], device=dev)
            G = len(items)
            gk = gam[ic, ib, :dl, :cl, :cm]
            gk1 = gam[ic, ib + 1, :dr, :cm, :cr]
            ll = lam[ic, ib, :cl]
            lm = lam[ic, ib + 1, :cm]
            lr = lam[ic, ib + 2, :cr]
            left = gk * (ll[:, None, :, None] * lm[:, None, None, :])
            right = gk1 * lr[:, None, None, :]
            th = torch.matmul(left.reshape(G, dl * cl, cm), right.permute(0, 2, 1, 3).reshape(
                G, cm, dr * cr).contiguous())                       # [(i a), (j c)]
            th = th.reshape(G, dl, cl, dr, cr).permute(0, 1, 3, 2, 4).reshape(G, dl * dr, cl * cr)
            g = gates[ib][:, :dl * dr, :dl * dr].contiguous()
            a = torch.matmul(g, th.contiguous()).reshape(G, dl, dr, cl, cr)
            a = a.permute(0, 1, 3, 2, 4).reshape(G, dl * cl, dr * cr)
            u, s, vh = torch.linalg.svd(a, full_matrices=False)
            K = min(s.shape[1], chi_max)
            s2 = s * s
            tot = s2.sum(-1, keepdim=True)
            tail = (tot - torch.cumsum(s2, -1)) / tot
            cp = torch.clamp((tail > eps).sum(-1) + 1, max=K)       # smallest c with w(c) <= eps
            keep = torch.arange(K, device=dev)[None, :] < cp[:, None]
            sk = torch.where(keep, s[:, :K], torch.zeros_like(s[:, :K]))
            nrm = torch.sqrt((sk * sk).sum(-1, keepdim=True))
            inv_l = torch.where(ll > floor_, 1.0 / ll, torch.zeros_like(ll))
            inv_r = torch.where(lr > floor_, 1.0 / lr, torch.zeros_like(lr))
            uk = u[:, :, :K] * keep[:, None, :]
            vk = vh[:, :K, :] * keep[:, :, None]
            gam[ic, ib] = 0
            gam[ic, ib + 1] = 0
            gam[ic, ib, :dl, :cl, :K] = uk.reshape(G, dl, cl, K) * inv_l[:, None, :, None]
            gam[ic, ib + 1, :dr, :K, :cr] = (vk.reshape(G, K, dr, cr).permute(0, 2, 1, 3)
                                              * inv_r[:, None, None, :])
            lam[ic, ib + 1] = 0
            lam[ic, ib + 1, :K] = sk / nrm
            new_chi.append((items, cp))
        got = torch.cat([cp for _, cp in new_chi]).cpu().numpy()
        i = 0
        for items, _ in new_chi:
            for (c, b) in items:
                chi[c, b + 1] = got[i]
                i += 1

    torch.cuda.synchronize()
    t0 = time.perf_counter()
    done = 0
    last = t0
    for _ in range(steps):
        sweep(0, gh)
        sweep(1, gf)
        sweep(0, gh)
        done += 1
        now = time.perf_counter()
        if now - last > 20.0:
            _progress(f"full-SVD comparator: {done} steps, {now - t0:.0f} s")
            last = now
        if now - t0 > budget_s:
            break
    torch.cuda.synchronize()
    return time.perf_counter() - t0, int(chi.max()), done


# ---------------------------------------------------------------------------
def _threads():
    try:
        from threadpoolctl import threadpool_info
        return max([x.get("num_threads", 1) for x in threadpool_info()] or [1])
    except Exception:
        return 1


def oracle_tebd_seconds(dims, hb_oracle, dt, chi_max, steps, levels, eps=1e-10):
    """FP64 oracle TEBD (full LAPACK SVD per bond) of one chain."""
    from oracle import models as om, mps as omps
    cache = {}

    def gfn(b, tau):
        if (b, tau) not in cache:
            cache[(b, tau)] = om.gate(hb_oracle[b], tau)
        return cache[(b, tau)]
    for b in range(len(dims) - 1):  # gates outside the timed sample
        gfn(b, 0.5 * dt), gfn(b, dt)
    drv = omps.TEBD(omps.basis_product_state(dims, levels), gfn, dt, chi_max, eps, method="full")
    t0 = time.perf_counter()
    for _ in range(steps):
        drv.step()
    return time.perf_counter() - t0, max(drv.mps.chis())


def cpu_baseline_spin_boson():
    from oracle import models as om
    N = SB["N"]
    dims, hb = om.spin_boson_chain(N, SB["d"], 1.0, 0.5, 1.0, 0.5)
    sec, chimax = oracle_tebd_seconds(dims, hb, SB["dt"], SB["chi_max"], SB["steps"], [0] * N)
    upd = SB["steps"] * updates_per_step(N)
    return {"value": round(upd / sec, 2), "unit": "bond updates/s", "cores": int(_threads()),
            "kind": "oracle",
            "sample": f"chain 0 of the same workload, all {SB['steps']} steps from the product state "
                      f"({upd} bond updates, {sec:.1f} s, max chi {chimax}); FP64, full LAPACK "
                      f"SVD per bond, one chain (the 16 chains of the GPU run differ only in "
                      f"their random test matrices)"}


# ---------------------------------------------------------------------------
def tfim_line(args, torch, api, models, lib):
    """Plain TEBD: open TFIM N = 20, chi_max = 32, dt = 0.01, 100 steps."""
    N = TFIM["N"]
    dims, hb = models.transverse_ising(N, 1.0, 1.0)
    ev = Evolution(torch, api, dims, hb, [0] * N, 1, TFIM["chi_max"], TFIM["p"], TFIM["q"],
                   TFIM["dt"], TFIM["eps"], TFIM["seed"])
    reps = max(3, args.steps)
    times = ev.timed(TFIM["steps"], reps, 1)
    upd = TFIM["steps"] * updates_per_step(N)
    out = {"metric": "TEBD bond updates/s", "value": round(upd * reps / sum(times), 2),
           "unit": "bond updates/s", "ms_per_evolution": round(1e3 * sum(times) / reps, 3),
           "repetitions": reps,
           "config": {"workload": "open transverse-field Ising chain N=20, J=h=1, |0...0>, "
                                  "dt=0.01, 100 symmetric Trotter steps (2900 bond updates), "
                                  "chi_max=32, RRSVD p=10 q=2, w<=1e-10, adaptive rank"}}
    prof, hist = ev.profiled(TFIM["steps"], lib)
    w = history_work(lib, hist, dims, TFIM["chi_max"], TFIM["p"], TFIM["q"], True)
    out["roofline"] = kernel_roofline(prof, w, "tfim_n20")
    out["chi_final_max"] = int(hist[-1][2].max())
    if not args.no_cpu_baseline:
        from oracle import models as om
        odims, ohb = om.tfim(N, 1.0, 1.0)
        sec, _ = oracle_tebd_seconds(odims, ohb, TFIM["dt"], TFIM["chi_max"], TFIM["steps"],
                                     [0] * N)
        out["cpu_baseline"] = {"value": round(upd / sec, 2), "unit": "bond updates/s",
                               "cores": int(_threads()), "kind": "oracle",
                               "sample": f"the whole evolution ({upd} bond updates, {sec:.2f} s), "
                                         f"FP64 full LAPACK SVD per bond"}
    return out


def batched_rrsvd_line(args, torch, api, wl, lib):
    """256 complex128 square matrices, n in {256, 512, 1024, 2048}, one call."""
    import numpy as np
    sizes = wl.batched_rrsvd_sizes()
    mats = wl.batched_rrsvd_matrices_device(sizes)
    api.rrsvd_truncate(mats, 64, 10, 2, 1e-10, 1504, 0)  # warm-up (workspace, code)
    torch.cuda.synchronize()
    reps = max(3, args.steps)
    times = []
    out = None
    for r in range(reps):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        out = api.rrsvd_truncate(mats, 64, 10, 2, 1e-10, 1504, r + 1)
        torch.cuda.synchronize()
        times.append(time.perf_counter() - t0)
    chi = out[3].cpu().numpy()
    lib.tebd_profile_enable(True)
    api.rrsvd_truncate(mats, 64, 10, 2, 1e-10, 1504, reps + 1)
    torch.cuda.synchronize()
    prof = lib.tebd_profile_read()
    lib.tebd_profile_enable(False)
    w = Work(lib)
    l = 74
    for n, c in zip(sizes, chi):
        w.add("k_frob", 0.0, 16.0 * n * n)
        w.rrsvd_pass(n, n, l, 2, False, int(c))
    if "k_form_uv<1>" in w.k:   # the standalone call writes plain U, V^H
        w.k["k_form_uv<0>"] = w.k.pop("k_form_uv<1>")
    sk_ms = sum(v[0] for k, v in prof.items()
                if k.startswith(("k_sketch<", "k_sketch_wide<", "k_sketch_split<")))
    sk_fl = sum(v[0] for k, v in w.k.items() if k.startswith("k_sketch<"))
    ach = sk_fl / (sk_ms * 1e-3) / 1e12 if sk_ms > 0 else None
    res = {"metric": "RRSVD truncations/s", "value": round(len(sizes) * reps / sum(times), 2),
           "unit": "truncations/s", "ms_per_batch": round(1e3 * sum(times) / reps, 3),
           "config": {"workload": "256 complex128 square matrices, n in {256,512,1024,2048} "
                                  "(seeded), A = U diag(exp(-i/25)) V^H with Haar U, V, k=64, "
                                  "p=10, q=2, one call"},
           "roofline": kernel_roofline(prof, w, "batched_rrsvd_256"),
           "sketch_gemms": {"bound": "mfma", "achieved": round(ach, 3) if ach else None,
                            "peak": PEAK_FP64_TFLOPS, "unit": "TFLOP/s",
                            "frac": round(ach / PEAK_FP64_TFLOPS, 4) if ach else None,
                            "event_ms": round(sk_ms, 3)},
           "kernel_ms": kernel_table(prof)}
    # the same batch with the sketch and power-iteration products in complex
    # FP32 (precision 1): rate and the change of the singular values
    api.rrsvd_truncate(mats, 64, 10, 2, 1e-10, 1504, 0, precision=1)
    torch.cuda.synchronize()
    tm = []
    for r in range(reps):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        outm = api.rrsvd_truncate(mats, 64, 10, 2, 1e-10, 1504, r + 1, precision=1)
        torch.cuda.synchronize()
        tm.append(time.perf_counter() - t0)
    s64, s32 = torch.stack(out[1]), torch.stack(outm[1])
    res["mixed_precision"] = {
        "value": round(len(sizes) * reps / sum(tm), 2), "unit": "truncations/s",
        "ms_per_batch": round(1e3 * sum(tm) / reps, 3),
        "vs_fp64": round(sum(times) / sum(tm), 3),
        "max_rel_sigma_diff_vs_fp64": float(((s64 - s32).abs().max(dim=1).values
                                             / s64[:, 0]).max().item()),
        "chi_identical": bool((out[3] == outm[3]).all().item()),
        "note": "precision 1: the sketch and power-iteration products on complex FP32 matrix "
                "cores (A read from its complex64 copy, the other operand rounded when "
                "staged), the QRs, B and the small SVD in FP64"}
    if not args.no_cpu_baseline:
        from oracle import philox, rrsvd as orr
        per = {}
        t_all = 0.0
        for n in sorted(set(sizes)):
            ts = []
            idx = [i for i, x in enumerate(sizes) if x == n][:8 if n < 2048 else 4]
            for i in idx:
                a = mats[i].cpu().numpy()
                om_ = philox.gaussian_omega(n, l, 1504, i, 0)
                t0 = time.perf_counter()
                orr.truncate_rrsvd(a, om_, 2, 64, 1e-10)
                ts.append(time.perf_counter() - t0)
            per[n] = float(np.mean(ts))
            t_all += per[n] * sizes.count(n)
        res["cpu_baseline"] = {"value": round(len(sizes) / t_all, 3), "unit": "truncations/s",
                               "cores": int(_threads()), "kind": "oracle",
                               "sample": "extrapolated: the oracle's step-by-step RRSVD (same "
                                         "algorithm, FP64, LAPACK QR and SVD) timed on the first 8 "
                                         "matrices of each size in the batch (4 at n=2048), mean "
                                         "seconds per size "
                                         + json.dumps({str(k): round(v, 4) for k, v in per.items()})
                                         + " times the count of each size in the batch"}
    return res


def _golden_mixed():
    path = os.path.join(ROOT, "tests", "golden", "spin_boson_n100_chi128.txt")
    z, lam = {}, {}
    for line in open(path):
        if line.startswith("#") or not line.strip():
            continue
        f = line.split()
        if f[0] == "obs":
            z[int(f[1])] = float(f[2])
        elif f[0] == "lam":
            lam[int(f[1])] = [float(x) for x in f[2:]]
    return z, lam


def mixed_line(args, torch, api, models, lib):
    """chi_max = 128 with complex FP32 sketch and power-iteration products."""
    import numpy as np
    from paper_1504_00992_amd import gradient
    N, d, chi_max, steps = SB["N"], SB["d"], 128, SB["steps"]
    dims, hb = models.spin_boson(N, d, 1.0, 0.5, 1.0, 0.5)
    zop = torch.zeros((d, d), dtype=torch.complex128, device="cuda")
    zop[0, 0], zop[1, 1] = 1.0, -1.0
    res = {}
    for prec in (1, 0):
        ev = Evolution(torch, api, dims, hb, [0] * N, args.chains, chi_max, SB["p"], SB["q"],
                       SB["dt"], SB["eps"], SB["seed"], precision=prec)
        times = ev.timed(steps, 1, 1)
        upd = steps * updates_per_step(N) * args.chains
        r = {"value": round(upd / times[0], 2), "lam": ev.mps.lam[0].cpu().numpy(),
             "chi": ev.mps.chi[0].cpu().numpy()}
        # <sigma_z> of chain 0 at every 50th step, from a replay
        ev.reset()
        zs = {}
        for s in range(1, steps + 1):
            ev.run(1)
            if s % 50 == 0:
                zs[s] = float(gradient.expectation(ev.mps.gamma[0], ev.mps.lam[0], zop, 0).item())
        r["z"] = zs
        if prec == 1:
            prof, hist = ev.profiled(steps, lib)
            w = history_work(lib, hist, dims, chi_max, SB["p"], SB["q"], True, mixed=True)
            r["roofline"] = kernel_roofline(prof, w, "spin_boson_16x100_chi128_mixed")
            import numpy as np
            st = np.concatenate([h[3][:, h[0]::2].ravel() for h in hist])
            r["gram_qr_fallbacks"] = {"bond_updates_refused": int(((st & 2) != 0).sum()),
                                      "bond_updates": int(st.size),
                                      "note": "updates whose QRs tried CholeskyQR2 (problems of "
                                              "QR size class 2 or 3) and fell back to Householder "
                                              "(kappa beyond ~1e7)"}
            f32 = {k: v for k, v in prof.items() if k.startswith("k_sketch_f32")}
            ms = sum(v[0] for v in f32.values())
            fl = sum(w.k.get(k, (0, 0))[0] for k in f32)
            r["f32_sketches"] = {"bound": "mfma", "achieved": round(fl / (ms * 1e-3) / 1e12, 4),
                                 "peak": PEAK_FP32_MFMA_TFLOPS, "unit": "TFLOP/s",
                                 "frac": round(fl / (ms * 1e-3) / 1e12 / PEAK_FP32_MFMA_TFLOPS, 5),
                                 "event_ms": round(ms, 3)} if ms > 0 else None
        res[prec] = r
    out = {"config": {"workload": f"{args.chains} spin-boson chains N=100 d=10, chi_max=128, "
                                  "dt=0.05, 200 steps from the product state, adaptive rank, "
                                  "sketch and power-iteration products in complex FP32 (FP32 "
                                  "MFMA, FP32 accumulation), QRs, B = Q^H A, small SVD in FP64"},
           "value": res[1]["value"], "fp64_value": res[0]["value"], "unit": "bond updates/s",
           "roofline": res[1]["roofline"], "f32_sketches": res[1]["f32_sketches"],
           "gram_qr_fallbacks": res[1]["gram_qr_fallbacks"]}
    try:
        gz, glam = _golden_mixed()
        chi = res[1]["chi"]
        errs = [float(np.max(np.abs(res[1]["lam"][b, :len(v)] - np.array(v))))
                for b, v in glam.items() if chi[b + 1] == len(v)]
        out["vs_fp64_oracle"] = {
            "bond_dims_identical": bool(all(chi[b + 1] == len(v) for b, v in glam.items())),
            "max_abs_lambda_err": max(errs) if errs else None,
            "max_abs_sigma_z_err": max(abs(res[1]["z"][s] - gz[s]) for s in gz),
            "reference": "tests/golden/spin_boson_n100_chi128.txt (chain 0, FP64 oracle with "
                         "the same Omega, written by tests/golden/make_golden.py)"}
        out["vs_gpu_fp64"] = {
            "max_abs_lambda_diff": float(np.max(np.abs(res[1]["lam"] - res[0]["lam"]))),
            "max_abs_sigma_z_diff": max(abs(res[1]["z"][s] - res[0]["z"][s]) for s in gz)}
    except OSError:
        out["vs_fp64_oracle"] = None
    return out


def adjoint_line(args, torch, api, models, wl, lib, reps=3):
    """Time per gradient of <Z_0(T)> w.r.t. the 39 couplings (XX + fields, N=40)."""
    import numpy as np
    from paper_1504_00992_amd import gradient
    n, steps, dt, chi_max = 40, 50, 0.02, 64
    J, h = wl.xx_couplings(n, seed=1504)
    dims, hb = models.xx_chain(J, h)
    hop = 0.5 * (np.kron(models.PAULI_X, models.PAULI_X) + np.kron(models.PAULI_Y, models.PAULI_Y))
    g_half = torch.from_numpy(models.gate_stack(dims, hb, 0.5 * dt)).cuda()
    g_full = torch.from_numpy(models.gate_stack(dims, hb, dt)).cuda()
    z = torch.tensor([[1.0, 0.0], [0.0, -1.0]], dtype=torch.complex128, device="cuda")

    def gradient_once():
        mps = api.DeviceMPS.product_state(1, dims, wl.neel_levels(n), chi_max)
        drv = gradient.CheckpointedTEBD(mps, g_half, g_full, chi_max, 10, 2, 1e-10, 1504,
                                        adaptive=2, checkpoint=10)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        drv.forward(steps)
        gam = mps.gamma[0].clone().requires_grad_(True)
        lam = mps.lam[0].clone().requires_grad_(True)
        gradient.expectation(gam, lam, z, 0).backward()
        torch.cuda.synchronize()
        t1 = time.perf_counter()
        gb = torch.zeros_like(mps.gamma)
        lb = torch.zeros_like(mps.lam)
        gb[0] = gam.grad
        lb[0] = lam.grad
        gh, gf, _, _ = drv.backward(gb, lb)
        torch.cuda.synchronize()
        t2 = time.perf_counter()
        gh, gf = gh.cpu().numpy(), gf.cpu().numpy()
        grad = np.array([gradient.coupling_gradient(gh[b], hb[b], 0.5 * dt, hop)
                         + gradient.coupling_gradient(gf[b], hb[b], dt, hop) for b in range(n - 1)])
        return grad, (t1 - t0, t2 - t1, time.perf_counter() - t2)

    gradient_once()
    timings = []
    grad = None
    for _ in range(reps):
        grad, t = gradient_once()
        timings.append(t)
    lib.tebd_profile_enable(True)
    gradient_once()
    torch.cuda.synchronize()
    prof = lib.tebd_profile_read()
    lib.tebd_profile_enable(False)
    # forward kernels: every sweep runs twice (forward, then its segment's
    # recorded replay); the bond dimensions of the plain run are the same
    ev = Evolution(torch, api, dims, hb, wl.neel_levels(n), 1, chi_max, 10, 2, dt, 1e-10, 1504)
    hist = []
    ev.reset()
    ev.run(steps, record=hist)
    hist = [(p, b.cpu().numpy(), a.cpu().numpy(), s.cpu().numpy()) for p, b, a, s in hist]
    w = history_work(lib, hist, dims, chi_max, 10, 2, True, times=2)
    ref = np.loadtxt(os.path.join(ROOT, "tests", "golden", "xx_n40_gradient.txt"))
    scale = float(np.max(np.abs(ref[:, 3])))
    fw, bw, host = (float(np.median([t[i] for t in timings])) for i in range(3))
    out = {"config": {"workload": "XX chain + random fields, N=40, J_b~U[0.8,1.2], h_i~U[-1,1], "
                                  "Neel start, 50 steps dt=0.02, chi_max=64, w<=1e-10, "
                                  "checkpoint every 10 steps; gradient of <Z_0(T=1)> w.r.t. "
                                  "all 39 J_b"},
           "metric": "gradients/s", "value": round(1.0 / (fw + bw + host), 3),
           "ms_per_gradient": round(1e3 * (fw + bw + host), 2),
           "forward_ms": round(1e3 * fw, 2), "reverse_ms": round(1e3 * bw, 2),
           "host_frechet_ms": round(1e3 * host, 2),
           "rel_err_vs_exact_svd_reverse": float(np.max(np.abs(grad - ref[:, 2])) / scale),
           "rel_err_vs_finite_differences": float(np.max(np.abs(grad - ref[:, 3])) / scale),
           "rel_err_vs_free_fermions": float(np.max(np.abs(grad - ref[:, 4])) / scale),
           "note": "errors relative to max|dL/dJ_b|; references in tests/golden/xx_n40_gradient.txt",
           "roofline": kernel_roofline(prof, w, "adjoint_xx_n40"),
           "kernel_ms": kernel_table(prof)}
    if not args.no_cpu_baseline:
        from oracle import adjoint as oadj, models as om, mps as omps
        dims_o, hb_o = om.xx_field(J, h)
        hop_o = 0.5 * (np.kron(om.X, om.X) + np.kron(om.Y, om.Y))
        cache = {}

        def gfn(b, tau):
            if (b, tau) not in cache:
                cache[(b, tau)] = om.gate(hb_o[b], tau)
            return cache[(b, tau)]
        m0 = omps.basis_product_state(dims_o, wl.neel_levels(n))
        t0 = time.perf_counter()
        oadj.tebd_gradient(m0, gfn, lambda b: hb_o[b], lambda b, k: hop_o if b == k else None,
                           n - 1, dt, steps, chi_max, 1e-10, om.Z, 0)
        sec = time.perf_counter() - t0
        out["cpu_baseline"] = {"value": round(1.0 / sec, 4), "unit": "gradients/s",
                               "cores": int(_threads()), "kind": "oracle",
                               "sample": f"one whole gradient ({sec:.1f} s): the oracle's FP64 "
                                         f"full-SVD TEBD and its reverse mode (every triplet "
                                         f"coupled), no checkpointing"}
    return out


# Table II of the paper (Sec. V.B): GPU-RRSVD seconds per matrix on a K20s,
# PCIe copies included, for its mixed-state Theta samples (context only).
PAPER_TABLE2_GPU_RRSVD_S = {900: 0.25, 1600: 0.41, 2500: 0.61, 3600: 0.88, 4900: 1.48}


def table2_line(args, torch, api, wl, lib):
    """Mixed-state Theta shapes (d^2 chi x d^2 chi, chi = 100, d = 3..7) at
    k = p = 100, q = 2: seconds per matrix, 8 matrices per call."""
    import numpy as np
    out = {"config": {"workload": "the mixed-state Theta shapes of the paper's timing table: "
                                  "n = 100 d^2 for d = 3..7 (900 ... 4900), 8 square complex128 "
                                  "matrices per call with the rank-300 spectrum exp(-i/30) "
                                  "(synthetic: the paper's sampled matrices are not available), "
                                  "RRSVD k = p = 100, q = 2, w <= 1e-10"},
           "unit": "s per matrix", "sizes": {}}
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1504)
    for n in sorted(PAPER_TABLE2_GPU_RRSVD_S):
        r = 300
        mats = []
        s_ = torch.exp(-torch.arange(r, dtype=torch.float64, device="cuda") / 30.0)
        for _ in range(8):
            u, _ = torch.linalg.qr(torch.randn((n, r), dtype=torch.complex128, device="cuda",
                                               generator=gen))
            v, _ = torch.linalg.qr(torch.randn((n, r), dtype=torch.complex128, device="cuda",
                                               generator=gen))
            mats.append(((u * s_[None, :]) @ v.conj().transpose(0, 1)).contiguous())
        api.rrsvd_truncate(mats, 100, 100, 2, 1e-10, 1504, 0)
        torch.cuda.synchronize()
        reps = 2
        t0 = time.perf_counter()
        for k in range(reps):
            res = api.rrsvd_truncate(mats, 100, 100, 2, 1e-10, 1504, k + 1)
        torch.cuda.synchronize()
        per = (time.perf_counter() - t0) / (reps * len(mats))
        lib.tebd_profile_enable(True)
        api.rrsvd_truncate(mats, 100, 100, 2, 1e-10, 1504, reps + 1)
        torch.cuda.synchronize()
        prof = lib.tebd_profile_read()
        lib.tebd_profile_enable(False)
        w = Work(lib)
        chi = res[3].cpu().numpy()
        for c in chi:
            w.add("k_frob", 0.0, 16.0 * n * n)
            w.rrsvd_pass(n, n, 200, 2, False, int(c))
        if "k_form_uv<1>" in w.k:
            w.k["k_form_uv<0>"] = w.k.pop("k_form_uv<1>")
        out["sizes"][str(n)] = {"value": round(per, 5),
                                "paper_gpu_rrsvd_s_k20s": PAPER_TABLE2_GPU_RRSVD_S[n],
                                "roofline": kernel_roofline(prof, w, f"table2_{n}")}
        del mats
        torch.cuda.empty_cache()
    return out


def tedopa_line(args, torch, api, lib):
    """A TEDOPA chain (Sec. III): Ohmic bath mapped to 99 oscillators."""
    from paper_1504_00992_amd import models, tedopa
    N = 100
    dims = [2] + [10] * 20 + [8] * 30 + [6] * 49
    t0, om_, hop = tedopa.chain_coefficients(tedopa.ohmic(0.1, 1.0, 2.0), 2.0, N - 1)
    _, hb = models.spin_boson_tedopa(dims, t0, om_, hop)
    ev = Evolution(torch, api, dims, hb, [0] * N, args.chains, 100, 10, 2, 0.05, 1e-10, 1504)
    times = ev.timed(SB["steps"], 1, 1)
    upd = SB["steps"] * updates_per_step(N) * args.chains
    return {"config": {"workload": f"{args.chains} TEDOPA chains: spin + 99 oscillators from the "
                                   "Ohmic spectral density J = 2 pi alpha omega (alpha = 0.1, "
                                   "omega_c = 2) mapped by orthogonal polynomials, truncations "
                                   "10/8/6 along the chain, dt = 0.05, 200 steps, chi_max = 100"},
            "value": round(upd / times[0], 2), "unit": "bond updates/s",
            "ms_per_evolution": round(1e3 * times[0], 2),
            "chain": {"t0": round(t0, 6), "omega_first": [round(x, 6) for x in om_[:3]],
                      "t_first": [round(x, 6) for x in hop[:3]]},
            "chi_final_max": int(ev.mps.chi.max().item())}


def accuracy_line(args, torch, api, models, lib, ref_ev):
    """The headline evolution with the Accuracy Check (adaptive rank 3)."""
    from paper_1504_00992_amd import gradient
    N = SB["N"]
    dims, hb = models.spin_boson(N, SB["d"], 1.0, 0.5, 1.0, 0.5)
    ev = Evolution(torch, api, dims, hb, [0] * N, args.chains, SB["chi_max"], SB["p"], SB["q"],
                   SB["dt"], SB["eps"], SB["seed"], adaptive=3)
    times = ev.timed(SB["steps"], 1, 1)
    upd = SB["steps"] * updates_per_step(N) * args.chains
    zop = torch.zeros((SB["d"], SB["d"]), dtype=torch.complex128, device="cuda")
    zop[0, 0], zop[1, 1] = 1.0, -1.0
    za = float(gradient.expectation(ev.mps.gamma[0], ev.mps.lam[0], zop, 0).item())
    zb = float(gradient.expectation(ref_ev.mps.gamma[0], ref_ev.mps.lam[0], zop, 0).item())
    st = ev.drv.ws.status.cpu().numpy()
    return {"config": {"workload": "the headline evolution (16 spin-boson chains, N=100, d=10, "
                                   "chi_max=100, 200 steps) with the Accuracy Check of Sec. IV "
                                   "(Alg. 2): sketch from chi + p columns, probes of p = 10 "
                                   "columns against sqrt(eps) ||A||_F / ((10/3) pi)"},
            "value": round(upd / times[0], 2), "unit": "bond updates/s",
            "ms_per_evolution": round(1e3 * times[0], 2),
            "chi_final_max": int(ev.mps.chi.max().item()),
            "capped_bonds_last_sweep": int(((st & 128) != 0).sum()),
            "sigma_z_chain0_vs_two_stage_rank": abs(za - zb)}


def order4_line(args, torch, api, models, lib):
    """Fourth-order Trotter steps (15 sweeps each) on the headline chains."""
    from paper_1504_00992_amd import gradient
    N = SB["N"]
    dims, hb = models.spin_boson(N, SB["d"], 1.0, 0.5, 1.0, 0.5)
    steps, dt = 50, 0.2  # the same T = 10 as 200 steps of 0.05
    mps = api.DeviceMPS.product_state(args.chains, dims, [0] * N, SB["chi_max"])
    drv = api.TEBD(mps, hb, dt, SB["chi_max"], p=10, q=2, trunc_eps=1e-10, seed=1504,
                   adaptive=2, order=4)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        drv.step()
    torch.cuda.synchronize()
    sec = time.perf_counter() - t0
    upd = steps * 5 * updates_per_step(N) * args.chains
    return {"config": {"workload": "16 spin-boson chains N=100 d=10, chi_max=100, Suzuki "
                                   "fourth-order steps of dt = 0.2 (15 sweeps each) to T = 10"},
            "value": round(upd / sec, 2), "unit": "bond updates/s",
            "ms_per_evolution": round(1e3 * sec, 2),
            "chi_final_max": int(mps.chi.max().item())}


# ---------------------------------------------------------------------------
# rocprofv3 post-processing (host only)
COPY_PROBE_BYTES = 256 << 20


def short_kernel_name(n):
    """Kernel name without 'void', the tebd:: namespace and the argument list."""
    n = re.sub(r"^void ", "", n)
    if n.startswith("tebd::"):
        n = n[6:]
    depth = 0
    for i, ch in enumerate(n):
        if ch == "<":
            depth += 1
        elif ch == ">":
            depth -= 1
        elif ch == "(" and depth == 0:
            return n[:i]
    return n


def summarize_trace(db, command):
    """Per-kernel calls, total and mean duration (us) from a rocprofv3
    --kernel-trace results database (its `kernels` view): the library's
    kernels (k_*) one by one, every other kernel (input generation and copies
    by torch or its libraries, outside the timed regions) in one line."""
    import sqlite3
    con = sqlite3.connect(db)
    rows = con.execute("select name, count(*), sum(duration), avg(duration) from kernels "
                       "group by name order by sum(duration) desc").fetchall()
    merged = {}
    for name, n, tot, _ in rows:
        k = short_kernel_name(name)
        a = merged.get(k, (0, 0.0))
        merged[k] = (a[0] + n, a[1] + tot)
    ours = {k: v for k, v in merged.items() if k.startswith("k_")}
    rest = [v for k, v in merged.items() if not k.startswith("k_")]
    total = sum(v[1] for v in ours.values()) or 1.0
    out = ["# rocprofv3 --kernel-trace --stats summary (durations in microseconds; kernel names "
           "without namespace and arguments; pct of the library's kernel time)",
           f"# command: {command}",
           f"# {'kernel':<44} {'calls':>7} {'total_us':>12} {'avg_us':>9} {'pct':>6}"]
    for k, (n, tot) in sorted(ours.items(), key=lambda kv: -kv[1][1]):
        nm = k if len(k) <= 46 else k[:43] + "..."
        out.append(f"{nm:<46} {n:>7} {tot / 1e3:>12.1f} {tot / 1e3 / n:>9.2f} "
                   f"{100 * tot / total:>6.2f}")
    if rest:
        n, tot = sum(v[0] for v in rest), sum(v[1] for v in rest)
        out.append(f"# other kernels (inputs, copies; not the library's): {n} calls, "
                   f"{tot / 1e3:.1f} us")
    return "\n".join(out) + "\n"


def _counter_means(path, counter):
    """Per-kernel (dispatches, mean value) of one counter from a rocprofv3
    counter-collection CSV."""
    import csv
    acc = {}
    with open(path) as f:
        for row in csv.DictReader(f):
            if row["Counter_Name"] != counter:
                continue
            k = short_kernel_name(row["Kernel_Name"])
            a = acc.get(k, (0, 0.0))
            acc[k] = (a[0] + 1, a[1] + float(row["Counter_Value"]))
    return {k: (n, s / n) for k, (n, s) in acc.items()}


def summarize_traffic(fetch_csv, write_csv, probe_fetch_csv, probe_write_csv, command):
    """HBM bytes per launch of every kernel: FETCH_SIZE and WRITE_SIZE (KiB
    per dispatch), each scaled by COPY_PROBE_BYTES over what the same counter
    reads for the copy probe's kernel (the dispatch with the largest value)."""
    pf = max(_counter_means(probe_fetch_csv, "FETCH_SIZE").values(), key=lambda v: v[1])[1]
    pw = max(_counter_means(probe_write_csv, "WRITE_SIZE").values(), key=lambda v: v[1])[1]
    sf, sw = COPY_PROBE_BYTES / (1024.0 * pf), COPY_PROBE_BYTES / (1024.0 * pw)
    fe, wr = _counter_means(fetch_csv, "FETCH_SIZE"), _counter_means(write_csv, "WRITE_SIZE")
    out = ["# HBM traffic per kernel launch from rocprofv3 --pmc FETCH_SIZE and --pmc WRITE_SIZE "
           "(two runs of the command below), KiB per dispatch, scaled by the copy probe",
           f"# command: {command}",
           f"# copy probe (bench.py --copy-probe, {COPY_PROBE_BYTES} bytes read and written): "
           f"FETCH_SIZE {pf:.1f} KiB, WRITE_SIZE {pw:.1f} KiB per dispatch; scale factors "
           f"{sf:.4f} (fetch), {sw:.4f} (write)",
           f"# kernel sources sha256: {code_digest()}",
           "# kernel dispatches FETCH_KiB WRITE_KiB bytes_per_launch"]
    for k in sorted(fe, key=lambda k: -fe[k][0] * fe[k][1]):
        n, f = fe[k]
        w = wr.get(k, (0, 0.0))[1]
        out.append(f"{k} {n} {f:.2f} {w:.2f} {1024.0 * (f * sf + w * sw):.0f}")
    return "\n".join(out) + "\n"


def main():
    args = parse()
    if args.summarize_trace or args.summarize_traffic:
        text = (summarize_trace(args.summarize_trace, args.command) if args.summarize_trace
                else summarize_traffic(*args.summarize_traffic, args.command))
        path = args.out or (os.path.join(ROOT, "profiles", f"{args.workload}_hbm_traffic.txt")
                            if args.summarize_traffic else None)
        if path:
            with open(path, "w") as f:
                f.write(text)
        else:
            sys.stdout.write(text)
        return
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (got --gpus {args.gpus}): this build measures one "
              f"GPU's share of the workload; the multi-GPU layout is described, not launched.",
              file=sys.stderr)
        sys.exit(2)
    import numpy as np
    import torch
    if not torch.cuda.is_available():
        print("bench.py needs a HIP device", file=sys.stderr)
        sys.exit(1)
    if args.copy_probe:
        src = torch.ones((256 << 20) // 8, dtype=torch.float64, device="cuda")
        dst = torch.empty_like(src)
        torch.cuda.synchronize()
        for _ in range(3):
            torch.mul(src, 1.0, out=dst)  # an elementwise kernel: reads and writes 256 MiB
        torch.cuda.synchronize()
        print(json.dumps({"copy_probe_bytes": COPY_PROBE_BYTES, "copies": 3}))
        return
    from paper_1504_00992_amd import api, autotune, models, _lib
    import workloads as wl
    _lib.load()
    # tile shapes of the sketch products: the autotune cache (timed once per
    # box, then read from its JSON file)
    t0 = time.perf_counter()
    tuned = autotune.load()
    source = "cache " + autotune.cache_path()
    if not tuned:
        tuned = autotune.tune()
        source = "timed now, saved to " + autotune.cache_path()
    tune_entry = {"entries": tuned, "source": source, "seconds": round(time.perf_counter() - t0, 2)}
    _progress(f"autotune: {[(e['rows'], e['width'], e['variant']) for e in tuned]}")
    if args.only:
        args.no_cpu_baseline = True
        fn = {"tfim": lambda: tfim_line(args, torch, api, models, _lib),
              "batched": lambda: batched_rrsvd_line(args, torch, api, wl, _lib),
              "mixed": lambda: mixed_line(args, torch, api, models, _lib),
              "adjoint": lambda: adjoint_line(args, torch, api, models, wl, _lib),
              "table2": lambda: table2_line(args, torch, api, wl, _lib)}[args.only]
        print(json.dumps({"only": args.only, args.only: fn()}), flush=True)
        return

    adaptive = args.rank == "adaptive"
    N, steps = SB["N"], SB["steps"]
    dims, hb = models.spin_boson(N, SB["d"], 1.0, 0.5, 1.0, 0.5)
    ev = Evolution(torch, api, dims, hb, [0] * N, args.chains, SB["chi_max"], SB["p"], SB["q"],
                   SB["dt"], SB["eps"], SB["seed"], adaptive=2 if adaptive else 0)
    # the sweep table's entry for this evolution's capacities (d chi_max rows,
    # chi_max + p width) is tuned on the evolution itself (untimed runs)
    if not any(e.get("workload") == "spin_boson_16x100" for e in tuned):
        t1 = time.perf_counter()
        cap = ((SB["d"] * SB["chi_max"], SB["chi_max"] + SB["p"]),)
        wl_entries = autotune.tune_workload(lambda: ev.timed(steps, 1, 0), "spin_boson_16x100",
                                            buckets=cap, precision=autotune.SWEEP_TABLE)
        tune_entry["workload_entries"] = wl_entries
        tune_entry["workload_seconds"] = round(time.perf_counter() - t1, 2)
        _progress(f"autotune on the evolution: variant {wl_entries[0]['variant']} "
                  f"({wl_entries[0]['workload_s']} s per evolution for variants {list(autotune.VARIANTS)})")
    times = ev.timed(steps, args.steps, args.warmup)
    sec = sum(times)
    per_rep = steps * updates_per_step(N) * args.chains
    _progress(f"timed evolutions: {', '.join(f'{t:.3f}' for t in times)} s")
    line = {
        "metric": METRIC,
        "value": round(per_rep * args.steps / sec, 2),
        "unit": "bond updates/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(1e3 * sec / args.steps, 3),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "c128 (f64)",
        "data": "synthetic",
        "config": {"workload": f"batched TEBD: {args.chains} chain-mapped spin-boson chains, "
                               "N=100 (spin + 99 oscillators, d=10), t_n=0.5, w_n=1, dt=0.05, "
                               "chi_max=100, RRSVD p=10 q=2, w<=1e-10 per bond; one step = the "
                               "whole evolution, Trotter steps 1..200 from the product state "
                               f"({per_rep} bond updates)",
                   "rank": ("two-stage adaptive: k1 = chi + max(4, chi/4), k = chi_max when the "
                            "Frobenius residual needs it (second pass skipped on the host when no "
                            "bond needs it)" if adaptive else "fixed k = chi_max"),
                   "chains": args.chains, "trotter_steps": steps,
                   "chi_final_max": int(ev.mps.chi.max().item()),
                   "status_bits_seen": sorted(set(int(x) for x in
                                                  np.unique(ev.drv.ws.status.cpu().numpy())))},
        "rep_ms": [round(1e3 * t, 3) for t in times],
        "autotune": tune_entry,
    }
    if not args.no_profile:
        prof, hist = ev.profiled(steps, _lib)
        w = history_work(_lib, hist, dims, SB["chi_max"], SB["p"], SB["q"], adaptive)
        line["roofline"] = kernel_roofline(prof, w, "spin_boson_16x100")
        line["kernel_rooflines"] = kernel_rooflines(prof, w, "spin_boson_16x100")
        # the gate product (one per group of chains sharing a gate): HBM bytes
        # per launch, algorithmic against the counters' (when taken on these
        # kernel sources)
        gl = prof.get("k_gate", (0.0, 0))[1]
        if gl:
            alg = w.k.get("k_gate", (0.0, 0.0))[1] / gl
            meas, _ = measured_traffic("k_gate", "spin_boson_16x100")
            line["gate_hbm"] = {"algorithmic_bytes_per_launch": round(alg),
                                "measured_bytes_per_launch": round(meas) if meas else None,
                                "measured_over_algorithmic": round(meas / alg, 3)
                                if meas and alg else None}
        line["phase_ms"] = phase_table(prof)
        line["kernel_ms"] = kernel_table(prof)
        line["profiled_phase_ms_total"] = round(sum(v[0] for k, v in prof.items()
                                                    if not k.startswith("k_")), 3)
        _progress("profiled evolution done")
    if not args.no_other_rank:
        other = Evolution(torch, api, dims, hb, [0] * N, args.chains, SB["chi_max"], SB["p"],
                          SB["q"], SB["dt"], SB["eps"], SB["seed"], adaptive=0 if adaptive else 2)
        ot = other.timed(steps, 1, 0)
        line["other_rank_mode"] = {
            "rank": "fixed k = chi_max" if adaptive else "two-stage adaptive",
            "value": round(per_rep / ot[0], 2), "unit": "bond updates/s",
            "ms_per_step": round(1e3 * ot[0], 3),
            "chi_final_max": int(other.mps.chi.max().item())}
        del other
        torch.cuda.empty_cache()
        _progress(f"other rank mode: {ot[0]:.2f} s")
    if not args.no_graph and adaptive:
        gev = Evolution(torch, api, dims, hb, [0] * N, args.chains, SB["chi_max"], SB["p"],
                        SB["q"], SB["dt"], SB["eps"], SB["seed"], adaptive=1)
        t0 = time.perf_counter()
        graph = api.GraphTEBD(gev.drv, steps, steps_per_graph=25)
        cap = time.perf_counter() - t0
        gt = []
        for r in range(args.warmup + args.steps):
            gev.reset()
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            graph.replay()
            torch.cuda.synchronize()
            if r >= args.warmup:
                gt.append(time.perf_counter() - t0)
        same = (torch.equal(gev.mps.gamma, ev.mps.gamma) and torch.equal(gev.mps.lam, ev.mps.lam)
                and torch.equal(gev.mps.chi, ev.mps.chi))
        gval = per_rep * len(gt) / sum(gt)
        line["graph_replay"] = {
            "value": round(gval, 2), "unit": "bond updates/s",
            "ms_per_step": round(1e3 * sum(gt) / len(gt), 3),
            "vs_host_skip_mode": round(gval / line["value"], 4),
            "graphs": len(graph.graphs), "capture_s": round(cap, 2),
            "bitwise_equal_to_timed_run": bool(same),
            "note": "the same 200-step evolution captured in HIP graphs (25 steps each) with the "
                    "adaptive rank's second pass skipped on the device, replayed from the product "
                    "state; the headline value skips it on the host after one read per sweep"}
        del graph, gev
        torch.cuda.empty_cache()
        _progress(f"graph replay: {sum(gt) / len(gt):.3f} s per evolution")
    if not args.no_full_svd:
        fsec, fchi, fdone = full_svd_tebd(torch, models, dims, hb, args.chains, SB["chi_max"],
                                          SB["dt"], steps)
        fupd = fdone * updates_per_step(N) * args.chains
        line["full_svd"] = {"value": round(fupd / fsec, 2), "unit": "bond updates/s",
                            "seconds": round(fsec, 2), "trotter_steps": f"1..{fdone}",
                            "chi_final_max": fchi,
                            "note": "vendor full SVD (torch.linalg.svd) in a torch-only TEBD on "
                                    "the same GPU: every same-shape bond of a sweep in one batched "
                                    "call, truncation and reabsorption on the device, the same "
                                    "evolution of all chains from the product state (stopped "
                                    "after 150 s if unfinished: its later, larger steps would "
                                    "only lower its rate)"}
        line["speedup_vs_full_svd"] = round(line["value"] / line["full_svd"]["value"], 3)
        _progress(f"full-SVD comparator: {fsec:.1f} s")
    if not args.no_tfim:
        line["tfim"] = tfim_line(args, torch, api, models, _lib)
        _progress("tfim done")
    if not args.no_batched:
        line["batched_rrsvd"] = batched_rrsvd_line(args, torch, api, wl, _lib)
        _progress("batched RRSVD done")
    if not args.no_mixed:
        line["mixed_precision"] = mixed_line(args, torch, api, models, _lib)
        _progress("mixed precision done")
    if not args.no_adjoint:
        line["adjoint"] = adjoint_line(args, torch, api, models, wl, _lib)
        _progress("adjoint done")
    if not args.no_accuracy:
        line["accuracy_check"] = accuracy_line(args, torch, api, models, _lib, ev)
        line["accuracy_check"]["vs_two_stage_rank"] = round(
            line["accuracy_check"]["value"] / line["value"], 4)
        torch.cuda.empty_cache()
        _progress("accuracy check done")
    if not args.no_order4:
        line["order4"] = order4_line(args, torch, api, models, _lib)
        torch.cuda.empty_cache()
        _progress("order 4 done")
    if not args.no_tedopa:
        line["tedopa"] = tedopa_line(args, torch, api, _lib)
        torch.cuda.empty_cache()
        _progress("tedopa done")
    if not args.no_table2:
        line["table2_mixed_state"] = table2_line(args, torch, api, wl, _lib)
        _progress("table 2 shapes done")
    if not args.no_cpu_baseline:
        line["cpu_baseline"] = cpu_baseline_spin_boson()
        _progress("cpu baseline done")
    print(json.dumps(line), flush=True)


if __name__ == "__main__":
    main()
