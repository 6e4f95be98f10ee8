"""The work a program gives this framework, as cases that can be timed and checked.

A case is a dict of plain values. ``op`` says which entry points a pass calls, the
rest describes the particle set (``set``, ``n``, ``order``, the record kind ``rec``),
the storage formats (``store``), the smoothing kernel and the launch options a program
picks (``cells``, ``sub_bits``, ``tile``, ``sched``, ``split``, ``keep``). All particle sets are
synthetic and made on the GPU from the seed, with the recipes of
``paper_2512_05516_amd/inputs.py``: jittered lattices with h = eta dx, and a uniform
background with eight Gaussian blobs whose h follows the number density.
"""
import math

import numpy as np
import torch

from paper_2512_05516_amd import inputs, serve, sphmi
from paper_2512_05516_amd.pipeline import Pipeline

ETA, GAMMA = inputs.ETA, 5.0 / 3.0
ALPHA, BETA = 0.8, 3.0
DT = 1e-4
F_BLOB, SIGMA, NBLOBS = 0.19, 0.03, 8
PAIRS = 48                       # neighbours within H at the resolution eta

# op, particle set and launch options of a program that tuned nothing
PLAIN = {"set": "lattice", "n": 4096, "order": "blocked", "rec": "f32", "store": "f32",
         "kernel": "m4", "cells": "buffers", "sub_bits": 0, "tile": "", "sched": "", "split": False, "keep": False}


def _case(name, op, **kw):
    return {"name": name, "op": op, **PLAIN, **kw}


def listed():
    return [
        # a program's smallest step, everything at its defaults: launches and latency
        _case("step_small", "step", n=4096, order="shuffled"),
        # the benchmark's step: 128^3 lattice, tuned tiles, cell list kept between steps
        _case("step_lattice128", "step", n=2097152, sub_bits=1, tile="64x1", sched="grid",
              keep=True),
        # the largest step: cells of very uneven occupancy, loops split by occupancy,
        # list rebuilt every step
        _case("step_clustered4m", "step", set="clustered", n=4194304, sub_bits=2, tile="32x2",
              sched="grid", split=True),
        # the density loop as a program calls it first: no tile, no work list
        # (cells as small as the support radius allows, about 12 particles each)
        _case("density_default", "density", n=884736, order="shuffled", cells="tight"),
        # the force loop the same way, cells that hold buffers of 64
        _case("force_default", "force", n=884736, order="shuffled"),
        # density with FP16 storage on uneven cells, an odd particle count
        _case("density_clustered_fp16", "density", set="clustered", n=750019, store="fp16_store",
              sub_bits=2, tile="32x2", sched="grid"),
        # force on uneven cells
        _case("force_clustered", "force", set="clustered", n=1500007, sub_bits=2, tile="64x1",
              sched="grid"),
        # plain records without a conversion, FP64 records, Wendland kernel
        _case("aos_step_f64", "aos_step", n=262144, rec="f64", kernel="wendland_c2", sub_bits=1,
              tile="64x2", sched="grid"),
        # records in random order brought into cell order and back, all-FP16 storage
        _case("reorder_f64", "reorder", set="uniform", n=1500007, order="shuffled", rec="f64",
              store="fp16_all", sub_bits=1),
        # what streams over the slots: reductions, totals and the Courant step, kick and drift
        _case("linear", "linear", set="uniform", n=3000017),
        # smoothing lengths adapted to the density, from the records' start values
        _case("smoothing_length", "hiter", set="clustered", n=262144, sub_bits=2, tile="32x2",
              sched="grid"),
        # a burst of cell-pair tasks served over resident state
        _case("serve_burst", "serve", set="clustered", n=200003),
    ]


def draw(rng):
    op = rng.choice(["step", "step", "density", "force", "force", "aos_step", "reorder", "linear",
                     "hiter", "serve"])
    hi = {"step": 21, "density": 21, "force": 21, "aos_step": 19.5, "reorder": 21, "linear": 22,
          "hiter": 18.5, "serve": 18.5}[op]
    n = int(2 ** rng.uniform(15 if op == "serve" else 12, hi)) | rng.randint(0, 1)
    case = dict(PLAIN, op=op, set=rng.choice(["lattice", "clustered"]),
                order=rng.choice(["blocked", "shuffled"]), rec=rng.choice(["f32", "f32", "f64"]),
                store=rng.choice(["f32", "f32", "fp16_store", "fp16_all", "bf16_all"]),
                kernel=rng.choice(["m4", "m4", "wendland_c2"]),
                cells=rng.choice(["buffers", "tight"]))
    if op in ("hiter", "serve") or (op == "linear"):
        case.update(store="f32", kernel="m4")
    if op in ("reorder", "linear"):
        case["set"] = "uniform"
    if op in ("hiter", "serve"):
        case["set"] = "clustered"
    if case["set"] == "lattice":
        n = max(4, round(n ** (1 / 3) / 4)) * 4
        n = n ** 3
    case["n"] = n
    sb, tile, sched = rng.choice([(0, "", ""), (0, "", ""), (1, "64x1", "grid"), (1, "64x1", ""),
                                  (1, "64x2", "grid"), (2, "32x2", "grid"), (2, "64x1", "grid"),
                                  (1, "64x4", "static"), (2, "32x8", "grid"),
                                  (0, "128x2", "dynamic"), (2, "16x4", "grid")])
    case.update(sub_bits=sb, tile=tile, sched=sched)
    if op in ("step", "density", "force") and case["set"] == "clustered" and sched == "grid":
        case["split"] = rng.random() < 0.5
    if op == "serve":
        case.update(sub_bits=0, tile="", sched="")
    return case


# --- inputs ------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _gamma_k(case):
    return sphmi.GAMMA_K[sphmi.KERNELS[case["kernel"]]]


def _particles(case, seed):
    """x (n, 3) in [0, 1), v (n, 3), h (n,) in FP64, in input order; u = 1, m = 1/n."""
    n, g = case["n"], _gen(seed)
    rand = lambda *s: torch.rand(*s, generator=g, device="cuda", dtype=torch.float64)
    randn = lambda *s: torch.randn(*s, generator=g, device="cuda", dtype=torch.float64)
    if case["set"] == "lattice":
        side = round(n ** (1 / 3))
        k = torch.arange(side, device="cuda")
        gz, gy, gx = torch.meshgrid(k, k, k, indexing="ij")
        site = torch.stack([gx.reshape(-1), gy.reshape(-1), gz.reshape(-1)], 1)
        x = (site + 0.5 + 0.2 * (rand(n, 3) - 0.5)) / side
        h = torch.full((n,), ETA / side, device="cuda", dtype=torch.float64)
        grid = side // 4
    elif case["set"] == "uniform":
        x = rand(n, 3)
        h = torch.full((n,), ETA * n ** (-1 / 3), device="cuda", dtype=torch.float64)
        grid = 16
    else:
        nb = int(round(F_BLOB * n)) // NBLOBS
        c = rand(NBLOBS, 3)
        blob = (c[:, None, :] + SIGMA * randn(NBLOBS, nb, 3)).reshape(-1, 3)
        x = torch.cat([rand(n - nb * NBLOBS, 3), blob])
        x = x - x.floor()
        dens = torch.full((n,), n * (1 - F_BLOB), device="cuda", dtype=torch.float64)
        norm = n * F_BLOB / NBLOBS / ((2 * math.pi) ** 1.5 * SIGMA ** 3)
        for q in range(NBLOBS):
            d = x - c[q]
            d = d - d.round()
            dens += norm * torch.exp(-0.5 * (d * d).sum(1) / SIGMA ** 2)
        h = ETA * dens ** (-1 / 3)
        grid = 16
    x = torch.where(x >= 1.0, torch.zeros_like(x), x)
    v = 0.01 * randn(n, 3)
    if case["order"] == "shuffled":
        p = torch.argsort(rand(n))
    else:                                    # buffers of co-located particles
        b = (x * grid).long().clamp(max=grid - 1)
        p = torch.argsort((b[:, 2] * grid + b[:, 1]) * grid + b[:, 0], stable=True)
    return x[p], v[p], h[p]


def _n_c(case, h):
    """Cells per axis: cells that hold about 64 particles where these are spread evenly
    ("buffers"), else as small as the largest support radius allows (an h iteration has
    1.6 times that, so that h can grow)."""
    if case["cells"] == "buffers" and case["set"] != "clustered":
        return max(3, round(case["n"] ** (1 / 3)) // 4)
    room = 1.6 if case["op"] == "hiter" else 1.0
    return max(3, int(math.floor(1.0 / (room * _gamma_k(case) * float(h.float().max())))))


def _columns(buf, rec):
    """The record buffer as (n, words) views of its FP64, FP32 and int32 words."""
    words = rec.itemsize // 4
    return (buf.view(torch.float64).view(-1, words // 2), buf.view(torch.float32).view(-1, words),
            buf.view(torch.int32).view(-1, words))


def _field(buf, rec, name):
    """A field of the records on the device, as a strided view."""
    dt, off = rec.fields[name][:2]
    base, comps = (dt.base, dt.shape[0]) if dt.shape else (dt, 1)
    d, f, i = _columns(buf, rec)
    col = {"<f8": d, "<f4": f, "<i4": i}[np.dtype(base).str]
    at = off // base.itemsize
    return col[:, at:at + comps] if dt.shape else col[:, at]


def _records(case, seed):
    rec = inputs.AOS_F32 if case["rec"] == "f32" else inputs.AOS_F64
    x, v, h = _particles(case, seed)
    n = case["n"]
    buf = torch.zeros(n * rec.itemsize, dtype=torch.uint8, device="cuda")
    buf.view(torch.int64).view(n, -1)[:, 0] = torch.arange(n, device="cuda")
    _field(buf, rec, "x").copy_(x)
    _field(buf, rec, "v").copy_(v)
    _field(buf, rec, "m").fill_(1.0 / n)
    _field(buf, rec, "h").copy_(h)
    _field(buf, rec, "u").fill_(1.0)
    return buf.cpu().numpy().view(rec), _n_c(case, h)


def _precision(case):
    a = sphmi.ANCHOR_SUB(2)
    return {"f32": lambda: sphmi.precision(),
            "fp16_store": lambda: sphmi.precision("f16", "bf16", "f16", 21, 7, 0, a),
            "fp16_all": lambda: sphmi.precision("f16", "f16", "f16", 21, 7, 0, a),
            "bf16_all": lambda: sphmi.precision("bf16", "bf16", "bf16", 0, 0, 0, a)}[case["store"]]()


def _pipeline(case, seed):
    rec, n_c = _records(case, seed)
    kw = {}
    if case["tile"]:
        kw["til"] = sphmi.tile(*(int(t) for t in case["tile"].split("x")))
    if case["split"]:
        # sparse cells merged along x, the others with the loop's own tile
        kw["split"] = {"density": (48, (32, 2), "grid", 4), "force": (48, (64, 2), "grid", 4)}
        kw["til_force"] = sphmi.tile(64, 1)
    return Pipeline(rec, n_c, prec=_precision(case), prm=sphmi.params(kernel=case["kernel"]),
                    sub_bits=case["sub_bits"], sched=case["sched"] or None,
                    keep_cells=case["keep"], **kw)


TASK_ROWS = 20000                # slots of either kind in a burst


def _tasks(start, n_c, seed):
    """A burst of cell-pair tasks, density first, then force, TASK_ROWS slots of each."""
    t = serve.make_tasks(start, n_c, 3000, seed)
    out = []
    for kind in (0, 1):
        part = t[t[:, 0] == kind]
        end = np.cumsum(part[:, 4] - part[:, 3])
        part = part[: int(np.searchsorted(end, TASK_ROWS)) + 1].copy()
        part[-1, 4] -= int((part[:, 4] - part[:, 3]).sum()) - TASK_ROWS
        out.append(part)
    return np.concatenate(out)


class _Served:
    """A server with the burst of tasks a pass submits and the pinned result records."""

    def __init__(self, pipe, seed):
        tasks = _tasks(pipe.cells.cell_start.cpu().numpy(), pipe.n_c, seed)
        self.buf = torch.zeros(2 * TASK_ROWS * serve.RESULT.itemsize, dtype=torch.uint8,
                               pin_memory=True)
        self.req, _ = serve.requests(tasks, 0, self.buf.data_ptr())
        self.out = self.buf.numpy().view(serve.RESULT)
        torch.cuda.synchronize()
        self.server = serve.Server(pipe)

    def __del__(self):
        if hasattr(self, "server"):
            self.server.close()


def _rates(n, seed):
    """Rates and neighbour counts of a slot, as the pair loops would leave them."""
    g = _gen(seed + 1)
    out = {k: s * torch.randn(n, generator=g, device="cuda")
           for k, s in (("A_X", 30.0), ("A_Y", 30.0), ("A_Z", 30.0), ("DU", 0.3))}
    out["VSIG"] = 2.0 + torch.rand(n, generator=g, device="cuda")
    for k in ("NNGB", "NFORCE"):
        out[k] = torch.randint(30, 70, (n,), generator=g, device="cuda", dtype=torch.int32)
    return out


def prepare(case, seed):
    pipe = _pipeline(case, seed)
    state = {"case": case, "pipe": pipe}
    op = case["op"]
    if op in ("density", "force", "hiter", "serve", "linear"):
        pipe.bin()
        pipe.convert("full")
    if op in ("force", "serve"):
        pipe.density()
    if op == "serve":
        state["served"] = _Served(pipe, seed)
    if op == "linear":
        for k, t in _rates(pipe.n, seed).items():
            pipe.soa[k].copy_(t)
        state["totals"] = torch.zeros(8, dtype=torch.float64, device="cuda")
    return state


# --- a pass --------------------------------------------------------------------
STEP_FLOATS = ("x", "v", "u", "rho", "wcount", "rho_dh", "f", "P", "c", "a", "du", "vsig")
STEP_WHOLE = ("nngb", "nforce", "cell")
DENS = ("RHO", "WCOUNT", "RHO_DH", "F", "P", "C")
FORCE = ("A_X", "A_Y", "A_Z", "DU", "VSIG")


def _record_fields(pipe, names):
    return {k: _field(pipe.aos, pipe.dtype, k) for k in names}


def run(state):
    pipe, op = state["pipe"], state["case"]["op"]
    if op == "step":
        pipe.soa_step(DT, DT)
        return _record_fields(pipe, STEP_FLOATS + STEP_WHOLE)
    if op == "aos_step":
        pipe.aos_step(DT, DT)
        return _record_fields(pipe, STEP_FLOATS + STEP_WHOLE[:2])
    if op == "density":
        pipe.density()
        return {k: pipe.soa[k] for k in DENS + ("NNGB",)}
    if op == "force":
        pipe.force()
        return {k: pipe.soa[k] for k in FORCE + ("NFORCE",)}
    if op == "reorder":
        pipe.bin()
        pipe.convert("full")
        pipe.writeback("full")
        return {**{k: pipe.soa[k] for k in ("OFF_X", "VQ_X", "M", "H", "U", "X_Z", "V_Y", "UK")},
                "perm": pipe.cells.perm, "cell": pipe.cells.cell, "start": pipe.cells.cell_start,
                "sub_start": pipe.cells.sub_start, "hmax": pipe.cells.hmax,
                "anc": pipe.soa["ANC"], **_record_fields(pipe, ("x", "v", "u"))}
    if op == "linear":
        pipe.reduce()
        sphmi.step_totals(pipe.soa, pipe.cells, state["totals"], pipe.red_ws, pipe.prm)
        pipe.kick_drift(DT, DT)
        return {"sums": pipe.red_out, "totals": state["totals"], "moved": pipe.moved,
                **{k: pipe.soa[k] for k in ("X_X", "X_Y", "X_Z", "V_X", "V_Y", "V_Z", "UK")}}
    if op == "hiter":
        pipe.convert("density")
        _, left = pipe.smoothing_length(write_back=False)
        return {"H": pipe.soa["H"], "left": left}
    served = state["served"]
    served.server.run(served.req)
    o, k = served.out, TASK_ROWS
    return {"density": [o["v"][:k, c] for c in range(3)], "nngb": o["count"][:k],
            "force": [o["v"][k:, c] for c in range(5)], "nforce": o["count"][k:]}


# --- what a pass cannot do without ------------------------------------------------
def work(case):
    n = case["n"]
    rec = 128 if case["rec"] == "f32" else 200
    w = 4 if case["store"] == "f32" else 2
    if case["op"] in ("step", "aos_step"):      # records in and out, both pair sums
        return {"bytes": n * 2 * rec, "flops": n * PAIRS * 140}
    if case["op"] == "density":                 # offsets, m, h, u; seven outputs
        return {"bytes": n * (6 * w + 28), "flops": n * PAIRS * 40}
    if case["op"] == "force":                   # offsets, v, m, h, rho, f, P, c; six outputs
        return {"bytes": n * (8 * w + 16 + 24), "flops": n * PAIRS * 100}
    if case["op"] == "reorder":                 # records in and out; list, views
        return {"bytes": n * (2 * rec + 8 + 9 * w + 40), "flops": n * 60}
    if case["op"] == "linear":                  # kick view in and out, rates, m, h, v, counts
        return {"bytes": n * (96 + 20 + 12), "flops": n * 60}
    if case["op"] == "hiter":                   # a density sum for each of about four Newton steps
        return {"bytes": n * 4 * 30, "flops": n * PAIRS * 40 * 4}
    # slots in, records out, and the tests of a task's pairs with a cell of about 32
    return {"bytes": 2 * TASK_ROWS * 92, "flops": 2 * TASK_ROWS * 32 * 9}


# --- the same in 64 bits ------------------------------------------------------------
class _Exact:
    """FP64 sums over pairs found with a cell list, in input order."""

    CHUNK = 1 << 25

    def __init__(self, case, seed):
        rec, n_c = _records(case, seed)
        dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float64)).cuda()
        self.case, self.n, self.n_c = case, case["n"], n_c
        self.x, self.v = dev(rec["x"]), dev(rec["v"])
        self.m, self.h, self.u = dev(rec["m"]), dev(rec["h"]), dev(rec["u"])
        self.gk = _gamma_k(case)
        self.prm = {k: float(v) for k, v in (("g", GAMMA), ("al", ALPHA), ("be", BETA))}
        c = self.cells(n_c)
        self.cell = c[:, 0] + n_c * (c[:, 1] + n_c * c[:, 2])
        self.by_cell = torch.argsort(self.cell, stable=True)
        cnt = torch.bincount(self.cell, minlength=n_c ** 3)
        self.count = cnt
        self.start = torch.cumsum(cnt, 0) - cnt

    def cells(self, k):
        return (self.x * k).floor().long().clamp(0, k - 1)

    def perm(self):
        """Slot order: cell, then the sub-cell's Morton code, then input order."""
        R = 1 << self.case["sub_bits"]
        sub = (self.cells(self.n_c * R) - self.cells(self.n_c) * R).clamp(0, R - 1)
        key = self.cell * R ** 3
        for b in range(self.case["sub_bits"]):
            for a in range(3):
                key = key + (((sub[:, a] >> b) & 1) << (3 * b + a))
        return torch.argsort(key, stable=True)

    def ragged(self, i, cj, keep, add):
        """Every j of cell cj[k] against i[k]: add(k, j, d, r) for the pairs keep(k, j, r2)."""
        cnt = self.count[cj]
        end = torch.cumsum(cnt, 0)
        total, a = int(end[-1]) if len(end) else 0, 0
        while a < len(i):
            base = int(end[a - 1]) if a else 0
            b = int(torch.searchsorted(end, torch.tensor([base + self.CHUNK], device="cuda"),
                                       right=True)) if base + self.CHUNK < total else len(i)
            b = max(b, a + 1)
            k = torch.repeat_interleave(torch.arange(a, b, device="cuda"), cnt[a:b])
            first = (end - cnt)[a:b] - base
            j = self.start[cj[k]] + torch.arange(len(k), device="cuda") - first[k - a]
            j = self.by_cell[j]
            d = self.x[i[k]] - self.x[j]
            d = d - d.round()
            r2 = (d * d).sum(1)
            ok = keep(k, j, r2).nonzero()[:, 0]
            add(k[ok], j[ok], d[ok], r2[ok].sqrt())
            a = b

    def around(self, keep, add):
        """ragged() over the 27 cells around every particle's cell."""
        c = self.cells(self.n_c)
        i = self.by_cell
        for q in range(27):
            o = torch.tensor([q % 3 - 1, q // 3 % 3 - 1, q // 9 - 1], device="cuda")
            t = (c[i] + o) % self.n_c
            cj = t[:, 0] + self.n_c * (t[:, 1] + self.n_c * t[:, 2])
            self.ragged(i, cj, lambda k, j, r2: keep(i[k], j, r2),
                        lambda k, j, d, r: add(i[k], j, d, r))

    def w_dw(self, u):
        if self.case["kernel"] == "m4":
            t, s = (1 - u).clamp(min=0), (0.5 - u).clamp(min=0)
            return (16 / math.pi * (t ** 3 - 4 * s ** 3), -48 / math.pi * (t ** 2 - 4 * s ** 2))
        t = (1 - u).clamp(min=0)
        return 21 / (2 * math.pi) * t ** 4 * (1 + 4 * u), -210 / math.pi * u * t ** 3

    def density(self, h=None, around=None):
        h = self.h if h is None else h
        H = self.gk * h
        z = lambda: torch.zeros(self.n, dtype=torch.float64, device="cuda")
        rho, wc, dh = z(), z(), z()

        def add(i, j, d, r):
            u = r / H[i]
            w, dw = self.w_dw(u)
            rho.index_add_(0, i, self.m[j] * w)
            wc.index_add_(0, i, w)
            dh.index_add_(0, i, self.m[j] * (3 * w + u * dw))
        (around or self.around)(lambda i, j, r2: r2 < H[i] ** 2, add)
        rho, wc, dh = rho / H ** 3, 4 * math.pi / 3 * wc, -self.gk * dh / H ** 4
        g = self.prm["g"]
        return {"RHO": rho, "WCOUNT": wc, "RHO_DH": dh, "F": 1 / (1 + h * dh / (3 * rho)),
                "P": (g - 1) * rho * self.u, "C": (g * (g - 1) * self.u).sqrt()}

    def force_terms(self, dens):
        H, rho, c = self.gk * self.h, dens["RHO"], dens["C"]
        A = dens["F"] * dens["P"] / rho ** 2

        def terms(i, j, d, r):
            e = torch.where(r[:, None] > 0, d / r.clamp(min=1e-300)[:, None], torch.zeros_like(d))
            gi = self.w_dw(r / H[i])[1] / H[i] ** 4
            gj = self.w_dw(r / H[j])[1] / H[j] ** 4
            w = ((self.v[i] - self.v[j]) * e).sum(1)
            mu = w.clamp(max=0)
            vs = c[i] + c[j] - self.prm["be"] * mu
            visc = -self.prm["al"] * vs * mu / (rho[i] + rho[j])
            gb = 0.5 * (gi + gj)
            kc = self.m[j] * (A[i] * gi + A[j] * gj + visc * gb)
            return -kc[:, None] * e, self.m[j] * (A[i] * gi + 0.5 * visc * gb) * w, vs
        return (lambda i, j, r2: (r2 < torch.maximum(H[i], H[j]) ** 2) & (i != j)), terms

    def force(self, dens):
        keep, terms = self.force_terms(dens)
        a = torch.zeros(self.n, 3, dtype=torch.float64, device="cuda")
        du, vsig = torch.zeros_like(a[:, 0]), torch.zeros_like(a[:, 0])

        def add(i, j, d, r):
            da, dd, vs = terms(i, j, d, r)
            a.index_add_(0, i, da)
            du.index_add_(0, i, dd)
            vsig.scatter_reduce_(0, i, vs, "amax")
        self.around(keep, add)
        return {"A_X": a[:, 0], "A_Y": a[:, 1], "A_Z": a[:, 2], "DU": du, "VSIG": vsig}

    def smoothing_length(self):
        h = self.h.clone()
        for _ in range(12):
            d = self.density(h)
            t = ETA * (self.m / d["RHO"]) ** (1 / 3)
            new = h - (h - t) / (1 + t / (3 * d["RHO"]) * d["RHO_DH"])
            new = torch.minimum(torch.maximum(new, 0.5 * h), 2 * h)
            new = new.clamp(max=1.0 / (self.n_c * self.gk))
            far = float(((new - h).abs() / h).max())
            h = new
            if far < 1e-10:
                break
        return h

    def tasks(self, tasks, perm):
        """The sums of each task's slots over one neighbouring cell, in record order."""
        t = torch.from_numpy(tasks.astype(np.int64)).cuda()
        size = t[:, 4] - t[:, 3]
        row = torch.repeat_interleave(torch.arange(len(t), device="cuda"), size)
        off = torch.arange(len(row), device="cuda") - (torch.cumsum(size, 0) - size)[row]
        i, cj = perm[t[row, 3] + off], t[row, 2]
        k0 = TASK_ROWS
        dens = self.density()
        H = self.gk * self.h
        o = [torch.zeros(len(row), dtype=torch.float64, device="cuda") for _ in range(5)]

        def add_d(k, j, d, r):
            u = r / H[i[k]]
            w, dw = self.w_dw(u)
            for c, val in enumerate((self.m[j] * w, w, self.m[j] * (3 * w + u * dw))):
                o[c].index_add_(0, k, val)
        self.ragged(i[:k0], cj[:k0], lambda k, j, r2: r2 < H[i[k]] ** 2, add_d)
        Hi = H[i[:k0]]
        out_d = [o[0][:k0] / Hi ** 3, 4 * math.pi / 3 * o[1][:k0], -self.gk * o[2][:k0] / Hi ** 4]
        i_f, cj_f = i[k0:], cj[k0:]
        keep, terms = self.force_terms(dens)
        f = [torch.zeros(len(i_f), dtype=torch.float64, device="cuda") for _ in range(5)]

        def add_f(k, j, d, r):
            da, dd, vs = terms(i_f[k], j, d, r)
            for c in range(3):
                f[c].index_add_(0, k, da[:, c])
            f[3].index_add_(0, k, dd)
            f[4].scatter_reduce_(0, k, vs, "amax")
        self.ragged(i_f, cj_f, lambda k, j, r2: keep(i_f[k], j, r2), add_f)
        return out_d, f


def exact(case, seed):
    op = case["op"]
    if op == "reorder":
        return None                             # rounding and order only
    if op == "linear":
        return _exact_linear(case, seed)
    e = _Exact(case, seed)
    if op == "hiter":
        return {"H": e.smoothing_length()[e.perm()], "left": None}
    if op == "serve":
        start = torch.cat([e.start, torch.tensor([e.n], device="cuda")]).cpu().numpy()
        d, f = e.tasks(_tasks(start, e.n_c, seed), e.perm())
        return {"density": d, "nngb": None, "force": f, "nforce": None}
    d = e.density()
    if op == "density":
        p = e.perm()
        return {**{k: d[k][p] for k in DENS}, "NNGB": None}
    f = e.force(d)
    if op == "force":
        p = e.perm()
        return {**{k: f[k][p] for k in FORCE}, "NFORCE": None}
    a = torch.stack([f["A_X"], f["A_Y"], f["A_Z"]], 1)
    v = e.v + a * DT
    x = e.x + v * DT
    return {"x": x - x.floor(), "v": v, "u": e.u + f["DU"] * DT, "rho": d["RHO"],
            "wcount": d["WCOUNT"], "rho_dh": d["RHO_DH"], "f": d["F"], "P": d["P"], "c": d["C"],
            "a": a, "du": f["DU"], "vsig": f["VSIG"],
            **{k: None for k in STEP_WHOLE[:2 if op == "aos_step" else 3]}}


def _exact_linear(case, seed):
    e = _Exact(case, seed)
    p, f32 = e.perm(), lambda t: t.float().double()
    x, v, m, h, u = e.x[p], f32(e.v[p]), f32(e.m[p]), f32(e.h[p]), f32(e.u[p])
    r = {k: t.double() for k, t in _rates(case["n"], seed).items()}
    a, du = torch.stack([r["A_X"], r["A_Y"], r["A_Z"]], 1), r["DU"]
    va = (v * a).sum(1)
    sums = [*(m[:, None] * a).sum(0), (m * (va + du)).sum(), (m * a.norm(dim=1)).sum(),
            (m * (va.abs() + du.abs())).sum(), r["NNGB"].sum(), r["NFORCE"].sum()]
    tot = [*(m[:, None] * v).sum(0), 0.5 * (m * (v * v).sum(1)).sum(), (m * u).sum(), m.sum(),
           (sphmi.C_CFL * _gamma_k(case) * h / r["VSIG"]).min(),
           torch.tensor(float(len(m)), device="cuda", dtype=torch.float64)]
    vn = v + a * DT
    xn = x + vn * DT
    xn = xn - xn.floor()
    return {"sums": torch.stack(sums), "totals": torch.stack(tot), "moved": None,
            "X_X": xn[:, 0], "X_Y": xn[:, 1], "X_Z": xn[:, 2], "V_X": vn[:, 0], "V_Y": vn[:, 1],
            "V_Z": vn[:, 2], "UK": u + du * DT}
