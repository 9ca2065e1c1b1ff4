"""The work that users of this package have it do, as measurable cases.

A case is a dict of plain values.  `kind` says which public call it times:

  sweep    Lattice.sweep: n checkerboard sweeps of one resident lattice
  measure  Lattice.measure: B, M, Q, the sigma-h histogram and C(r, t)
  quench   run_quench: a lattice from creation to its last measurement
  group    group_sweep: n sweeps of many lattices, as the serving loop's ticks
  read     Lattice.read: the whole lattice as int8 spins on the host

Sizes are those of the benchmark (4-bit Ising at L = 2^17, Blume-Capel at
2^16 and below, 512 ... 8192 in batches), of the parity workload (L = 256 with
every distance) and generic ones between, multiples of 64 that are no powers
of two among them."""
import math

import numpy as np
import torch

import paper_2502_18624_amd as mcl
from paper_2502_18624_amd import quench as mcl_quench

BETA_C = math.log(1.0 + math.sqrt(2.0)) / 2.0
MODEL = {"ising": mcl.ISING, "bc": mcl.BC, "lut": mcl.ISING_LUT}
BITS = {"ising": 4, "bc": 4, "lut": 1}
CORR = {"none": mcl.CORR_NONE, "full": mcl.CORR_FULL, "protocol": mcl.CORR_PROTOCOL}


def _beta(model):
    return 1.0 / 1.4 if model == "bc" else BETA_C


def _d(model):
    return 1.0 if model == "bc" else 0.0


def listed():
    return [
        # one sweep of a small lattice: what a program pays that sweeps and looks in turn
        {"name": "sweep-bc-256x1", "kind": "sweep", "model": "bc", "L": 256, "n": 1},
        # the parity workload: a small quench with every distance at t = 2^k
        {"name": "quench-ising-256", "kind": "quench", "model": "ising", "L": 256, "n": 64, "corr": "full"},
        # a middle size that is no power of two, in one long call
        {"name": "sweep-ising-3008x32", "kind": "sweep", "model": "ising", "L": 3008, "n": 32},
        # the paper's middle sizes (Table 2)
        {"name": "sweep-bc-16384x4", "kind": "sweep", "model": "bc", "L": 16384, "n": 4},
        # the headline lattice: its sweeps, then its measurement
        {"name": "sweep-ising-131072x2", "kind": "sweep", "model": "ising", "L": 131072, "n": 2},
        {"name": "measure-ising-131072", "kind": "measure", "model": "ising", "L": 131072, "corr": "protocol", "t": 8},
        # the protocol's measurement of Blume-Capel, with Q
        {"name": "measure-bc-32768", "kind": "measure", "model": "bc", "L": 32768, "corr": "protocol", "t": 8},
        # every distance of a lattice that is no power of two
        {"name": "measure-full-ising-2112", "kind": "measure", "model": "ising", "L": 2112, "corr": "full", "t": 8},
        # a short quench in the paper's own cells: creation, sweeps and measurements at t = 1, 2, 4
        {"name": "quench-lut-65536", "kind": "quench", "model": "lut", "L": 65536, "n": 4, "corr": "protocol"},
        # a tick of the serving loop: replicas of all models and sizes, temperatures of their own
        {"name": "group-mixed-48", "kind": "group", "model": "mixed", "count": 48, "lo": 512, "hi": 8192, "n": 4},
        # a parameter scan over small lattices of one size
        {"name": "group-small-512", "kind": "group", "model": "both", "count": 512, "lo": 256, "hi": 256, "n": 16},
        # a snapshot of the spins
        {"name": "read-ising-4096", "kind": "read", "model": "ising", "L": 4096, "t": 4},
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _size(rng, model, lo, hi):
    unit = 256 if model == "lut" else 64
    return max(unit, int(_log_uniform(rng, lo, hi) / unit + 0.5) * unit)


def draw(rng):
    kind = rng.choice(["sweep", "sweep", "sweep", "measure", "measure", "measure", "quench", "group", "read"])
    model = rng.choice(["ising", "bc", "lut"])
    if kind == "sweep":
        L = _size(rng, model, 64, 49152)
        # up to 2^32 updates a call, one sweep of the largest
        n = max(1, int(_log_uniform(rng, 1, max(1.5, min(256.0, 2.0 ** 32 / (L * L))))))
        return {"kind": kind, "model": model, "L": L, "n": n}
    if kind == "measure":
        corr = rng.choice(["protocol", "protocol", "full", "none"])
        if corr == "protocol":
            L = 1 << rng.randint(8 if model == "lut" else 6, 15)
        else:
            L = _size(rng, model, 64, 3072 if corr == "full" else 32768)
        return {"kind": kind, "model": model, "L": L, "corr": corr, "t": rng.randint(1, 200 if L <= 4096 else 12)}
    if kind == "quench":
        L = 1 << rng.randint(8 if model == "lut" else 6, 13)
        n = int(_log_uniform(rng, 2, 128 if L <= 2048 else 12))
        corr = rng.choice(["protocol", "none"] + (["full"] if L <= 1024 else []))
        return {"kind": kind, "model": model, "L": L, "n": n, "corr": corr}
    if kind == "group":
        if rng.random() < 0.5:
            hi = int(_log_uniform(rng, 1024, 8192))
            return {"kind": kind, "model": "mixed", "count": rng.randint(2, 56), "lo": 256, "hi": hi,
                    "n": rng.randint(1, 4)}
        L = _size(rng, "bc", 64, 1024)
        count = max(2, min(1024, int(_log_uniform(rng, 2.0 ** 20, 2.0 ** 27) / (L * L))))
        return {"kind": kind, "model": "both", "count": count, "lo": L, "hi": L, "n": rng.randint(1, 24)}
    return {"kind": kind, "model": model, "L": _size(rng, model, 64, 4096), "t": rng.randint(1, 16)}


def _planes(lat, name):
    """The lattice's cells: its two colour planes, in the caller's buffer."""
    off = lat.ptr - lat.mem.data_ptr()
    return lat.mem[off:off + lat.L * lat.L * BITS[name] // 8].view(torch.int64)


def _replicas(case, seed):
    """(model, L, seed, beta, D, n) of each replica of a batch: the sizes by the case, the parameters by the seed."""
    sizes, rng = np.random.default_rng(case["count"] + case["hi"]), np.random.default_rng(seed)
    out = []
    for i in range(case["count"]):
        model = ("ising", "bc", "lut")[i % 3] if case["model"] == "mixed" else ("ising", "bc")[i % 2]
        unit = 256 if model == "lut" else 64
        L = int(sizes.integers(case["lo"] // unit, case["hi"] // unit + 1)) * unit
        beta = BETA_C / rng.uniform(0.5, 1.5)
        D = float(rng.choice([0.0, 0.5, 1.0])) if model == "bc" else 0.0
        out.append((model, L, seed + 1000 * i, beta, D, case["n"]))
    return out


def prepare(case, seed):
    kind = case["kind"]
    if kind == "quench":
        return {"case": case, "seed": seed}
    if kind == "group":
        reps = _replicas(case, seed)
        lats = []
        state = {"case": case}
        if case["lo"] == case["hi"]:
            # replicas of one size, in one buffer
            L = reps[0][1]
            size = max(mcl.query_bytes(MODEL[r[0]], L) for r in reps)
            stride = (size + 511) // 256 * 256
            buf = torch.empty((len(reps) + 1) * stride, dtype=torch.uint8, device="cuda")
            skip = -buf.data_ptr() % 256
            state["cells"] = buf[skip:skip + len(reps) * stride].view(len(reps), stride)[:, :L * L // 2]
            mems = [buf[skip + i * stride:skip + (i + 1) * stride] for i in range(len(reps))]
        else:
            mems = [None] * len(reps)
        for (model, L, s, *_), mem in zip(reps, mems):
            lats.append(mcl.Lattice(MODEL[model], L, s, mem=mem))
        if "cells" not in state:
            state["cells"] = [_planes(l, r[0]) for l, r in zip(lats, reps)]
        state.update(lats=lats, n=[r[5] for r in reps], beta=[r[3] for r in reps], D=[r[4] for r in reps])
        return state
    model = case["model"]
    lat = mcl.Lattice(MODEL[model], case["L"], seed)
    # a quench on its way: sweep cases go on from t = 2, measured lattices from t
    lat.sweep(case.get("t", 2), _beta(model), _d(model))
    return {"case": case, "lat": lat, "cells": _planes(lat, model)}


def _flat(rows):
    """Measurements of a quench as a few arrays: the integer sums, C(r) and the derived values."""
    has_r = "Cx_norm" in rows[0]
    out = {
        "sums": np.array([[m["t"], m["B"], m["M"], m["Q"], m["invalid"], *m["counts"], *m["sd"]] for m in rows],
                         dtype=np.int64),
        "derived": np.array([[m["E"], m["schwinger_dyson"]] for m in rows], dtype=np.float64),
    }
    if has_r:
        for key in ("r", "Cx", "Cy", "nsrc", "Cx_norm", "Cy_norm"):
            out[key] = np.concatenate([m[key] for m in rows])
        out["xi"] = np.array([[math.nan if m[k] is None else m[k] for k in ("xi12", "xi23", "L_over_xi12")]
                              for m in rows], dtype=np.float64)
    return out


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "sweep":
        state["lat"].sweep(case["n"], _beta(case["model"]), _d(case["model"]))
        return state["cells"]
    if kind == "measure":
        return state["lat"].measure(CORR[case["corr"]])
    if kind == "group":
        mcl.group_sweep(state["lats"], state["n"], state["beta"], state["D"])
        return state["cells"]
    if kind == "read":
        return state["lat"].read()
    m = case["model"]
    return _flat(list(mcl_quench.run_quench(MODEL[m], case["L"], state["seed"], _beta(m), _d(m), case["n"],
                                            corr=CORR[case["corr"]])))


# ---------------------------------------------------------------------------
# What a pass cannot do without.  A sweep reads its own and the other colour
# and writes its own, for each colour; an update takes its share of a
# 10-round generator block (60 integer operations for 4 draws, 16 cells
# sharing two blocks in the 1-bit mode) and about ten more.  A measurement
# reads the lattice once and multiplies and adds every pair it sums.
# ---------------------------------------------------------------------------
def _sweep_work(model, L, n):
    ops = 10 + (60 / 4 if model != "lut" else 60 / 8)
    return n * 3 * L * L * BITS[model] / 8, n * L * L * ops


def _measure_work(model, L, corr, t):
    flops = 10.0 * L * L
    if corr != "none":
        nr = len(mcl.rset(CORR[corr], L, t))
        every = nr if corr == "full" else min(nr, 33)
        flops += 2 * 2 * (every * L * L + (nr - every) * (L // 16) ** 2)
    return L * L * BITS[model] / 8, flops


def work(case):
    kind = case["kind"]
    if kind == "sweep":
        b, f = _sweep_work(case["model"], case["L"], case["n"])
    elif kind == "measure":
        b, f = _measure_work(case["model"], case["L"], case["corr"], case["t"])
    elif kind == "read":
        b, f = case["L"] ** 2 * (BITS[case["model"]] / 8 + 1), 0.0
    elif kind == "group":
        b = f = 0.0
        for model, L, _, _, _, n in _replicas(case, 1):
            db, df = _sweep_work(model, L, n)
            b, f = b + db, f + df
    else:
        m, L = case["model"], case["L"]
        b, f = _sweep_work(m, L, case["n"])
        b += L * L * BITS[m] / 8
        f += 15 * L * L
        t = 1
        while t <= case["n"]:
            db, df = _measure_work(m, L, case["corr"], t)
            b, f, t = b + db, f + df, 2 * t
    return {"bytes": float(b), "flops": float(f)}


# ---------------------------------------------------------------------------
# The same quench in plain numpy.  All other outputs are whole numbers.
# ---------------------------------------------------------------------------
def _philox(c0, c1, c2, c3, seed):
    """Philox4x32-10 (Salmon et al., SC'11) of counter arrays."""
    mask = np.uint64(0xFFFFFFFF)
    c = [np.asarray(v, dtype=np.uint64) for v in np.broadcast_arrays(c0, c1, c2, c3)]
    k0, k1 = seed & 0xFFFFFFFF, (seed >> 32) & 0xFFFFFFFF
    for _ in range(10):
        p0, p1 = c[0] * np.uint64(0xD2511F53), c[2] * np.uint64(0xCD9E8D57)
        c = [(p1 >> np.uint64(32)) ^ c[1] ^ np.uint64(k0), p1 & mask,
             (p0 >> np.uint64(32)) ^ c[3] ^ np.uint64(k1), p0 & mask]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return np.stack(c, axis=-1)


def _draws(index, per, a, b, seed):
    """Word index % per of block index / per, counter words 2 and 3 given."""
    blk = np.unique(index // per)
    w = _philox(blk & 0xFFFFFFFF, blk >> 32, a, b, seed)
    return w[np.searchsorted(blk, index // per), index % per]


def _np_init(model, L, seed):
    w = _draws(np.arange(L * L), 4, 0, 4, seed).reshape(L, L)
    if model == "bc":
        return ((w * np.uint64(3)) >> np.uint64(32)).astype(np.int64) - 1
    return np.where(w < (1 << 31), 1, -1).astype(np.int64)


def _field(s):
    return np.roll(s, 1, 0) + np.roll(s, -1, 0) + np.roll(s, 1, 1) + np.roll(s, -1, 1)


def _threshold(beta, dE):
    return np.minimum(np.floor(np.ldexp(np.exp(-beta * dE), 32)), 2.0 ** 32 - 1)


def _np_sweep(s, model, L, seed, t, beta, D):
    y, x = np.divmod(np.arange(L * L), L)
    for c in (0, 1):
        site = np.nonzero((x + y) % 2 == c)[0]
        k = site >> 1
        flat = s.reshape(-1)
        own, h = flat[site], _field(s).reshape(-1)[site]
        if model == "lut":
            p = math.exp(-4.0 * beta)
            T, cum = [], 0.0
            for j in range(16):
                T.append(math.floor(math.ldexp(cum, 32)))
                q = 1.0
                for i in range(4):
                    q *= p if (j >> i) & 1 else 1.0 - p
                cum += q
            bit = []
            for e in (0, 1):
                u = _draws(k >> 2, 4, t, 8 + 2 * c + e, seed)
                pat = np.searchsorted(np.array(T, dtype=np.uint64), u, side="right") - 1
                bit.append((pat >> (k & 3)) & 1)
            al = own * h
            flip = (al <= 0) | ((al == 2) & (bit[0] == 1)) | ((al == 4) & (bit[0] & bit[1] == 1))
            flat[site] = np.where(flip, -own, own)
            continue
        u = _draws(k, 4, t, c, seed).astype(np.float64)
        if model == "ising":
            new, dE = -own, 2.0 * own * h
        else:
            b = (_draws(k >> 5, 4, t, 2 + c, seed).astype(np.int64) >> (k & 31)) & 1
            new = (own + 2 + b) % 3 - 1
            dE = -(h * (new - own)).astype(np.float64) + D * (new * new - own * own)
        accept = (dE <= 0) | (u < _threshold(beta, dE))
        flat[site] = np.where(accept, new, own)


def _np_corr(s, r, sampled):
    cx, cy = [], []
    for d, few in zip(r, sampled):
        a, b = s * np.roll(s, -d, 1), s * np.roll(s, -d, 0)
        cx.append(int((a[::16, ::16] if few else a).sum()))
        cy.append(int((b[::16, ::16] if few else b).sum()))
    return np.array(cx, dtype=np.int64), np.array(cy, dtype=np.int64)


def _np_distances(mode, L, t):
    half = L // 2
    if mode == "full":
        return list(range(half + 1)), half + 1
    rc = max(256, math.floor(6 * math.sqrt(math.log(L / 65536) / 3.3 ** 2 + 1) * math.sqrt(t) + 0.5))
    r = list(range(min(half, 32) + 1))
    every = len(r)
    r += range(33, min(half, rc) + 1)
    for e in range(1, 32 * (L.bit_length() - 2) + 1):
        d = math.floor(2.0 ** (e / 32.0))
        if rc < d <= half and d != r[-1]:
            r.append(d)
    return r, every


def _np_xi(r, C, k):
    stop = np.nonzero(C <= 0)[0]
    n = int(stop[0]) if stop.size else len(C)
    r, C = r[:n].astype(np.float64), C[:n]

    def area(p):
        f = r ** p * C
        return float((0.5 * (f[1:] + f[:-1]) * np.diff(r)).sum())

    return area(k + 1) / area(k)


def exact(case, seed):
    if case["kind"] != "quench" or case["L"] > 512:
        return None
    model, L, corr = case["model"], case["L"], case["corr"]
    beta, D = _beta(model), _d(model)
    s = _np_init(model, L, seed)
    rows, t = [], 0
    for t in range(1, case["n"] + 1):
        _np_sweep(s, model, L, seed, t - 1, beta, D)
        if t & (t - 1):
            continue
        sh = s * _field(s)
        B, Q = int(sh.sum()) // 2, int((s * s).sum())
        m = {"t": t, "B": B, "M": int(s.sum()), "Q": Q, "invalid": 0,
             "counts": [int((s == v).sum()) for v in (-1, 0, 1)],
             "sd": [int((sh == v).sum()) for v in range(-4, 5)],
             "E": -B + D * Q if D else -B,
             "schwinger_dyson": float(np.exp(-2.0 * beta * sh).sum()) / (L * L)}
        if corr != "none":
            r, every = _np_distances(corr, L, t)
            sampled = [j >= every for j in range(len(r))]
            m["r"] = np.array(r, dtype=np.int32)
            m["Cx"], m["Cy"] = _np_corr(s, r, sampled)
            m["nsrc"] = np.where(sampled, (L // 16) ** 2, L * L).astype(np.int64)
            m["Cx_norm"], m["Cy_norm"] = m["Cx"] / m["nsrc"], m["Cy"] / m["nsrc"]
            C = 0.5 * (m["Cx_norm"] + m["Cy_norm"])
            ok = C[1] > 0
            m["xi12"] = _np_xi(m["r"], C, 1) if ok else None
            m["xi23"] = _np_xi(m["r"], C, 2) if ok else None
            m["L_over_xi12"] = L / m["xi12"] if m["xi12"] else None
        rows.append(m)
    return _flat(rows)
