"""What a user of this library has it do, as cases that can be timed.

A case names one kind of work and its sizes:

* "program": a whole propagation kept as a device program, run on a fresh set
  (Algorithm 1 through pp_create + pp_batch_run), the usual way in;
* "calls": the same steps one C call at a time, as a program that looks at
  the set between layers does;
* "batch": many ring propagations of uneven size advancing together;
* "ingest": an observable of many rows merged by orbit representative.

Every pass returns the expectation and the final representative set (key
order), which is what Algorithm 1 ends with.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2512_12094_amd import _lib as L
from paper_2512_12094_amd import driver
from paper_2512_12094_amd import workloads as W


def _case(name, kind, model, n, steps, theta, eps, wmax, group, dtype, **more):
    return dict(name=name, kind=kind, model=model, n=n, steps=steps, theta=theta, eps=eps,
                wmax=wmax, group=group, dtype=dtype, **more)


def listed():
    return [
        # the smallest job: a ring small enough to keep every string
        _case("ring8_exact", "program", "xxz", 8, 6, 0.1, 0.0, -1, "Zn", "f64", delta=1.0),
        # the benchmark's propagation: a truncated ring at one-word keys
        _case("ring32", "program", "xxz_pairs", 32, 20, 0.05, 1e-4, 8, "Zn", "f64", delta=1.5),
        # the same circuit without symmetry merging, the method's comparison
        _case("ring32_plain", "program", "xxz_pairs", 32, 20, 0.05, 1e-4, 8, "none", "f64",
              delta=1.5),
        # a served-size ring whose keys do not fit 64 bits (wide merge)
        _case("ring48_wide", "program", "xxz", 48, 16, 0.08, 1e-5, -1, "Zn", "f64", delta=1.2),
        # FP32 coefficients and the dihedral group
        _case("ring24_dihedral_f32", "program", "xxz", 24, 15, 0.08, 5e-6, -1, "Dn", "f32",
              delta=0.8),
        # a program that steps the layers itself (one C call per operation)
        _case("ring32_calls", "calls", "xxz_pairs", 32, 8, 0.05, 1e-4, 8, "Zn", "f64", delta=1.5),
        # the paper's tilted-field Ising ring, untruncated
        _case("ising12_exact", "program", "ising", 12, 7, 0.25, 0.0, -1, "Zn", "f64", delta=0.0),
        # all-to-all circuit under S_n with noise: sub-layers of 2016 rotations
        _case("all_to_all64", "program", "all_to_all", 64, 1, 0.02, 1e-5, -1, "Sn", "f64",
              delta=1.0, subs=2),
        # power-law couplings on a torus: 120 rotations a sub-layer, 2D translations
        _case("torus4x4", "program", "torus", 16, 1, 0.1, 1e-4, -1, "T2", "f64", delta=-1.8),
        # the largest: a ring grown to millions of representatives
        _case("ring32_grown", "program", "xxz_pairs", 32, 5, 0.2, 1e-6, 12, "Zn", "f64",
              delta=1.5),
        # twelve rings of uneven size and depth advancing together
        _case("batch12", "batch", "xxz", 48, 10, 0.06, 1e-5, -1, "Zn", "f64", delta=1.2, count=12),
        # a large observable: 2^20 rows, 32 rotations of each string
        _case("ingest_2p20", "ingest", "records", 32, 1, 0.0, 0.0, 8, "Zn", "f64", delta=0.0,
              rows=1 << 20, dup=32),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    """One more case of the same ranges."""
    kind = rng.choice(["exact", "ring", "ring", "wide", "calls", "ising", "all_to_all", "torus",
                       "batch", "ingest"])
    dtype = rng.choice(["f64", "f64", "f32"])
    theta = round(rng.uniform(0.03, 0.08), 4)
    delta = round(rng.uniform(0.5, 2.0), 3)
    eps = float("%.3g" % _log_uniform(rng, 1e-5, 1e-3))
    if kind == "exact":
        return dict(kind="program", model="xxz", n=rng.randint(4, 9), steps=rng.randint(2, 8),
                    theta=round(rng.uniform(0.05, 0.3), 4), eps=0.0, wmax=-1,
                    group=rng.choice(["Zn", "Dn"]), dtype=dtype, delta=delta)
    if kind == "ring":
        return dict(kind="program", model="xxz_pairs", n=rng.randint(13, 32),
                    steps=rng.randint(6, 20), theta=theta, eps=max(eps, 5e-5),
                    wmax=rng.choice([-1, 8, 10]), group=rng.choice(["Zn", "Zn", "Dn", "none"]),
                    dtype=dtype, delta=delta)
    if kind == "wide":
        return dict(kind="program", model="xxz", n=rng.randint(33, 64), steps=rng.randint(5, 14),
                    theta=theta, eps=eps, wmax=rng.choice([-1, 8]),
                    group=rng.choice(["Zn", "Dn"]), dtype=dtype, delta=delta)
    if kind == "calls":
        return dict(kind="calls", model="xxz_pairs", n=rng.randint(9, 32), steps=rng.randint(2, 8),
                    theta=theta, eps=max(eps, 5e-5), wmax=8, group="Zn", dtype=dtype, delta=delta)
    if kind == "ising":
        return dict(kind="program", model="ising", n=rng.randint(5, 12), steps=rng.randint(3, 7),
                    theta=round(rng.uniform(0.1, 0.3), 3), eps=0.0, wmax=-1,
                    group=rng.choice(["Zn", "Zn", "none"]), dtype=dtype, delta=0.0)
    if kind == "all_to_all":
        return dict(kind="program", model="all_to_all", n=rng.randint(10, 64), steps=1,
                    theta=0.02, eps=max(eps, 3e-5), wmax=-1, group="Sn", dtype=dtype, delta=1.0,
                    subs=2)
    if kind == "torus":
        return dict(kind="program", model="torus", n=4 * rng.randint(2, 4), steps=1,
                    theta=round(rng.uniform(0.05, 0.1), 4), eps=max(eps, 1e-4), wmax=-1,
                    group="T2", dtype=dtype, delta=-1.8)
    if kind == "batch":
        return dict(kind="batch", model="xxz", n=rng.randint(16, 64), steps=rng.randint(3, 10),
                    theta=theta, eps=eps, wmax=-1, group="Zn", dtype=dtype, delta=delta,
                    count=rng.randint(2, 16))
    return dict(kind="ingest", model="records", n=rng.randint(14, 32), steps=1, theta=0.0,
                eps=0.0, wmax=8, group=rng.choice(["Zn", "Zn", "Dn"]), dtype=dtype, delta=0.0,
                rows=int(_log_uniform(rng, 1 << 12, 1 << 20)), dup=rng.choice([1, 4, 32]))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _bloch(rng):
    v = rng.normal(size=3)
    v /= np.linalg.norm(v)
    return float(v[0]), float(v[1]), float(v[2])


def _program(case, rng, n=None, steps=None):
    """The case's circuit.  The seed picks the state, the observable's sign
    and, on even rings, the sense of the XX and YY rotations: other
    coefficients on the same strings, so the work stays the case's."""
    n, steps = n or case["n"], steps or case["steps"]
    scale = float(rng.choice([-1.0, 1.0]))
    sense = float(rng.choice([-1.0, 1.0])) if n % 2 == 0 else 1.0
    theta = case["theta"]
    kw = dict(eps=case["eps"], wmax=case["wmax"])
    bloch = _bloch(rng)
    model = case["model"]
    if model in ("xxz", "xxz_pairs"):
        obs = W.sum_ring_pairs(n, "X", scale) if model == "xxz_pairs" else W.sum_single(n, "Z", scale)
        return W.xxz_ring(n, steps, sense * theta, sense * case["delta"], obs=obs, bloch=bloch,
                          group=case["group"], **kw)
    if model == "ising":
        prog = W.tilted_ising_ring(n, steps, theta, **kw)
        prog.obs = [(x, z, c * scale) for x, z, c in prog.obs]
        prog.bloch = bloch
        return prog.with_group(case["group"])
    if model == "all_to_all":
        prog = W.heisenberg_all_to_all(n, steps, theta, p=1e-3, obs=W.sum_single(n, "Z", scale),
                                       bloch=bloch, **kw)
        prog.sublayers = prog.sublayers[-case["subs"]:]
        return prog
    if model == "torus":
        return W.power_law_xxz_torus(4, n // 4, steps, theta, delta=case["delta"],
                                     obs=W.sum_single(n, "Z", scale), bloch=bloch, **kw)
    raise ValueError(model)


def _rotate(v, s, n):
    """Bit masks v rotated left by s within n bits (uint64 arrays)."""
    n64, one = np.uint64(n), np.uint64(1)
    mask = (one << n64) - one
    return np.where(s == 0, v, ((v << s) | (v >> ((n64 - s) % n64))) & mask)


def _records(case, rng):
    """Strings of weight at most wmax (the case's), each in `dup` random
    rotations, with coefficients over four decades; also the unrotated
    strings and their row numbers."""
    n, rows = case["n"], case["rows"]
    nbase = max(1, rows // case["dup"])
    seeded, rng = rng, np.random.default_rng(n)
    w = rng.integers(1, case["wmax"] + 1, size=nbase)
    pos = np.argsort(rng.random((nbase, n), dtype=np.float32), axis=1)[:, :case["wmax"]]
    letters = rng.integers(1, 4, size=pos.shape)
    sel = np.arange(pos.shape[1])[None, :] < w[:, None]
    one = np.uint64(1)
    bit = one << pos.astype(np.uint64)
    rng = seeded
    x = np.where(sel & (letters != 3), bit, 0).sum(axis=1, dtype=np.uint64)
    z = np.where(sel & (letters != 1), bit, 0).sum(axis=1, dtype=np.uint64)
    base = rng.permutation(np.resize(np.arange(nbase), rows))
    s = rng.integers(0, n, size=rows).astype(np.uint64)
    coef = rng.normal(size=rows) * 10.0 ** rng.uniform(-4, 0, size=rows)
    return x, z, base, s, coef


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    st = dict(case=case, allocator=L.TorchAllocator(0), stream=torch.cuda.Stream())
    st["handle"] = int(st["stream"].cuda_stream)
    if case["kind"] == "ingest":
        x, z, base, s, coef = _records(case, rng)
        st["rows"] = (_rotate(x[base], s, case["n"]).reshape(-1, 1),
                      _rotate(z[base], s, case["n"]).reshape(-1, 1), coef)
        st["bloch"] = _bloch(rng)
    elif case["kind"] == "batch":
        progs = []
        for k in range(case["count"]):           # sizes and depths around the case's
            n = max(8, case["n"] - 8 * (k % 4))
            progs.append(_program(case, rng, n, 1 + (case["steps"] - 1) * (k + 1) // case["count"]))
        st["progs"] = progs
        st["device"] = [driver.DeviceProgram(p) for p in progs]
    else:
        st["prog"] = _program(case, rng)
        if case["kind"] == "calls":
            st["layers"] = driver.heisenberg_layers(st["prog"])
        else:
            st["device"] = driver.DeviceProgram(st["prog"])
    torch.cuda.synchronize()
    return st


def _set(st, prog):
    return driver.PauliSet.from_program(prog, None, st["handle"], st["allocator"],
                                        st["case"]["dtype"])


def _result(ps, expectation):
    x, z, c = ps.export()
    return dict(expectation=float(expectation), x=x.view(np.int64), z=z.view(np.int64), coef=c)


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "program":
        ps = _set(st, st["prog"])
        e = L.pp_batch_run([ps.h], [st["device"].h], st["handle"])[0]
        out = _result(ps, e)
        ps.close()
        return out
    if kind == "calls":
        ps = _set(st, st["prog"])
        driver.run_layers(ps, st["layers"])
        out = _result(ps, ps.expectation(st["prog"].bloch))
        ps.close()
        return out
    if kind == "batch":
        sets = [_set(st, p) for p in st["progs"]]
        e = L.pp_batch_run([s.h for s in sets], [d.h for d in st["device"]], st["handle"])
        out = [_result(s, v) for s, v in zip(sets, e)]
        for s in sets:
            s.close()
        return out
    x, z, c = st["rows"]
    ps = driver.PauliSet(case["n"], case["group"], x, z, c, st["handle"], st["allocator"],
                         case["dtype"])
    out = _result(ps, ps.expectation(st["bloch"]))
    ps.close()
    return out


# ---------------------------------------------------------------------------
# work and the 64-bit values
# ---------------------------------------------------------------------------
_WORK = {}


def work(case):
    """Bytes: for every sub-layer (or the ingest) its set read once and the
    representatives it leaves written once.  Operations: three per
    anticommuting string and rotation (cos c - sin d).  How far a set grows
    is only known by running it, so the counts come from the library's work
    counters (which the tests hold equal to the CPU oracle's)."""
    key = repr(sorted((k, v) for k, v in case.items() if k != "name"))
    if key in _WORK:
        return dict(_WORK[key])
    st = prepare(case, 1)
    rec = 16 * W.n_words(case["n"]) + (4 if case["dtype"] == "f32" else 8)
    counts = []
    if case["kind"] == "ingest":
        x, z, c = st["rows"]
        ps = driver.PauliSet(case["n"], case["group"], x, z, c, st["handle"], st["allocator"],
                             case["dtype"])
        counts.append((len(c) + ps.num_terms(), 0))
        ps.close()
    else:
        progs = st.get("progs") or [st["prog"]]
        for p in progs:
            ps = _set(st, p)
            dp = driver.DeviceProgram(p)
            L.pp_batch_run([ps.h], [dp.h], st["handle"])
            wc = L.pp_work_counters(ps.h)
            counts.append((2 * wc["merge_out"], 3 * wc["anticommuting"]))
            ps.close()
            dp.close()
    _WORK[key] = dict(bytes=float(rec * sum(a for a, _ in counts)),
                      flops=float(sum(b for _, b in counts)))
    return dict(_WORK[key])


def _letters_key(x, z):
    """The integer that orders strings: qubit q the base-4 digit of weight
    4^q, I X Y Z = 0 1 2 3 (one-word strings, n <= 32)."""
    def spread(v):
        v = v & np.uint64(0xFFFFFFFF)
        for s, m in ((16, 0x0000FFFF0000FFFF), (8, 0x00FF00FF00FF00FF), (4, 0x0F0F0F0F0F0F0F0F),
                     (2, 0x3333333333333333), (1, 0x5555555555555555)):
            v = (v | (v << np.uint64(s))) & np.uint64(m)
        return v
    return (spread(z) << np.uint64(1)) | spread(x ^ z)


def _parity(v):
    for s in (32, 16, 8, 4, 2, 1):
        v = v ^ (v >> np.uint64(s))
    return (v & np.uint64(1)).astype(bool)


def _count(v):
    v = v - ((v >> np.uint64(1)) & np.uint64(0x5555555555555555))
    v = (v & np.uint64(0x3333333333333333)) + ((v >> np.uint64(2)) & np.uint64(0x3333333333333333))
    v = (v + (v >> np.uint64(4))) & np.uint64(0x0F0F0F0F0F0F0F0F)
    return ((v * np.uint64(0x0101010101010101)) >> np.uint64(56)).astype(np.int64)


def _reflect(v, n):
    out = np.zeros_like(v)
    for q in range(n):
        out |= ((v >> np.uint64(q)) & np.uint64(1)) << np.uint64(n - 1 - q)
    return out


def _merge(x, z, c, n, group):
    """Orbit representatives (the smallest integer of each orbit) and the
    exact orbit sums (extended precision, rounded once), in key order."""
    images = []
    if group in ("Zn", "Dn"):
        for s in range(n):
            sh = np.full(len(x), s, dtype=np.uint64)
            images.append((_rotate(x, sh, n), _rotate(z, sh, n)))
        if group == "Dn":
            images += [(_reflect(a, n), _reflect(b, n)) for a, b in images]
    else:
        images.append((x, z))
    bx, bz = images[0]
    bk = _letters_key(bx, bz)
    for a, b in images[1:]:
        k = _letters_key(a, b)
        less = k < bk
        bx, bz, bk = np.where(less, a, bx), np.where(less, b, bz), np.where(less, k, bk)
    keys, first, inv = np.unique(bk, return_index=True, return_inverse=True)
    sums = np.zeros(len(keys), dtype=np.longdouble)
    np.add.at(sums, inv.reshape(-1), c.astype(np.longdouble))
    return bx[first], bz[first], sums.astype(np.float64)


def _expect(x, z, c, bloch):
    v = c.astype(np.longdouble)
    for count, b in ((_count(x & ~z), bloch[0]), (_count(x & z), bloch[1]),
                     (_count(z & ~x), bloch[2])):
        v = v * np.longdouble(b) ** count
    return float(v.sum())


def _gate(x, z, c, g):
    """exp(-i theta/2 P) in the Heisenberg picture on a set of distinct strings."""
    px, pz = np.uint64(g.x), np.uint64(g.z)
    anti = _parity((x & pz) ^ (z & px))
    qx, qz, q = x[anti], z[anti], c[anti]
    rx, rz = qx ^ px, qz ^ pz
    phi = (_count(np.broadcast_to(px & pz, qx.shape)) + _count(qx & qz) + 2 * _count(pz & qx) -
           _count(rx & rz))
    child = np.where(phi % 4 == 3, 1.0, -1.0) * (math.sin(g.theta) * q)
    c = c.copy()
    c[anti] = math.cos(g.theta) * q
    key = _letters_key(x, z)
    order = np.argsort(key, kind="stable")
    rk = _letters_key(rx, rz)
    at = np.minimum(np.searchsorted(key, rk, sorter=order), max(len(key) - 1, 0))
    hit = key[order[at]] == rk if len(key) else np.zeros(0, bool)
    np.add.at(c, order[at[hit]], child[hit])
    return (np.concatenate([x, rx[~hit]]), np.concatenate([z, rz[~hit]]),
            np.concatenate([c, child[~hit]]))


def exact(case, seed):
    """Plain numpy in 64 bits (orbit sums and the expectation in extended
    precision): the untruncated small circuits and the ingest."""
    rng = np.random.default_rng(seed)
    n = case["n"]
    if case["kind"] == "ingest":
        x, z, base, s, coef = _records(case, rng)
        bloch = _bloch(rng)
        if case["dtype"] == "f32":
            coef = coef.astype(np.float32).astype(np.float64)
        if case["group"] == "Dn" and case["rows"] // case["dup"] > 1 << 18:
            return None
        x, z, c = _merge(x[base] if case["dup"] == 1 else x, z[base] if case["dup"] == 1 else z,
                         coef if case["dup"] == 1 else _sum_by(base, coef, len(x)), n,
                         case["group"])
    else:
        small = n <= 8 or (n == 9 and case["steps"] <= 4)
        if case["kind"] != "program" or case["model"] not in ("xxz", "ising") or \
                case["eps"] > 0 or case["wmax"] >= 0 or not small:
            return None
        prog = _program(case, rng)
        x = np.array([o[0] for o in prog.obs], dtype=np.uint64)
        z = np.array([o[1] for o in prog.obs], dtype=np.uint64)
        c = np.array([o[2] for o in prog.obs], dtype=np.float64)
        x, z, c = _merge(x, z, c, n, case["group"])
        for sub in reversed(prog.sublayers):
            for g in reversed(sub.gates):
                x, z, c = _gate(x, z, c, g)
            if sub.merge:
                x, z, c = _merge(x, z, c, n, case["group"])
        bloch = prog.bloch
        order = np.argsort(_letters_key(x, z))
        x, z, c = x[order], z[order], c[order]
    return dict(expectation=_expect(x, z, c, bloch), x=x.reshape(-1, 1).view(np.int64),
                z=z.reshape(-1, 1).view(np.int64), coef=c)


def _sum_by(base, coef, count):
    """Sum of the coefficients of each unrotated string (a rotation stays in
    its orbit), in extended precision."""
    out = np.zeros(count, dtype=np.longdouble)
    np.add.at(out, base, coef.astype(np.longdouble))
    return out
