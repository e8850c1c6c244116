"""Calls that a handle's limits or its allocator refuse leave the handle usable
and exact: a refused call repeated without the store growing, a program stopped
inside a sub-layer and resumed, memory that is not to be had for a layer op.
What runs afterwards equals, bitwise, a handle that met no refusal."""
import numpy as np
import pytest

from paper_2512_12094_amd import workloads as W

pytestmark = pytest.mark.gpu

CAPACITY, NOMEM = -4, -3


@pytest.fixture(scope="module")
def gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2512_12094_amd import _lib
    _lib.lib()
    torch.cuda.set_device(0)
    stream = torch.cuda.Stream()
    return dict(torch=torch, stream=stream, handle=int(stream.cuda_stream),
                alloc=_lib.TorchAllocator(0))


class Refusing:
    """A caller's allocator that refuses what `deny(bytes)` names; `held` is
    what the library has from it."""

    def __init__(self, inner, deny=lambda nbytes: False):
        from paper_2512_12094_amd import _lib as L
        self.inner, self.deny, self.held, self.refused = inner, deny, {}, 0

        def alloc(nbytes, stream, ctx):
            if self.deny(nbytes):
                self.refused += 1
                return None
            p = inner._alloc(nbytes, stream, ctx)
            if p:
                self.held[p] = nbytes
            return p

        def free(p, stream, ctx):
            self.held.pop(p, None)
            inner._free(p, stream, ctx)

        self._alloc, self._free = L.ALLOC_FN(alloc), L.FREE_FN(free)
        self.struct = L.PPAllocator(self._alloc, self._free, None)


def staging(nbytes):
    """The layer op's staging arrays: 8 bytes for each of a power of two of slots
    (a store is one allocation of another size)."""
    return nbytes >= 1 << 16 and nbytes & (nbytes - 1) == 0


def layer(gates, eps=0.0, wmax=-1):
    from paper_2512_12094_amd import driver
    prog = W.Program("layer", 20, "none", [], [W.SubLayer(gates, eps=eps, wmax=wmax)],
                     W.ZERO_STATE, {})
    return driver.heisenberg_layers(prog)[0]


def strings(n, rows, seed):
    rng = np.random.default_rng(seed)
    x = rng.permutation(1 << n)[:rows].astype(np.uint64).reshape(-1, 1)
    z = rng.integers(0, 1 << n, size=(rows, 1), dtype=np.uint64)
    return x, z, rng.normal(size=rows)


@pytest.mark.parametrize("grow", [False, True])
def test_refused_calls_leave_the_gate_table_usable(gpu, grow):
    """A merge leaves the gate table to the next call's recount.  Calls that
    are refused at the store limit (without a growth, or after one) enter the
    set and give it back; after ten of them the table still finds every
    string."""
    from paper_2512_12094_amd import _lib as L
    from paper_2512_12094_amd import driver
    print(f"[case] refused calls, grow {grow}", flush=True)
    x, z, c = strings(20, 1500, 3)
    x[:, 0] &= np.uint64(0xFFFFF)
    z[:, 0] &= np.uint64(0x7FFFF)                     # Z on qubit 19: few strings
    z[:40, 0] |= np.uint64(1 << 19)
    big = layer([W.Gate(1 << q, 0, 0.3) if q % 2 else W.Gate(0, 1 << q, 0.4)
                 for q in range(10)] + [W.Gate(1 << q, 1 << q, 0.2) for q in range(10)])
    fits = layer([W.Gate(1 << 19, 0, 0.3), W.Gate(1 << 19, 0, 0.5), W.Gate(1 << 19, 0, 0.7)])

    def fresh():
        ps = driver.PauliSet(20, "none", x, z, c, gpu["handle"], gpu["alloc"])
        ps.merge()
        return ps

    ref, ps = fresh(), fresh()
    L.pp_set_max_terms(ps.h, 16384 if grow else 4096)
    before = (ps.as_dict(), ps.counters())
    for _ in range(10):
        with pytest.raises(L.PPError) as e:
            ps.apply_layer(big)
        assert e.value.code == CAPACITY and "as before the call" in str(e.value)
    assert (ps.as_dict(), ps.counters()) == before
    for s in (ref, ps):
        s.apply_layer(fits)
        s.apply_layer(fits)
    assert ps.as_dict() == ref.as_dict()
    assert ps.counters() == ref.counters()
    ref.close()
    ps.close()


def wide_program():
    """120 commuting rotations on one string that 15 of them anticommute with
    (2^15 strings), fields, then 120 more."""
    pairs = lambda k, t: [W.Gate(*W.two_site(k, a, b), t) for a in range(16) for b in range(a)]
    subs = [W.SubLayer(pairs("Z", 0.11), eps=2e-3, wmax=9),
            W.SubLayer([W.Gate(0, 1 << q, 0.2) for q in range(16)], eps=1e-3),
            W.SubLayer(pairs("X", 0.4), wmax=12)]      # applied last to first
    return W.Program("wide16", 16, "none", [(0, 1, 1.0), (0, 0b10010, 0.5), (0b11, 0, 0.25)],
                     subs, W.ZERO_STATE, {})


@pytest.mark.parametrize("limit", [40, 700, 6000])
@pytest.mark.parametrize("both", [False, True])
def test_program_resumes_inside_a_wide_sublayer(gpu, limit, both):
    """pp_batch_run is refused inside a sub-layer of more than 64 rotations;
    the batched form then resumes the program, alone or beside another."""
    from paper_2512_12094_amd import _lib as L
    from paper_2512_12094_amd import driver
    prog = wide_program()
    print(f"[case] resume in a wide sub-layer, limit {limit}, both {both}", flush=True)
    dp = driver.DeviceProgram(prog)
    make = lambda: driver.PauliSet.from_program(prog, None, gpu["handle"], gpu["alloc"])
    ref, ps, other = make(), make(), make()
    want = float(L.pp_batch_run([ref.h], [dp.h], gpu["handle"])[0])
    L.pp_set_max_terms(ps.h, 4096 + limit)
    with pytest.raises(L.PPError) as e:
        L.pp_batch_run([ps.h], [dp.h], gpu["handle"])
    assert e.value.code == CAPACITY
    assert ps.num_terms() > 3                          # inside the sub-layer
    L.pp_set_max_terms(ps.h, 0)
    sets = [other, ps] if both else [ps]
    for _ in range(200):
        done, got = L.pp_batch_step([s.h for s in sets], [dp.h] * len(sets), gpu["handle"], 8)
        assert (done >= 0).all()
        if done.all():
            break
    assert done.all() and all(float(g) == want for g in got)
    for s in sets:
        assert s.as_dict() == ref.as_dict()
        assert s.counters() == ref.counters()
    for s in (ref, ps, other):
        s.close()
    dp.close()


def crowded_set():
    """All 2^11 strings of one closed set, which no bucket's share of the
    staging holds, and 511 strings that commute with everything: rotating them
    makes no new string."""
    k = 11
    obs = [(s, (1 << k) - 1, 1.0 / (1 + s)) for s in range(1 << k)]
    obs += [(s, 0, 0.5 + s / 1024) for s in range(1, 512)]
    xs = [W.Gate(1 << q, 0, 0.3 + 0.01 * q) for q in range(k)]
    return W.Program("crowded", 12, "none", obs, [W.SubLayer(xs), W.SubLayer(xs[::-1])],
                     W.ZERO_STATE, {})


@pytest.mark.parametrize("form", ["calls", "program"])
def test_staging_overflow_at_the_store_limit(gpu, form):
    """A layer op whose staging overflows in a store that may not grow goes on
    to exact placement."""
    from paper_2512_12094_amd import _lib as L
    from paper_2512_12094_amd import driver
    prog = crowded_set()
    print(f"[case] staging overflow at the limit, {form}", flush=True)
    out = {}
    for mode in (0, 1):
        L.pp_set_layer_ops(mode)
        try:
            dp = driver.DeviceProgram(prog)
            ps = driver.PauliSet.from_program(prog, None, gpu["handle"], gpu["alloc"])
            if mode:
                L.pp_set_max_terms(ps.h, 2 * len(prog.obs))      # the capacity it has
            if form == "calls":
                driver.run_layers(ps, driver.heisenberg_layers(prog))
            else:
                L.pp_batch_run([ps.h], [dp.h], gpu["handle"])
            out[mode] = (ps.as_dict(), ps.counters())
            st = L.pp_layer_stats(ps.h)
            ps.close()
            dp.close()
        finally:
            L.pp_set_layer_ops(1)
    assert out[0] == out[1]
    assert st["layer_ops"] == 2 and st["fallbacks"] == 0 and st["overflow_runs"] > 0, st


@pytest.mark.parametrize("form", ["calls", "program", "batch"])
def test_no_memory_for_the_layer_staging(gpu, form):
    """Without memory for a layer op's staging its gate launches run."""
    from paper_2512_12094_amd import _lib as L
    from paper_2512_12094_amd import driver
    prog = W.xxz_ring(16, 2, 0.3, 0.8, eps=1e-7, name="z16")
    print(f"[case] no memory for the layer staging, {form}", flush=True)
    dp = driver.DeviceProgram(prog)

    def run(alloc, mode):
        L.pp_set_layer_ops(mode)
        try:
            sets = [driver.PauliSet.from_program(prog, None, gpu["handle"], alloc)
                    for _ in range(2 if form == "batch" else 1)]
            if form == "calls":
                driver.run_layers(sets[0], driver.heisenberg_layers(prog))
            else:
                L.pp_batch_run([s.h for s in sets], [dp.h] * len(sets), gpu["handle"])
        finally:
            L.pp_set_layer_ops(1)
        out = [(s.as_dict(), s.counters(), L.pp_layer_stats(s.h)["layer_ops"]) for s in sets]
        return sets, out

    plain, want = run(gpu["alloc"], 0 if form == "calls" else 1)
    short = Refusing(gpu["alloc"], staging)
    tight, got = run(short, 1)
    assert short.refused
    for g, w in zip(got, want):
        assert g[:2] == w[:2] and g[2] == 0
    short.deny = lambda nbytes: False                  # memory again: layer ops again
    if form == "calls":
        la = driver.heisenberg_layers(prog)[0]
        for s in (plain[0], tight[0]):
            s.apply_layer(la)
        assert L.pp_layer_stats(tight[0].h)["layer_ops"] == 1
        assert tight[0].as_dict() == plain[0].as_dict()
    for s in plain + tight:
        s.close()
    dp.close()
    assert not short.held


def test_refused_calls_keep_one_staging(gpu):
    """Layer ops refused at the store limit, with and without exact placement,
    hold one staging between them, whatever the number of calls."""
    from paper_2512_12094_amd import _lib as L
    from paper_2512_12094_amd import driver
    print("[case] one staging", flush=True)
    prog = crowded_set()
    alloc = Refusing(gpu["alloc"])
    ps = driver.PauliSet.from_program(prog, None, gpu["handle"], alloc)
    plain = sum(alloc.held.values())
    L.pp_set_max_terms(ps.h, 2 * len(prog.obs))
    fields = layer([W.Gate(0, 1 << q, 0.3) for q in range(12)])       # outgrows the store
    before = (ps.as_dict(), ps.counters())
    held = []
    for k in range(6):
        with pytest.raises(L.PPError) as e:
            ps.apply_layer(fields)
        assert e.value.code == CAPACITY
        held.append(sum(alloc.held.values()))
    assert (ps.as_dict(), ps.counters()) == before
    assert len(set(held[1:])) == 1, held
    # exact placement adds 16 bytes an entry and the bucket bases to what is there
    for la in driver.heisenberg_layers(prog):
        ps.apply_layer(la)
    cap, slots = 2 * len(prog.obs), 1 << 15            # 5118 entries: four times 2^13 slots
    exact = 16 * cap + 4 * (slots >> 6)
    stats = L.pp_layer_stats(ps.h)
    assert stats["layer_ops"] == 2 and stats["fallbacks"] == 0, stats
    assert held[-1] < sum(alloc.held.values()) <= held[-1] + exact + 4 * 256
    assert held[-1] - plain < 33 * slots + (1 << 17)   # the staging and the call's backup
    ps.close()
    assert not alloc.held


@pytest.mark.parametrize("staged", [True, False])
@pytest.mark.parametrize("form", ["calls", "program", "batch"])
def test_growth_without_memory_for_the_staging(gpu, form, staged):
    """A store that can be had only without the layer op's staging grows
    without it; the staging is asked for again by the next layer op (`staged`:
    and given)."""
    from paper_2512_12094_amd import _lib as L
    from paper_2512_12094_amd import driver
    prog = W.xxz_ring(16, 2, 0.3, 0.8, eps=1e-7, name="z16")
    print(f"[case] growth without the staging, {form}, staged {staged}", flush=True)
    dp = driver.DeviceProgram(prog)
    short = Refusing(gpu["alloc"])

    def run(alloc):
        sets = [driver.PauliSet.from_program(prog, None, gpu["handle"], alloc)
                for _ in range(2 if form == "batch" else 1)]
        if alloc is short:
            def deny(nbytes):                          # the first store it grows into
                return (nbytes >= 1 << 20 and not short.refused) or \
                    (short.refused > 0 and not staged and staging(nbytes))
            short.deny = deny
        if form == "calls":
            driver.run_layers(sets[0], driver.heisenberg_layers(prog))
        else:
            L.pp_batch_run([s.h for s in sets], [dp.h] * len(sets), gpu["handle"])
        return sets, [(s.as_dict(), s.counters()) for s in sets]

    plain, want = run(gpu["alloc"])
    tight, got = run(short)
    assert short.refused and got == want
    stats = L.pp_layer_stats(tight[0].h)
    assert stats["layer_ops"] > 0 and stats["fallbacks"] == 0, stats
    for s in plain + tight:
        s.close()
    dp.close()
    assert not short.held


def test_growth_without_memory_for_exact_placement(gpu):
    """A store that can be had only without what exact placement adds."""
    from paper_2512_12094_amd import _lib as L
    from paper_2512_12094_amd import driver
    print("[case] growth without exact placement", flush=True)
    prog = crowded_set()
    fields = layer([W.Gate(0, 1 << q, 0.3) for q in range(12)])
    short = Refusing(gpu["alloc"])
    sets = [driver.PauliSet.from_program(prog, None, gpu["handle"], a) for a in (gpu["alloc"], short)]
    for s in sets:
        L.pp_set_max_terms(s.h, 2 * len(prog.obs))
        driver.run_layers(s, driver.heisenberg_layers(prog))       # exact from here on
        L.pp_set_max_terms(s.h, 0)
        short.deny = lambda nbytes: nbytes >= 1 << 20 and not short.refused
        s.apply_layer(fields)
    assert short.refused == 1
    assert sets[0].as_dict() == sets[1].as_dict()
    assert sets[0].counters() == sets[1].counters()
    for s in sets:
        s.close()
    assert not short.held


def test_call_backup_takes_what_there_is_and_goes_back(gpu):
    """The copy a call may roll back to: without memory for its headroom the
    bytes it needs do, and a large one is not kept between calls."""
    from paper_2512_12094_amd import driver
    print("[case] call backup", flush=True)
    alloc = Refusing(gpu["alloc"])
    x, z, c = strings(20, 1500, 5)
    ps = driver.PauliSet(20, "none", x, z, c, gpu["handle"], alloc)
    alloc.deny = lambda nbytes: nbytes > 2 * 9 * 1500 and not alloc.refused
    ps.merge()
    assert alloc.refused == 1 and ps.num_terms() == 1500
    ps.close()
    rows = 1 << 21
    i = np.arange(rows, dtype=np.uint64).reshape(-1, 1)
    ps = driver.PauliSet(24, "none", i, np.zeros_like(i), np.ones(rows), gpu["handle"], alloc)
    before = sum(alloc.held.values())
    ps.merge()
    assert sum(alloc.held.values()) < before + (1 << 20)
    assert ps.num_terms() == rows
    ps.close()
    assert not alloc.held


def test_growth_gives_up_the_workspace_of_large_buckets(gpu):
    """A store that cannot be had beside the workspace of buckets in HBM (which
    a closed set of 2^13 strings asked for) is had without it."""
    from paper_2512_12094_amd import _lib as L
    from paper_2512_12094_amd import driver
    print("[case] growth without the large buckets' workspace", flush=True)
    k = 13
    fields = [layer([W.Gate(x << q, z << q, 0.3 + 0.01 * q) for q in range(k)])
              for x, z in ((1, 0), (0, 1))]
    alloc = Refusing(gpu["alloc"])
    sets = [driver.PauliSet(20, "none", [[0]], [[(1 << k) - 1]], [1.0], gpu["handle"], a)
            for a in (gpu["alloc"], alloc)]
    huge = lambda: [b for b in alloc.held.values() if (64 << 20) < b < (256 << 20)]
    for s in sets:
        s.apply_layer(fields[0])                       # 2^13 strings in one closed set
        assert L.pp_layer_stats(s.h)["fallbacks"] == 0
    assert huge()
    more = layer([W.Gate(0, 1 << q, 0.1) for q in range(3)])       # gate launches
    for s in sets:
        alloc.deny = lambda nbytes: nbytes >= 1 << 20 and bool(huge())
        for _ in range(4):
            s.apply_layer(more)
        s.apply_layer(layer([W.Gate(1 << 15, 1 << q, 0.2) for q in range(2)]))
    assert alloc.refused and not huge()
    assert sets[0].as_dict() == sets[1].as_dict()
    assert sets[0].counters() == sets[1].counters()
    for s in sets:
        s.close()
    assert not alloc.held


@pytest.mark.parametrize("what", ["exact", "huge"])
def test_no_memory_for_what_a_failing_layer_op_lacks(gpu, what):
    """Exact placement, or the workspace of buckets in HBM, that cannot be had:
    the op's gate launches run (and with memory again, exact placement)."""
    from paper_2512_12094_amd import _lib as L
    from paper_2512_12094_amd import driver
    print(f"[case] no memory for {what}", flush=True)
    if what == "exact":
        prog = crowded_set()
        size = 8 * 2 * len(prog.obs)                   # the patterns, one per entry
        deny = lambda nbytes: size <= nbytes < size + 256
    else:
        xs = [W.Gate(1 << q, 0, 0.3 + 0.01 * q) for q in range(13)]
        prog = W.Program("field13", 13, "none", [(0, (1 << 13) - 1, 1.0)],
                         [W.SubLayer(xs), W.SubLayer(xs[::-1])], W.ZERO_STATE, {})
        deny = lambda nbytes: (64 << 20) < nbytes < (256 << 20)
    layers = driver.heisenberg_layers(prog)
    alloc = Refusing(gpu["alloc"], deny)
    sets = [driver.PauliSet.from_program(prog, None, gpu["handle"], a)
            for a in (gpu["alloc"], alloc)]
    if what == "exact":
        L.pp_set_max_terms(sets[1].h, 2 * len(prog.obs))
        L.pp_set_gate_fusion(1)                        # (fused launches ask for more room)
    try:
        for s in sets:
            s.apply_layer(layers[0])
    finally:
        L.pp_set_gate_fusion(3)
    stats = L.pp_layer_stats(sets[1].h)
    assert alloc.refused and stats["fallbacks"] == 1 and stats["layer_ops"] == 0, stats
    alloc.deny = lambda nbytes: False
    L.pp_set_max_terms(sets[1].h, 0)
    for s in sets:
        s.apply_layer(layers[1])
    if what == "exact":
        stats = L.pp_layer_stats(sets[1].h)
        assert stats["fallbacks"] == 1 and stats["layer_ops"] == 1, stats
    assert sets[0].as_dict() == sets[1].as_dict()
    assert sets[0].counters() == sets[1].counters()
    for s in sets:
        s.close()
    assert not alloc.held


@pytest.mark.parametrize("both", [False, True])
def test_program_resumes_at_the_start_of_a_wide_sublayer(gpu, both):
    """The refusal meets the first rotations of the sub-layer, with none
    applied: the batched form finishes the program all the same."""
    from paper_2512_12094_amd import _lib as L
    from paper_2512_12094_amd import driver
    print(f"[case] resume at the start of a wide sub-layer, both {both}", flush=True)
    x, z, c = strings(16, 2000, 9)
    obs = [(int(a), int(b), float(v)) for a, b, v in zip(x[:, 0], z[:, 0], c)]
    pairs = [W.Gate(*W.two_site("X", a, b), 0.2) for a in range(16) for b in range(a)]
    prog = W.Program("start16", 16, "none", obs,
                     [W.SubLayer([W.Gate(0, 1 << q, 0.2) for q in range(16)], eps=0.1),
                      W.SubLayer(pairs, eps=0.3, wmax=13)], W.ZERO_STATE, {})
    dp = driver.DeviceProgram(prog)
    make = lambda: driver.PauliSet.from_program(prog, None, gpu["handle"], gpu["alloc"])
    ref, ps, other = make(), make(), make()
    want = float(L.pp_batch_run([ref.h], [dp.h], gpu["handle"])[0])
    L.pp_set_max_terms(ps.h, 4096)
    with pytest.raises(L.PPError) as e:
        L.pp_batch_run([ps.h], [dp.h], gpu["handle"])
    assert e.value.code == CAPACITY and ps.num_terms() == len(obs)
    L.pp_set_max_terms(ps.h, 0)
    sets = [other, ps] if both else [ps]
    for _ in range(200):
        done, got = L.pp_batch_step([s.h for s in sets], [dp.h] * len(sets), gpu["handle"], 8)
        if done.all():
            break
    assert (done == 1).all() and all(float(g) == want for g in got)
    for s in sets:
        assert s.as_dict() == ref.as_dict()
        assert s.counters() == ref.counters()
    for s in (ref, ps, other):
        s.close()
    dp.close()
