"""Handles: rows uploaded into a new store (sizes around the words the
liveness flags are written in, one and two key words, both coefficient types)
come out of the export unchanged, and handles made and destroyed by several
threads on their own streams, which take each other's pinned blocks, give the
results of one at a time."""
import threading

import numpy as np
import pytest

from paper_2512_12094_amd import workloads as W

pytestmark = pytest.mark.gpu


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


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n,rows", [(20, 0), (20, 1), (20, 7), (20, 9), (20, 2047), (20, 5001),
                                    (70, 1), (70, 15), (70, 5001)])
def test_rows_come_back(gpu, n, rows, dtype):
    from paper_2512_12094_amd import driver
    words = W.n_words(n)
    rng = np.random.default_rng(rows + n)
    x = np.zeros((rows, words), dtype=np.uint64)
    z = np.zeros((rows, words), dtype=np.uint64)
    x[:, 0] = np.arange(rows, dtype=np.uint64)                     # distinct strings
    for w in range(words):
        bits = min(64, n - 64 * w)
        z[:, w] = rng.integers(0, 1 << min(bits, 62), size=rows, dtype=np.uint64)
    if words > 1:
        x[:, 1] = rng.integers(0, 1 << (n - 64), size=rows, dtype=np.uint64)
    c = rng.normal(size=rows)
    if dtype == "f32":
        c = c.astype(np.float32).astype(np.float64)
    print(f"[case] rows {rows} n {n} {dtype}", flush=True)
    ps = driver.PauliSet(n, "none", x, z, c, gpu["handle"], gpu["alloc"], dtype)
    ox, oz, oc = ps.export()
    ps.close()
    got = sorted(zip(map(tuple, ox.tolist()), map(tuple, oz.tolist()), oc.tolist()))
    want = sorted(zip(map(tuple, x.tolist()), map(tuple, z.tolist()), c.tolist()))
    assert got == want


def test_threads_share_the_pinned_blocks(gpu):
    from paper_2512_12094_amd import _lib as L
    from paper_2512_12094_amd import driver
    torch = gpu["torch"]
    progs = [W.config1(), W.xxz_ring(16, 2, 0.3, 0.8, eps=1e-7, name="z16"),
             W.tilted_ising_ring(8, 2, 0.25)]
    dps = [driver.DeviceProgram(p) for p in progs]

    def once(k, stream, alloc):
        h = int(stream.cuda_stream)
        ps = driver.PauliSet.from_program(progs[k], None, h, alloc)
        e = float(L.pp_batch_run([ps.h], [dps[k].h], h)[0])
        out = (e, ps.as_dict())
        ps.close()
        return out

    want = [once(k, gpu["stream"], gpu["alloc"]) for k in range(len(progs))]
    got, errors = {}, []

    def work(t):
        try:
            torch.cuda.set_device(0)
            stream, alloc = torch.cuda.Stream(), L.TorchAllocator(0)
            for rep in range(4):
                k = (t + rep) % len(progs)
                got[t, rep] = (k, once(k, stream, alloc))
        except Exception as exc:                                   # reported below
            errors.append(exc)

    print("[case] four threads", flush=True)
    threads = [threading.Thread(target=work, args=(t,)) for t in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    assert len(got) == 16
    for k, out in got.values():
        assert out == want[k]
    for d in dps:
        d.close()
