"""GPU tests of scratch that cannot be allocated.

HGT_ALLOC_MAX=bytes makes every larger device allocation of the library fail on
the host, as if memory had run out; no kernel runs without its buffers.
"""
import numpy as np
import pytest

from paper_2512_21009_amd import workloads as W

from .gpu_harness import Pair, compare_counts, compare_store

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("route", ["batch", "round", "graph"])
def test_scratch_that_does_not_fit_refuses_the_batch(gpu_lib, monkeypatch, route):
    """40 hyperedges built, then 20 deletions and 600 insertions whose 2-hop tables
    (8 MB) are refused after the batch was planned: HGT_ENOMEM, the graph as it was and
    not poisoned; with the memory back the same batch matches the oracle."""
    import torch
    hgt = gpu_lib
    st = W.plain_stream("refused", 60, 40, ("uniform", 6, 6), 0.0, 0.0, 1, 600, 20, W.SEED_BASE + 160)
    p = Pair(st, track=("hyperedge",))
    args, finish = p.prepare(st.batches[0], "refused")

    def apply():
        if route == "batch":
            return p.g.apply_batch(*args, raise_on_error=False)
        rc, status, outs = hgt.apply_batches([(p.g,) + args], raise_on_error=False, graph=route == "graph")
        assert status == [rc]
        return rc, outs[0]

    monkeypatch.setenv("HGT_ALLOC_MAX", str(4 << 20))
    rc, _ = apply()
    assert rc == hgt.ENOMEM
    compare_store(p.g, p.o, "refused")
    compare_counts(p.g, p.o, p.track, "refused")
    monkeypatch.delenv("HGT_ALLOC_MAX")
    rc, out = apply()
    torch.cuda.synchronize()
    assert rc == hgt.OK
    finish(out)
    compare_store(p.g, p.o, "applied")
    compare_counts(p.g, p.o, p.track, "applied")
    p.close()


def test_temporal_lists_that_do_not_fit(gpu_lib, monkeypatch):
    """The lists of the temporal family (4 to 8 bytes a column and entry of 29M) refused at
    the first column and at the third: the 2-hop kernels give the counts that the lists
    give, and what was taken for the first columns is not kept."""
    import torch
    monkeypatch.setenv("HGT_WAVE_SLOTS", "4096")  # per-wave hashes of 64 MB in all
    st = W.temporal_stream("lists", 50, 1000, 9000, 1, 50.0, 4, 4, 100.0, 10**7, 800, W.SEED_BASE + 161)

    def run(limit):
        monkeypatch.setenv("HGT_ALLOC_MAX", str(limit))
        torch.cuda.empty_cache()
        free = torch.cuda.mem_get_info()[0]
        p = Pair(W.Stream("lists", st.n_vertices, st.initial, window=st.window), track=("temporal",))
        p.g.profile(True)
        args, _ = p.prepare(st.batches[0], "lists")
        p.g.apply_batch(*args)
        counts = p.g.triad_counts("temporal")
        held = free - torch.cuda.mem_get_info()[0]
        expanded = p.g.profile_read()["temporal"]["events"]  # by the 2-hop kernels
        p.close()
        return counts, held, expanded

    want, most, none = run(1 << 40)
    one, held1, n1 = run(100 << 20)
    three, held3, n3 = run(200 << 20)
    assert sum(want) > 0 and one == want and three == want
    assert none == 0 and n1 == n3 > 0
    assert most > held1 + (700 << 20)
    assert abs(held3 - held1) < 64 << 20, (held1, held3)


def test_temporal_lists_leave_and_return_memory(gpu_lib, monkeypatch):
    """Lists as above (0.8 GB) where 1.5 GB are free: not taken, the 2-hop kernels run.
    Taken, they are given back when another allocation fails; the call that failed
    leaves the graph as it was, and the next one takes them again.  Buffers grow by half
    at least, which counts: a last batch that needs 1.27 times the lists held would fit
    half of 1.2 GB free, 1.5 times do not."""
    import torch
    hgt = gpu_lib
    st = W.temporal_stream("lists", 50, 1000, 9000, 3, 50.0, 4, 4, 100.0, 10**7, 800, W.SEED_BASE + 161)
    b = st.batches[2]
    st.batches[2] = W.Batch(b.del_handles, b.ins.rows(np.arange(8000)), b.ins_handles[:8000])
    p, q = (Pair(W.Stream("lists", st.n_vertices, st.initial, window=st.window), track=("temporal",)) for _ in range(2))
    args = [q.prepare(b, "lists")[0] for b in st.batches]

    def expanded(g, a):
        g.profile(True)
        g.apply_batch(*a)
        g.sync()
        return g.profile_read()["temporal"]["events"]

    monkeypatch.setenv("HGT_FREE_MEMORY", str(1500 << 20))
    assert expanded(q.g, args[0]) > 0
    monkeypatch.delenv("HGT_FREE_MEMORY")
    assert expanded(p.g, args[0]) == 0
    want = p.g.triad_counts("temporal")
    assert sum(want) > 0 and q.g.triad_counts("temporal") == want
    held = torch.cuda.mem_get_info()[0]
    monkeypatch.setenv("HGT_ALLOC_MAX", "4096")
    rc, _ = p.g.apply_batch(*args[1], raise_on_error=False)
    assert rc == hgt.ENOMEM
    assert torch.cuda.mem_get_info()[0] > held + (700 << 20)
    assert p.g.triad_counts("temporal") == want
    monkeypatch.delenv("HGT_ALLOC_MAX")
    assert expanded(p.g, args[1]) == 0
    q.g.apply_batch(*args[1])
    assert q.g.triad_counts("temporal") == p.g.triad_counts("temporal")
    monkeypatch.setenv("HGT_FREE_MEMORY", str(1200 << 20))
    assert expanded(p.g, args[2]) > 0
    monkeypatch.delenv("HGT_FREE_MEMORY")
    assert expanded(q.g, args[2]) == 0
    assert q.g.triad_counts("temporal") == p.g.triad_counts("temporal")
    p.close()
    q.close()


@pytest.mark.parametrize("limit_mb", [5, 33])
def test_fewer_arenas_where_memory_is_short(gpu_lib, monkeypatch, limit_mb):
    """Batches whose centres all reach the global stage, with room for one of its arenas (4 MB
    each, 512 at most) and for eight: fewer workgroups, the same counts."""
    monkeypatch.setenv("HGT_ALLOC_MAX", str(limit_mb << 20))
    monkeypatch.setenv("HGT_FORCE_STAGE", "2")
    monkeypatch.setenv("HGT_WAVE_SLOTS", "64")
    st = W.plain_stream("arenas", 90, 100, ("uniform", 1, 6), 0.0, 0.0, 2, 40, 50, W.SEED_BASE + 162)
    p = Pair(st, track=("hyperedge",), pool_words=1 << 16)
    compare_counts(p.g, p.o, p.track, "arenas build")
    for k, b in enumerate(st.batches):
        p.apply(b, f"arenas batch {k}")
        compare_store(p.g, p.o, f"arenas batch {k}")
        compare_counts(p.g, p.o, p.track, f"arenas batch {k}")
    p.close()
