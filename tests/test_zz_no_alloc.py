"""helios_dedup_noalloc (the entry point that allocates nothing: its scratch is a fixed array in the
library's device image) gives exactly what helios_dedup gives, call after call on the same array."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def helios():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2310_00837_amd import helios as hl
    return hl


def _both(h, ids_np, unique_cap=None):
    """(unique, inverse, n_unique) from helios_dedup and from helios_dedup_noalloc on the same input."""
    n = ids_np.size
    ids = torch.from_numpy(ids_np).cuda()
    cap = max(n, 1) if unique_cap is None else unique_cap
    res = []
    for call in (h.dedup, h.dedup_noalloc):
        uq = torch.full((max(cap, 1),), -3, dtype=torch.int32, device="cuda")
        inv = torch.full((max(n, 1),), -3, dtype=torch.int32, device="cuda")
        nu = torch.full((1,), -3, dtype=torch.int64).pin_memory()
        call(ids, uq, inv, nu, n_ids=n)
        h.sync()
        res.append((uq.cpu().numpy(), inv.cpu().numpy(), int(nu[0])))
    return res


def test_noalloc_dedup_equals_dedup_on_consecutive_calls(helios, oracle):
    n_nodes = 50_000
    h = helios.Helios(0)
    try:
        h.csr_load(torch.zeros(n_nodes + 1, dtype=torch.int64, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda"))
        rng = np.random.default_rng(7)
        # the second call is smaller than the first (it meets the first call's leftovers in the shared
        # array), then a larger one again, a single-tile one, the tile edges, an empty one and the maximum
        sizes = [70_001, 4_097, 130_000, 300, 1024, 1025, 0, helios.DEDUP_NOALLOC_MAX_IDS]
        for k, n in enumerate(sizes):
            print("noalloc dedup", k, n, flush=True)
            span = 3 if k == 3 else max(1, min(n_nodes, n // 2 + 1))     # many repeats / few repeats
            ids = rng.integers(0, span, n).astype(np.int32)
            (uq_a, inv_a, nu_a), (uq_b, inv_b, nu_b) = _both(h, ids)
            assert nu_a == nu_b
            assert np.array_equal(uq_a, uq_b), "unique differs (sentinels past n_unique included)"
            assert np.array_equal(inv_a, inv_b), "inverse differs"
            want_u, want_inv = oracle.dedup(n_nodes, ids)
            assert nu_b == want_u.size
            assert np.array_equal(uq_b[:nu_b], want_u) and np.array_equal(inv_b[:n], want_inv)
    finally:
        h.close()


def test_noalloc_dedup_on_two_contexts_and_errors(helios):
    n_nodes = 1000
    a, b = helios.Helios(0), helios.Helios(0)
    try:
        for ctx in (a, b):
            ctx.csr_load(torch.zeros(n_nodes + 1, dtype=torch.int64, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda"))
        rng = np.random.default_rng(11)
        for ctx, n in ((a, 5000), (b, 777), (a, 64)):                 # one after the other: the contexts share the array
            ids = rng.integers(0, n_nodes, n).astype(np.int32)
            (uq_a, inv_a, nu_a), (uq_b, inv_b, nu_b) = _both(ctx, ids)
            assert nu_a == nu_b and np.array_equal(uq_a, uq_b) and np.array_equal(inv_a, inv_b)
        # capacity and data errors are reported as by helios_dedup
        ids = torch.arange(100, dtype=torch.int32, device="cuda")
        uq = torch.full((40,), -3, dtype=torch.int32, device="cuda")
        nu = torch.zeros(1, dtype=torch.int64).pin_memory()
        a.dedup_noalloc(ids, uq, None, nu)
        with pytest.raises(helios.HeliosError) as e:
            a.sync()
        assert e.value.code == helios.ECAPACITY and int(nu[0]) == 100
        assert np.array_equal(uq.cpu().numpy(), np.arange(40, dtype=np.int32))
        bad = torch.tensor([1, 2, n_nodes, 3, -1], dtype=torch.int32, device="cuda")
        uq5 = torch.full((5,), -3, dtype=torch.int32, device="cuda")
        a.dedup_noalloc(bad, uq5, None, nu)
        with pytest.raises(helios.HeliosError) as e:
            a.sync()
        assert e.value.code == helios.EDATA
        # more IDs than the fixed array has room for: refused on the host, nothing launched
        too_many = torch.zeros(helios.DEDUP_NOALLOC_MAX_IDS + 1, dtype=torch.int32, device="cuda")
        uqm = torch.empty(8, dtype=torch.int32, device="cuda")
        with pytest.raises(helios.HeliosError) as e:
            a.dedup_noalloc(too_many, uqm, None, nu)
        assert e.value.code == helios.EINVAL and "at most" in str(e.value)
        a.sync()
    finally:
        a.close()
        b.close()


@pytest.mark.parametrize("n", [300, 1_025, 41_237, 262_144])
def test_captured_noalloc_dedup_replayed_between_direct_calls(helios, oracle, n):
    """The call in a HIP graph, replayed with new IDs, with direct calls of other lengths (one tile, several, the longest) on the
    shared array in between: every result is the oracle's."""
    n_nodes = 50_000
    rng = np.random.default_rng(n)
    stream = torch.cuda.Stream()
    h = helios.Helios(0, stream=stream)
    try:
        off, idx = torch.zeros(n_nodes + 1, dtype=torch.int64, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
        torch.cuda.synchronize()
        h.csr_load(off, idx)

        def buffers(m):
            return (torch.zeros(m, dtype=torch.int32, device="cuda"), torch.full((m,), -3, dtype=torch.int32, device="cuda"),
                    torch.full((m,), -3, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int64).pin_memory())

        def fill(t):
            ids = (n_nodes * rng.random(t.numel()) ** 2).astype(np.int32)
            t.copy_(torch.from_numpy(ids))
            torch.cuda.synchronize()
            return ids

        def check(ids, bufs):
            want_u, want_inv = oracle.dedup(n_nodes, ids)
            u = int(bufs[3][0])
            assert u == want_u.size and np.array_equal(bufs[1][:u].cpu().numpy(), want_u) and np.array_equal(bufs[2].cpu().numpy(), want_inv)

        captured, graph = buffers(n), torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=stream):
            h.dedup_noalloc(*captured)
        for k, m in enumerate([700, 5_000, 262_144, 1, 70_001]):
            print("captured noalloc dedup", n, k, m, flush=True)
            ids = fill(captured[0])
            with torch.cuda.stream(stream):
                graph.replay()
            h.sync()
            check(ids, captured)
            direct = buffers(m)
            ids = fill(direct[0])
            h.dedup_noalloc(*direct)
            h.sync()
            check(ids, direct)
            if k == 2:                                             # twice in a row without a wait
                ids = fill(captured[0])
                with torch.cuda.stream(stream):
                    graph.replay()
                    graph.replay()
                h.sync()
                check(ids, captured)
    finally:
        h.close()
