"""GPU parity of the hotness order's radix sort at the edges of its tiles (8192 nodes) and for every set of digits (11 bits) that
can vary: a pass whose digit is the same in all counts is left out.  Against the oracle, exactly."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
SIZES = [1, 2, 65, 8191, 8192, 8193, 70_001]
KINDS = {"zero": lambda r, n: np.zeros(n), "equal": lambda r, n: np.full(n, 123_456_789), "low": lambda r, n: r.integers(0, 2048, n),
         "few": lambda r, n: r.poisson(0.7, n), "middle": lambda r, n: r.integers(0, 2048, n) << 11,
         "high": lambda r, n: r.integers(0, 512, n) << 22, "low and high": lambda r, n: (r.integers(0, 3, n) << 29) | r.integers(0, 9, n),
         "all": lambda r, n: r.integers(0, 1 << 31, n), "low and middle": lambda r, n: r.integers(0, 1 << 14, n),
         "few and hubs": lambda r, n: np.where(r.random(n) < 0.01, r.integers(0, 5000, n), r.poisson(0.7, n))}      # waves with and without high bits


@pytest.mark.parametrize("kind", KINDS)
def test_hotness_order_at_tile_edges(oracle, kind):
    from paper_2310_00837_amd import helios
    h = helios.Helios(0)
    for n in SIZES + ([8192 * 512 + 77] if kind in ("few", "all", "few and hubs") else []):        # the last: more tiles than workgroups
        print("hotness order", kind, n, flush=True)
        counts = KINDS[kind](np.random.default_rng(n), n).astype(np.int32)
        h.csr_load(torch.zeros(n + 1, dtype=torch.int64, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda"))
        t, order = torch.from_numpy(counts).cuda(), torch.full((n,), -9, dtype=torch.int32, device="cuda")
        for _ in range(2):
            h.hotness_order(t, order)
            h.sync()
            assert np.array_equal(order.cpu().numpy(), oracle.hotness_order(counts))
            assert np.array_equal(t.cpu().numpy(), counts)
    h.close()


@pytest.mark.parametrize("kind", ["zero", "low", "low and middle", "high", "all"])          # one pass, two, three
@pytest.mark.parametrize("n", [8193, 8192 * 600 + 5])               # the second: more tiles than workgroups
def test_hotness_order_in_the_memory_of_the_counts(oracle, kind, n):
    from paper_2310_00837_amd import helios
    h = helios.Helios(0)
    counts = KINDS[kind](np.random.default_rng(n), n).astype(np.int32)
    h.csr_load(torch.zeros(n + 1, dtype=torch.int64, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda"))
    want = oracle.hotness_order(counts)
    for shift in (0, 1000, -1000):                                 # order = counts, behind it, before it
        t = torch.zeros(n + 2000, dtype=torch.int32, device="cuda")
        t[1000:1000 + n] = torch.from_numpy(counts)
        order = t[1000 + shift:1000 + shift + n]
        h.hotness_order(t[1000:1000 + n], order)
        h.sync()
        assert np.array_equal(order.cpu().numpy(), want)
    h.close()


@pytest.mark.parametrize("kind", ["random", "ascending", "descending", "hot", "repeats", "a bucket too full"])
@pytest.mark.parametrize("n", [1_999_999, 2_000_000, 2_097_153, 8_388_607, 8_388_609, 16_777_216, 16_777_217])
# (scattered stores; buckets of 4096, 8192, 16384 and 32768 nodes, all 512 buckets of 32768; scattered stores again)
def test_cache_map_by_buckets(kind, n):
    """The map that helios_cache_build makes of an order, read back by a gather whose rows are the ranks: by scattered stores below
    2 M nodes and by buckets from there on, which use the scratch of a hotness order; and orders that are no permutation."""
    from paper_2310_00837_amd import helios
    print("cache map", kind, n, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(n)
    h = helios.Helios(0)
    h.csr_load(torch.zeros(n + 1, dtype=torch.int64, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda"))
    counts = torch.randint(0, 9, (n,), device="cuda", generator=gen).int()
    order = torch.empty(n, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    h.hotness_order(counts, order)
    h.sync()
    if kind in ("random", "repeats", "a bucket too full"):
        order = torch.randperm(n, device="cuda", generator=gen).int()
    elif kind != "hot":
        order = torch.arange(n, device="cuda").int()
        if kind == "descending":
            order = order.flip(0).contiguous()
    bad = kind in ("repeats", "a bucket too full")
    if kind == "repeats":
        order[5::1000] = order[4::1000][:order[5::1000].numel()]
        order[77] = -3
    if kind == "a bucket too full":
        order[1000:30_000] = 4099
    at = torch.arange(n, device="cuda")
    node = (order >= 0) & (order < n)
    times = torch.zeros(n, dtype=torch.int64, device="cuda").index_add_(0, order[node].long(), torch.ones_like(at[node]))
    table = torch.zeros((n, 2), dtype=torch.int64, device="cuda")
    table[:, 0] = at
    out = torch.empty((n, 2), dtype=torch.int64, device="cuda")
    lists, stats = [torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(3)], torch.zeros(4, dtype=torch.int64).pin_memory()
    ids = at.int()
    for _ in range(2):
        out.fill_(-9)
        torch.cuda.synchronize()
        h.cache_build(order, n, 0, 16, table, None, None)
        h.gather(ids, out, *lists, stats)
        if bad:
            with pytest.raises(helios.HeliosError) as e:
                h.sync()
            assert e.value.code == helios.EDATA
        else:
            h.sync()
        known = times > 0
        assert stats.tolist() == [n, int(known.sum()), 0, 0]
        got = out[:, 0]
        assert torch.equal(order[got[known]].long(), at[known])          # (any of its ranks for a node that is there twice)
        assert bool((got[~known] == -9).all())
    h.close()


def test_captured_cache_build_outlives_the_scratch_of_a_hotness_order():
    """A cache map captured after a hotness order and replayed after a larger one, which frees the scratch of the first."""
    from paper_2310_00837_amd import helios
    n, larger = 2_100_000, 3_000_000
    gen = torch.Generator(device="cuda").manual_seed(3)
    stream = torch.cuda.Stream()
    h = helios.Helios(0, stream=stream)
    off, idx = torch.zeros(larger + 1, dtype=torch.int64, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    counts, order = torch.zeros(larger, dtype=torch.int32, device="cuda"), torch.empty(larger, dtype=torch.int32, device="cuda")
    at = torch.arange(n, device="cuda")
    table = torch.zeros((n, 2), dtype=torch.int64, device="cuda")
    table[:, 0] = at
    given = torch.arange(n, device="cuda").int()
    torch.cuda.synchronize()
    h.csr_load(off[:n + 1], idx)
    h.hotness_order(counts[:n], order[:n])
    h.cache_build(given, n, 0, 16, table, None, None)              # (the map's own memory is there before the capture)
    h.sync()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        h.cache_build(given, n, 0, 16, table, None, None)
    h.csr_load(off, idx)
    h.hotness_order(counts, order)
    h.csr_load(off[:n + 1], idx)
    h.cache_build(given, n, 0, 16, table, None, None)
    h.sync()
    ids, out = at.int(), torch.empty((n, 2), dtype=torch.int64, device="cuda")
    lists, stats = [torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(3)], torch.zeros(4, dtype=torch.int64).pin_memory()
    for _ in range(3):
        given.copy_(torch.randperm(n, device="cuda", generator=gen))
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            graph.replay()
        h.gather(ids, out, *lists, stats)
        h.sync()
        assert stats.tolist() == [n, n, 0, 0] and torch.equal(given[out[:, 0]].long(), at)
    h.close()


@pytest.mark.parametrize("kind", ["sparse counts", "blocks", "blocks with repeats", "ascending with repeats", "descending with a gap"])
@pytest.mark.parametrize("n", [2_000_003, 8_388_609])
def test_cache_map_of_neighbouring_nodes(kind, n):
    """Orders in which neighbouring nodes follow each other, whose ranks are stored without the buckets: every node's rank is one at
    which the order has it, also where the map held that of another order before; a node that no rank points to has none."""
    from paper_2310_00837_amd import helios
    print("neighbouring nodes", kind, n, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(n)
    h = helios.Helios(0)
    h.csr_load(torch.zeros(n + 1, dtype=torch.int64, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda"))
    at = torch.arange(n, device="cuda")
    counts = torch.where(torch.rand(n, device="cuda", generator=gen) < 0.03, torch.randint(1, 50, (n,), device="cuda", generator=gen), 0).int()
    order = torch.empty(n, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    h.hotness_order(counts, order)
    h.sync()
    orders = [torch.randperm(n, device="cuda", generator=gen).int(), order]
    if kind.startswith("blocks"):
        size = 64
        blocks = torch.randperm(n // size, device="cuda", generator=gen)[:, None] * size + torch.arange(size, device="cuda")
        order = torch.cat([blocks.flatten(), at[n // size * size:]]).int()
    elif kind.startswith("ascending"):
        order = at.int()
    elif kind.startswith("descending"):
        order = at.flip(0).int()
    if kind.endswith("repeats"):
        order[5::1000] = order[4::1000][:order[5::1000].numel()]
        order[100_000:100_064] = order[300_000:300_064]
    if kind.endswith("gap"):
        order[n // 2] = -7
    orders += [order, order]
    table = torch.zeros((n, 2), dtype=torch.int64, device="cuda")
    table[:, 0] = at
    ids, out = at.int(), torch.empty((n, 2), dtype=torch.int64, device="cuda")
    lists, stats = [torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(3)], torch.zeros(4, dtype=torch.int64).pin_memory()
    for order in orders:
        known = torch.zeros(n, dtype=torch.bool, device="cuda")
        known[order[(order >= 0) & (order < n)].long()] = True
        whole = bool(known.all())
        out.fill_(-9)
        torch.cuda.synchronize()
        h.cache_build(order, n, 0, 16, table, None, None)
        h.gather(ids, out, *lists, stats)
        if whole:
            h.sync()
        else:
            with pytest.raises(helios.HeliosError) as e:
                h.sync()
            assert e.value.code == helios.EDATA
        assert stats.tolist() == [n, int(known.sum()), 0, 0]
        got = out[:, 0]
        assert torch.equal(order[got[known]].long(), at[known]) and bool((got[~known] == -9).all())
    h.close()
