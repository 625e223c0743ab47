"""GPU parity at the edges of the scan kernels' tiles (512 items; one item per thread up to 131 072 items, four beyond;
workgroups loop once a list has more tiles than a launch has workgroups: 512 of a list by itself, 256 of a stage or hop of a
batch, 128 of a member of a gang of four): de-duplication, cache lookup, count pass and the
compactions of a batch, element by element against the oracle (tolerance zero: indexing and byte copies)."""
import numpy as np
import pytest
import torch

from pathlib_helios import GpuCache, assert_same, gangs_in_flight, gpu_path, oracle_path, to_bytes

pytestmark = pytest.mark.gpu
ONE_ITEM_MAX = 131_072
EDGES = [1, 63, 65, 511, 512, 513, 1025, ONE_ITEM_MAX - 1, ONE_ITEM_MAX, ONE_ITEM_MAX + 1, 262_144, 262_145, 256 * 2048 + 3,
         512 * 2048 - 1, 512 * 2048, 512 * 2048 + 1, 1025 * 2048 + 3]


@pytest.fixture(scope="module")
def helios():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2310_00837_amd import helios as hl
    return hl


@pytest.fixture()
def h(helios):
    ctx = helios.Helios(0)
    yield ctx
    ctx.close()


def _graph(rng, n, max_deg):
    deg = rng.integers(0, max_deg + 1, n)
    off = np.zeros(n + 1, np.int64)
    off[1:] = np.cumsum(deg)
    idx = rng.integers(0, n, int(off[-1])).astype(np.int32)
    return off, idx


@pytest.mark.parametrize("n_ids", EDGES)
def test_dedup_and_lookup_at_tile_edges(h, oracle, n_ids):
    print("tile edge", n_ids, flush=True)
    rng = np.random.default_rng(n_ids)
    n = 50_000
    h.csr_load(torch.zeros(n + 1, dtype=torch.int64, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda"))
    ids = (n * rng.random(n_ids) ** 2).astype(np.int32)
    t = torch.from_numpy(ids).cuda()
    wu, wi = oracle.dedup(n, ids)
    for call in (h.dedup, h.dedup_noalloc) if n_ids <= 262_144 else (h.dedup,):
        uniq = torch.full((n_ids,), -9, dtype=torch.int32, device="cuda")
        inv, nu = torch.full_like(uniq, -9), torch.full((1,), -9, dtype=torch.int64).pin_memory()
        for _ in range(2):
            call(t, uniq, inv, nu)
            h.sync()
            assert int(nu[0]) == wu.size
            assert np.array_equal(uniq[:wu.size].cpu().numpy(), wu)
            assert np.array_equal(inv.cpu().numpy(), wi)
    feats = torch.from_numpy(rng.integers(0, 1 << 30, (n, 4)).astype(np.int32))
    order = torch.from_numpy(rng.permutation(n).astype(np.int32))
    n_hbm, n_host = 9_000, 21_000
    cache = GpuCache(h, feats, order, n_hbm, n_host)  # noqa: F841  (keeps the tables alive)
    out = torch.zeros((n_ids, 16), dtype=torch.uint8, device="cuda")
    miss = [torch.full((n_ids,), -9, dtype=torch.int32, device="cuda") for _ in range(3)]
    stats = torch.zeros(4, dtype=torch.int64).pin_memory()
    for _ in range(3):                                # (a ticket that is not put back to zero shows in the call after)
        h.gather(t, out, *miss, stats)
        h.sync()
    by_rank = to_bytes(feats)[order.numpy()]
    want = np.zeros((n_ids, 16), np.uint8)
    lists = oracle.gather(ids, oracle.rank_build(order.numpy()), n_hbm, n_host, np.ascontiguousarray(by_rank[:n_hbm]),
                          np.ascontiguousarray(by_rank[n_hbm:n_hbm + n_host]), want)
    assert np.array_equal(stats.numpy(), lists[3])
    assert np.array_equal(out.cpu().numpy(), want)
    for got, w in zip(miss, lists[:3]):
        assert np.array_equal(got[:w.size].cpu().numpy(), w)


@pytest.mark.parametrize("n_ids", [1_000, 300_001])
def test_dedup_reports_bad_ids_and_keeps_the_rest(h, helios, oracle, n_ids):
    """IDs outside [0, n) in a short and in a long list: reported, left out of unique, -1 in inverse."""
    rng = np.random.default_rng(n_ids)
    n = 5_000
    h.csr_load(torch.zeros(n + 1, dtype=torch.int64, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda"))
    ids = rng.integers(0, n, n_ids).astype(np.int32)
    bad = rng.choice(n_ids, 37, replace=False)
    ids[bad] = rng.choice([-1, -(1 << 31), n, (1 << 31) - 1], 37)
    uniq = torch.full((n_ids,), -9, dtype=torch.int32, device="cuda")
    inv, nu = torch.full_like(uniq, -9), torch.zeros(1, dtype=torch.int64).pin_memory()
    h.dedup(torch.from_numpy(ids).cuda(), uniq, inv, nu)
    with pytest.raises(helios.HeliosError) as e:
        h.sync()
    assert e.value.code == helios.EDATA
    good = np.ones(n_ids, bool)
    good[bad] = False
    wu, wi = oracle.dedup(n, ids[good])
    assert int(nu[0]) == wu.size and np.array_equal(uniq[:wu.size].cpu().numpy(), wu)
    got = inv.cpu().numpy()
    assert np.array_equal(got[good], wi) and (got[bad] == -1).all()


@pytest.mark.parametrize("n_seeds,fanouts", [(2_048, [4, 3]), (2_049, [4, 3]), (2_049, [25, 3]), (8_192, [33, 2]), (8_193, [33, 2]), (16_384, [32, 1]),
                                              (16_385, [32, 1]), (32_768, [9, 1]), (32_769, [9, 1]), (16_384, [8, 1]), (16_385, [8, 1]), (32_768, [8, 1]), (3_000, [0, 2]), (3_000, [5, 0]), (4_000, [64, 1]), (4_000, [65, 1]), (ONE_ITEM_MAX + 5, [1, 2]), (60_000, [4, 2]),
                                              (150_000, [4, 4]), (512 * 2048 + 1, [1, 1])])
def test_whole_path_with_long_lists(h, helios, oracle, n_seeds, fanouts):
    """Seed lists on both sides of the folded count pass and of the launch that counts and samples (512 tiles by lane group), stages and hops longer than one item per thread serves, and such
    that have more tiles than workgroups (the last two: stages of about 0.5 to 2 M items; 513 tiles in the last one's count pass)."""
    print("long lists", n_seeds, fanouts, flush=True)
    rng = np.random.default_rng(n_seeds)
    n = 200_000
    off, idx = _graph(rng, n, 9)
    seeds = rng.integers(0, n, n_seeds).astype(np.int32)
    h.csr_load(torch.from_numpy(off).cuda(), torch.from_numpy(idx).cuda())
    feats = torch.from_numpy(rng.integers(0, 1 << 30, (n, 4)).astype(np.int32))
    order = torch.from_numpy(rng.permutation(n).astype(np.int32))
    n_hbm, n_host = 50_000, 60_000
    cache = GpuCache(h, feats, order, n_hbm, n_host)  # noqa: F841
    by_rank = to_bytes(feats)[order.numpy()]
    tabs = [np.ascontiguousarray(x) for x in (by_rank[:n_hbm], by_rank[n_hbm:n_hbm + n_host], by_rank[n_hbm + n_host:])]
    want = oracle_path(oracle, off, idx, seeds, fanouts, 99, oracle.rank_build(order.numpy()), n_hbm, n_host, *tabs, 16)
    for _ in range(2):
        assert_same(gpu_path(h, helios, torch.from_numpy(seeds), fanouts, 99, fused=True), want)
    assert_same(gpu_path(h, helios, torch.from_numpy(seeds), fanouts, 99, fused=False), want)


@pytest.mark.parametrize("n_seeds,fan", [(2_049, 8), (9_000, 25), (3_000, 64), (3_000, 65)])
def test_long_seed_lists_cut_off_and_with_bad_seeds(h, helios, oracle, n_seeds, fan):
    """Samples that do not fit, and seeds that are no nodes: what there is room for is right, nothing is written behind it."""
    rng = np.random.default_rng(n_seeds + fan)
    n = 20_000
    off, idx = _graph(rng, n, 90)
    off, idx = np.concatenate([off, off[-1:]]), idx            # (node n has no neighbours)
    h.csr_load(torch.from_numpy(off).cuda(), torch.from_numpy(idx).cuda())
    seeds = rng.integers(0, n, n_seeds).astype(np.int32)
    bad = seeds.copy()
    at = [0, 700, n_seeds - 1]
    bad[at] = [-1, n + 1, -2**31]
    lone = seeds.copy()
    lone[at] = n
    for kind in ("short", "bad"):
        print("long seed lists", n_seeds, fan, kind, flush=True)
        frontier, indptr, flat = oracle.sample(off, idx, lone if kind == "bad" else seeds, [fan], 12)[0]
        cap = flat.size // 3 if kind == "short" else flat.size
        room = torch.full((flat.size + 4096,), -9, dtype=torch.int32, device="cuda")
        hops = [helios.HopBuffers(torch.empty(n_seeds, dtype=torch.int32, device="cuda"), torch.empty(n_seeds + 1, dtype=torch.int64, device="cuda"), room[:cap])]
        sizes = torch.zeros(2, dtype=torch.int64).pin_memory()
        given = bad if kind == "bad" else seeds
        t = torch.from_numpy(given).cuda()
        torch.cuda.synchronize()
        h.sample(t, [fan], 12, hops, sizes)
        with pytest.raises(helios.HeliosError) as e:
            h.sync()
        assert e.value.code == (helios.ECAPACITY if kind == "short" else helios.EDATA)
        assert sizes.tolist() == [n_seeds, flat.size]
        assert np.array_equal(hops[0].frontier.cpu().numpy(), given) and np.array_equal(hops[0].indptr.cpu().numpy(), indptr)
        assert np.array_equal(room[:cap].cpu().numpy(), flat[:cap]) and bool((room[cap:] == -9).all())


def test_gang_with_more_tiles_than_workgroups(helios, oracle):
    """A gang of four with hops and stages beyond 128 tiles of one item per thread, several batches one after the other."""
    rng = np.random.default_rng(77)
    n, b, fanouts, n_hbm, n_host = 100_000, 2_048, [35, 1], 40_000, 30_000
    off = np.arange(n + 1, dtype=np.int64) * 40
    idx = rng.integers(0, n, 40 * n).astype(np.int32)
    feats = torch.from_numpy(rng.integers(0, 1 << 30, (n, 4)).astype(np.int32))
    order = torch.from_numpy(rng.permutation(n).astype(np.int32))
    by_rank = to_bytes(feats)[order.numpy()]
    tabs = [np.ascontiguousarray(x) for x in (by_rank[:n_hbm], by_rank[n_hbm:n_hbm + n_host], by_rank[n_hbm + n_host:])]
    tabs_dev = (torch.from_numpy(tabs[0]).cuda(), torch.from_numpy(tabs[1]).pin_memory(), torch.from_numpy(tabs[2]).pin_memory())
    seeds = [rng.integers(0, n, b).astype(np.int32) for _ in range(12)]
    jobs = [(torch.from_numpy(s).cuda(), 50 + k) for k, s in enumerate(seeds)]
    torch.cuda.synchronize()
    got = gangs_in_flight(helios, torch.from_numpy(off).cuda(), torch.from_numpy(idx).cuda(), order.cuda(), n_hbm, n_host, 16, tabs_dev, b,
                          fanouts, jobs, members=4, n_gangs=1)
    rank = oracle.rank_build(order.numpy())
    for k, s in enumerate(seeds):
        assert got[k]["hops"][0][2].size > 128 * 512
        assert_same(got[k], oracle_path(oracle, off, idx, s, fanouts, 50 + k, rank, n_hbm, n_host, *tabs, 16))


@pytest.mark.parametrize("n_seeds", [1, 255, 256, 257, 1023, 1024, 1025, 2047])
def test_folded_count_pass_edges(h, helios, oracle, n_seeds):
    """Seed counts at the edges of the folded count pass (256, 1024, 2048 seeds), with fan-outs that fill a lane group exactly
    (no lane left for the seed itself) and that do not."""
    rng = np.random.default_rng(n_seeds)
    n = 20_000
    off, idx = _graph(rng, n, 80)
    seeds = rng.integers(0, n, n_seeds).astype(np.int32)
    h.csr_load(torch.from_numpy(off).cuda(), torch.from_numpy(idx).cuda())
    feats = torch.from_numpy(rng.integers(0, 1 << 30, (n, 4)).astype(np.int32))
    order = torch.from_numpy(rng.permutation(n).astype(np.int32))
    cache = GpuCache(h, feats, order, 8_000, 6_000)  # noqa: F841
    by_rank = to_bytes(feats)[order.numpy()]
    tabs = [np.ascontiguousarray(x) for x in (by_rank[:8_000], by_rank[8_000:14_000], by_rank[14_000:])]
    rank = oracle.rank_build(order.numpy())
    for fanouts in ([8, 3], [7, 8], [16, 2], [9, 16], [32, 2], [25, 10], [64, 2], [40, 1], [70, 2], [0, 3]):
        print("folded", n_seeds, fanouts, flush=True)
        want = oracle_path(oracle, off, idx, seeds, fanouts, 7, rank, 8_000, 6_000, *tabs, 16)
        assert_same(gpu_path(h, helios, torch.from_numpy(seeds), fanouts, 7, fused=True), want)


# steps of the copy beside the lookup (rows / (512 / lanes)) on both sides of every line of its rule, for rows of every copy
# shape, in lists of one item per thread and of four
@pytest.mark.parametrize("row_bytes,n,n_hbm,sizes", [
    (16, 600_000, 6_000, [1, 262_144, 262_145, 524_289]), (48, 300_000, 290_000, [131_073, 1_048_577]), (128, 300_000, 90_000, [262_144, 262_145]),
    (256, 200_000, 60_000, [131_072, 131_073]), (400, 200_000, 190_000, [131_072, 131_073]), (512, 200_000, 60_000, [65_536, 65_537]),
    (512, 140_000, 140_000, [262_144, 262_145]), (1024, 100_000, 30_000, [32_768, 32_769]), (1040, 60_000, 57_000, [65_536, 65_537, 131_100]),
    (2048, 60_000, 54_000, [131_080]),
    (2048, 60_000, 18_000, [65_536, 65_537]), (2064, 60_000, 60_000, [65_536, 131_100]), (4112, 30_000, 29_000, [8_193, 131_100])])
def test_gather_by_list_and_beside_the_lookup(h, helios, row_bytes, n, n_hbm, sizes):
    """helios_gather against torch indexing, exactly; the IDs include some that are no nodes."""
    gen = torch.Generator(device="cuda").manual_seed(row_bytes + n_hbm)
    h.csr_load(torch.zeros(n + 1, dtype=torch.int64, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda"))
    order = torch.randperm(n, device="cuda", generator=gen)
    rank = torch.empty_like(order)
    rank[order] = torch.arange(n, device="cuda")
    table = torch.randint(0, 256, (n_hbm, row_bytes), dtype=torch.uint8, device="cuda", generator=gen)
    order32 = order.int()
    h.cache_build(order32, n_hbm, 0, row_bytes, table, None, None)
    for n_ids in sizes:
        print("gather", row_bytes, n, n_hbm, n_ids, flush=True)
        ids = torch.randint(0, n, (n_ids,), device="cuda", generator=gen).int()
        bad = n_ids > 1000
        if bad:
            ids[n_ids // 3], ids[n_ids - 1] = -5, n
        node = (ids >= 0) & (ids < n)
        r = rank[ids.clamp(0, n - 1).long()]
        hit, miss = node & (r < n_hbm), node & (r >= n_hbm)
        out = torch.full((n_ids, row_bytes), 0xA5, dtype=torch.uint8, device="cuda")
        lists = [torch.full((n_ids,), -9, dtype=torch.int32, device="cuda") for _ in range(3)]
        stats = torch.zeros(4, dtype=torch.int64).pin_memory()
        torch.cuda.synchronize()
        h.gather(ids, out, *lists, stats)
        if bad:
            with pytest.raises(helios.HeliosError) as e:
                h.sync()
            assert e.value.code == helios.EDATA
        else:
            h.sync()
        n_miss = int(miss.sum())
        assert stats.tolist() == [n_ids, int(hit.sum()), 0, n_miss]
        assert torch.equal(out[hit], table[r[hit]]) and bool((out[~hit] == 0xA5).all())
        at = miss.nonzero()[:, 0]
        for got, want in zip(lists, (at, ids[at], r[at] - n_hbm)):
            assert torch.equal(got[:n_miss].long(), want.long()) and bool((got[n_miss:] == -9).all())


def _hash(x):
    h = x.astype(np.uint32) * np.uint32(0x9E3779B1)
    h ^= h >> np.uint32(15)
    h *= np.uint32(0x85EBCA77)
    return h ^ (h >> np.uint32(13))


@pytest.mark.parametrize("kind", ["one", "distinct", "one bucket", "one bucket and class", "bad", "few repeats far apart"])
@pytest.mark.parametrize("n_ids", [19_999, 20_000, 32_767, 32_768, 98_303, 98_304, 98_305, 262_145, 524_289, 1_000_003, 1_048_577, 1_572_864, 1_572_865, 2_097_152, 2_097_153])
def test_dedup_of_long_lists_by_parts(h, helios, kind, n_ids):
    """Long lists (32 768 to 2 097 152 IDs are taken apart by hash, from 20 000 on if the table is small) whose parts are as uneven as can be, against numpy."""
    print("by parts", kind, n_ids, flush=True)
    rng = np.random.default_rng(n_ids)
    n = 100_000_000
    if kind == "one":
        ids = np.full(n_ids, 77_777)
    elif kind in ("distinct", "bad"):
        ids = rng.permutation(n_ids) * 7
    elif kind == "few repeats far apart":
        ids = np.concatenate([np.arange(n_ids - n_ids // 9), np.arange(n_ids // 9)[::-1]])
    else:
        pool = np.arange(40_000_000)                      # about 78 k of them in a bucket (the hash's highest 9 bits)
        in_bucket = _hash(pool) >> np.uint32(23) == 5
        if kind == "one bucket and class":                # (its lowest bits)
            in_bucket &= _hash(pool) % np.uint32(8) == 3
        ids = rng.choice(pool[in_bucket], min(n_ids, 1_000_003))
        ids = np.concatenate([ids, rng.integers(0, n, n_ids - ids.size)])
    ids = ids.astype(np.int32)
    if kind == "bad":
        ids[[0, 5000, n_ids - 1]] = [-1, n, -2**31]
    h.csr_load(torch.zeros(n + 1, dtype=torch.int64, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda"))
    node = (ids >= 0) & (ids < n)
    values, first, back = np.unique(ids[node], return_index=True, return_inverse=True)
    order = np.argsort(first)
    place = np.empty_like(order)
    place[order] = np.arange(order.size)
    want = np.full(n_ids, -1, np.int64)
    want[node] = place[back]
    t = torch.from_numpy(ids).cuda()
    uniq = torch.full((n_ids,), -9, dtype=torch.int32, device="cuda")
    inv, nu = torch.full_like(uniq, -9), torch.full((1,), -9, dtype=torch.int64).pin_memory()
    for _ in range(2):
        h.dedup(t, uniq, inv, nu)
        if kind == "bad":
            with pytest.raises(helios.HeliosError) as e:
                h.sync()
            assert e.value.code == helios.EDATA
        else:
            h.sync()
        assert int(nu[0]) == values.size
        assert np.array_equal(uniq[:values.size].cpu().numpy(), values[order])
        assert np.array_equal(inv.cpu().numpy(), want)


@pytest.mark.parametrize("n_ids", [1, 512, 513, 64 * 512 + 1, 5 * 64 * 512 + 77])
@pytest.mark.parametrize("whole", [True, False])
def test_gather_counts_with_all_nodes_in_hbm(h, helios, n_ids, whole):
    """Stats and rows where the lookup only counts, at the edges of its steps (64 workgroups of 512, four steps read ahead); with
    an order that leaves nodes out, which are then in no class."""
    gen = torch.Generator(device="cuda").manual_seed(n_ids)
    n = 30_000
    h.csr_load(torch.zeros(n + 1, dtype=torch.int64, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda"))
    order = torch.randperm(n, device="cuda", generator=gen)
    if not whole:
        order[7::1000] = order[6]
    table = torch.randint(0, 256, (n, 64), dtype=torch.uint8, device="cuda", generator=gen)
    order32 = order.int()
    h.cache_build(order32, n, 0, 64, table, None, None)
    if not whole:
        with pytest.raises(helios.HeliosError):
            h.sync()
    known = torch.zeros(n, dtype=torch.bool, device="cuda")
    known[order] = True
    ids = torch.randint(0, n, (n_ids,), device="cuda", generator=gen).int()
    lists = [torch.full((n_ids,), -9, dtype=torch.int32, device="cuda") for _ in range(3)]
    once = torch.ones(n, dtype=torch.bool, device="cuda")
    once[order[6]] = whole                                    # (which of its ranks a repeated node has is open)
    rank = torch.empty(n, dtype=torch.int64, device="cuda")
    rank[order] = torch.arange(n, device="cuda")
    for _ in range(3):
        out = torch.full((n_ids, 64), 0xA5, dtype=torch.uint8, device="cuda")
        stats = torch.zeros(4, dtype=torch.int64).pin_memory()
        torch.cuda.synchronize()
        h.gather(ids, out, *lists, stats)
        h.sync()
        there = known[ids.long()]
        assert stats.tolist() == [n_ids, int(there.sum()), 0, 0]
        look = there & once[ids.long()]
        assert torch.equal(out[look], table[rank[ids.long()[look]]]) and bool((out[~there] == 0xA5).all())
        assert all(bool((x == -9).all()) for x in lists)


@pytest.mark.parametrize("which", [0, 1, 2])
@pytest.mark.parametrize("n_ids", [3_000, 130_000])
def test_gather_with_its_miss_list_in_the_memory_of_the_ids(h, which, n_ids):
    rng = np.random.default_rng(n_ids + which)
    n, n_hbm = 40_000, 20_000
    h.csr_load(torch.zeros(n + 1, dtype=torch.int64, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda"))
    order = torch.from_numpy(rng.permutation(n).astype(np.int32)).cuda()
    rank = torch.empty(n, dtype=torch.int64, device="cuda")
    rank[order.long()] = torch.arange(n, device="cuda")
    table = torch.from_numpy(rng.integers(0, 256, (n_hbm, 512)).astype(np.uint8)).cuda()
    h.cache_build(order, n_hbm, 0, 512, table, None, None)
    for _ in range(5):
        ids = torch.from_numpy(rng.integers(0, n, n_ids).astype(np.int32)).cuda()
        r = rank[ids.long()]
        at = (r >= n_hbm).nonzero()[:, 0]
        want = (at, ids[at].long(), r[at] - n_hbm)
        lists = [torch.empty(n_ids, dtype=torch.int32, device="cuda") for _ in range(3)]
        lists[which] = ids
        out, stats = torch.full((n_ids, 512), 0xA5, dtype=torch.uint8, device="cuda"), torch.zeros(4, dtype=torch.int64).pin_memory()
        torch.cuda.synchronize()
        h.gather(ids, out, *lists, stats)
        h.sync()
        assert stats.tolist() == [n_ids, n_ids - at.numel(), 0, at.numel()]
        assert torch.equal(out[r < n_hbm], table[r[r < n_hbm]]) and bool((out[at] == 0xA5).all())
        for got, w in zip(lists, want):
            assert torch.equal(got[:at.numel()].long(), w)


@pytest.mark.parametrize("noalloc", [False, True])
def test_dedup_of_uneven_lists_leaves_the_table_empty(h, helios, noalloc):
    """A list by parts whose buckets do not fit LDS goes by the call's table in memory; lists that go by the table altogether follow."""
    rng = np.random.default_rng(int(noalloc))
    n = 100_000_000
    pool = np.arange(40_000_000)
    many, some = pool[_hash(pool) >> np.uint32(23) == 5], pool[_hash(pool) >> np.uint32(23) == 300][:9_000]
    uneven = np.concatenate([many, some, rng.choice(some, 20_000), rng.integers(0, n, 60_000)])
    rng.shuffle(uneven)
    h.csr_load(torch.zeros(n + 1, dtype=torch.int64, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda"))
    call = h.dedup_noalloc if noalloc else h.dedup
    for ids in (uneven, uneven[:98_303], uneven, rng.integers(0, n, 90_000), uneven[5:300]):
        print("uneven", noalloc, ids.size, flush=True)
        values, first, back = np.unique(ids, return_index=True, return_inverse=True)
        order = np.argsort(first)
        place = np.empty_like(order)
        place[order] = np.arange(order.size)
        t = torch.from_numpy(ids.astype(np.int32)).cuda()
        uniq, inv, nu = torch.empty_like(t), torch.empty_like(t), torch.zeros(1, dtype=torch.int64).pin_memory()
        torch.cuda.synchronize()
        call(t, uniq, inv, nu)
        h.sync()
        assert int(nu[0]) == values.size
        assert np.array_equal(uniq[:values.size].cpu().numpy(), values[order])
        assert np.array_equal(inv.cpu().numpy(), place[back])


@pytest.mark.parametrize("share", [1.0, 0.9])
@pytest.mark.parametrize("n_ids", [3_000, 600_000, 2_200_000])
def test_gather_with_its_rows_in_the_memory_of_the_ids(h, share, n_ids):
    """The IDs lie in the first rows of `out`, or under the stats (all nodes in HBM, and not all)."""
    gen = torch.Generator(device="cuda").manual_seed(n_ids)
    n, row = 40_000, 64
    n_hbm = int(share * n)
    h.csr_load(torch.zeros(n + 1, dtype=torch.int64, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda"))
    order = torch.randperm(n, device="cuda", generator=gen).int()
    rank = torch.empty(n, dtype=torch.int64, device="cuda")
    rank[order.long()] = torch.arange(n, device="cuda")
    table = torch.randint(0, 256, (n_hbm, row), dtype=torch.uint8, device="cuda", generator=gen)
    h.cache_build(order, n_hbm, 0, row, table, None, None)
    for stats_too in (False, True):
        room = torch.empty(n_ids * row + 64, dtype=torch.uint8, device="cuda")
        want = torch.randint(0, n, (n_ids,), dtype=torch.int32, device="cuda", generator=gen)
        ids = room[:4 * n_ids].view(torch.int32)
        ids.copy_(want)
        if stats_too:                                         # rows of their own, the stats over the first IDs
            out, stats = torch.zeros((n_ids, row), dtype=torch.uint8, device="cuda"), room[:32].view(torch.int64)
        else:
            out, stats = room[:n_ids * row].view(n_ids, row), torch.zeros(4, dtype=torch.int64).pin_memory()
        lists = [torch.empty(n_ids, dtype=torch.int32, device="cuda") for _ in range(3)]
        torch.cuda.synchronize()
        h.gather(ids, out, *lists, stats)
        h.sync()
        r = rank[want.long()]
        hit = r < n_hbm
        assert torch.equal(out[hit], table[r[hit]])
        assert stats.tolist() == [n_ids, int(hit.sum()), 0, int((~hit).sum())]


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("n_ids", [32_768, 98_304, 100_003, 262_144])
def test_dedup_by_parts_in_place_cut_off_and_with_bad_ids(h, helios, n_ids, noalloc):
    """Lists by parts through both calls: `unique` in the memory of the IDs, the inverse there, no inverse, a `unique` that is too
    short, and IDs that are no nodes."""
    rng = np.random.default_rng(n_ids)
    n = 1_000_000
    h.csr_load(torch.zeros(n + 1, dtype=torch.int64, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda"))
    call = h.dedup_noalloc if noalloc else h.dedup
    good = (n * rng.random(n_ids) ** 3).astype(np.int32)
    bad = good.copy()
    bad[[0, n_ids // 2, n_ids - 1]] = [-1, n, -2**31]
    for kind in ("unique over ids", "inverse over ids", "no inverse", "short", "bad"):
        print("in place", n_ids, noalloc, kind, flush=True)
        ids = bad if kind == "bad" else good
        node = (ids >= 0) & (ids < n)
        values, first, back = np.unique(ids[node], return_index=True, return_inverse=True)
        order = np.argsort(first)
        place = np.empty_like(order)
        place[order] = np.arange(order.size)
        want = np.full(n_ids, -1, np.int64)
        want[node] = place[back]
        for _ in range(2):
            t = torch.from_numpy(ids).cuda()
            cap = values.size // 3 if kind == "short" else n_ids
            uniq = t if kind == "unique over ids" else torch.full((cap,), -9, dtype=torch.int32, device="cuda")
            inv = None if kind == "no inverse" else t if kind == "inverse over ids" else torch.full((n_ids,), -9, dtype=torch.int32, device="cuda")
            nu = torch.full((1,), -9, dtype=torch.int64).pin_memory()
            torch.cuda.synchronize()
            call(t, uniq, inv, nu)
            if kind in ("short", "bad"):
                with pytest.raises(helios.HeliosError) as e:
                    h.sync()
                assert e.value.code == (helios.ECAPACITY if kind == "short" else helios.EDATA)
            else:
                h.sync()
            assert int(nu[0]) == values.size
            fits = min(cap, values.size)
            assert np.array_equal(uniq[:fits].cpu().numpy(), values[order][:fits])
            assert inv is None or np.array_equal(inv.cpu().numpy(), want)


@pytest.mark.parametrize("n_ids", [263_000, 1_100_001, 1_600_001])
def test_dedup_by_parts_with_repeats_at_the_ends_of_tiles(h, n_ids):
    """Tiles whose flags fill no whole number of lines: repeats of first occurrences at the end of the same tile, and of some at the
    beginnings of all tiles before, in another list each time (what a call leaves in the scratch is wrong for the next)."""
    rng = np.random.default_rng(n_ids)
    most = 256 if n_ids <= 256 * 6144 else 512
    tile = -(-n_ids // (most * 64)) * 64
    assert tile > 1024 and tile % 512 != 0
    h.csr_load(torch.zeros(4 * n_ids + 1, dtype=torch.int64, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda"))
    at = np.arange(n_ids)
    inside, begin = at % tile, at - at % tile
    near = np.nonzero(inside >= tile - 8)[0]
    far = np.nonzero((inside >= tile // 2) & (inside < tile // 2 + 400) & (begin > 0))[0]
    for k in range(6):
        ids = rng.permutation(4 * n_ids)[:n_ids]
        ids[near] = ids[near - rng.integers(8, 300, near.size)]
        ids[far] = ids[rng.integers(0, begin[far] // tile) * tile + rng.integers(0, 400, far.size)]
        print("ends of tiles", n_ids, k, flush=True)
        values, first, back = np.unique(ids, return_index=True, return_inverse=True)
        order = np.argsort(first)
        place = np.empty_like(order)
        place[order] = np.arange(order.size)
        t = torch.from_numpy(ids.astype(np.int32)).cuda()
        uniq, inv, nu = torch.empty_like(t), torch.empty_like(t), torch.zeros(1, dtype=torch.int64).pin_memory()
        torch.cuda.synchronize()
        h.dedup(t, uniq, inv, nu)
        h.sync()
        assert int(nu[0]) == values.size
        assert np.array_equal(uniq[:values.size].cpu().numpy(), values[order])
        assert np.array_equal(inv.cpu().numpy(), place[back])


def test_launches_that_wait_on_several_streams(helios, oracle):
    """Hotness orders of all passes, lists by parts and long seed lists of four contexts in flight on four streams: launches whose
    workgroups wait for others of theirs, side by side.  Every call has inputs of its own: what an earlier one has left in the context's
    scratch is wrong for it."""
    rng = np.random.default_rng(31)
    n, m, n_seeds, fan = 1_200_000, 700_001, 9_001, [25]
    off, idx = _graph(rng, n, 5)
    off_d, idx_d = torch.from_numpy(off).cuda(), torch.from_numpy(idx).cuda()
    contexts, calls = [], []
    for _ in range(4):
        h = helios.Helios(0, stream=torch.cuda.Stream())
        h.csr_load(off_d, idx_d)
        h.reserve(m)
        contexts.append(h)
    for k in range(12):
        counts = rng.integers(0, 1 << 31, n).astype(np.int32)
        ids = rng.integers(0, n, m).astype(np.int32)
        near = rng.integers(300, m, m // 4)
        ids[near] = ids[near - rng.integers(1, 300, near.size)]           # (repeats within a tile, too)
        seeds = rng.integers(0, n, n_seeds).astype(np.int32)
        calls.append(dict(h=contexts[k % 4], counts=counts, ids=ids, seeds=seeds, counts_d=torch.from_numpy(counts).cuda(), ids_d=torch.from_numpy(ids).cuda(),
                          seeds_d=torch.from_numpy(seeds).cuda(), order=torch.empty(n, dtype=torch.int32, device="cuda"),
                          uniq=torch.empty(m, dtype=torch.int32, device="cuda"), inv=torch.empty(m, dtype=torch.int32, device="cuda"),
                          nu=torch.zeros(1, dtype=torch.int64).pin_memory(), hops=helios.alloc_hops(n_seeds, fan, "cuda"),
                          sizes=torch.zeros(2, dtype=torch.int64).pin_memory()))
    torch.cuda.synchronize()
    for k, u in enumerate(calls):
        u["h"].hotness_order(u["counts_d"], u["order"])
        u["h"].dedup(u["ids_d"], u["uniq"], u["inv"], u["nu"])
        u["h"].sample(u["seeds_d"], fan, 5 + k, u["hops"], u["sizes"])
    for h in contexts:
        h.sync()
    for k, u in enumerate(calls):
        assert np.array_equal(u["order"].cpu().numpy(), oracle.hotness_order(u["counts"]))
        wu, wi = oracle.dedup(n, u["ids"])
        assert int(u["nu"][0]) == wu.size and np.array_equal(u["uniq"][:wu.size].cpu().numpy(), wu)
        assert np.array_equal(u["inv"].cpu().numpy(), wi)
        frontier, indptr, flat = oracle.sample(off, idx, u["seeds"], fan, 5 + k)[0]
        assert u["sizes"].tolist() == [frontier.size, flat.size]
        for got, want in ((u["hops"][0].frontier, frontier), (u["hops"][0].indptr, indptr), (u["hops"][0].flat, flat)):
            assert np.array_equal(got[:want.size].cpu().numpy(), want)
    for h in contexts:
        h.close()
