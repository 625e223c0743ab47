"""GPU parity over many batches on one context: the hash tables of the de-duplication rotate, and a batch's last launch empties
the next one's, by the list of the batch that used it (short lists) or in full (long ones).  Direct and recorded batches of two
sizes, stand-alone de-duplications and batches that report an error follow each other; every result equals the oracle's."""
import numpy as np
import pytest
import torch

from pathlib_helios import GpuCache, assert_same, gpu_path, oracle_path, to_bytes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def helios():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2310_00837_amd import helios as hl
    return hl


@pytest.mark.parametrize("max_deg,fanouts", [(2, [25, 10]), (40, [3, 3])])
def test_tables_over_many_batches(helios, oracle, max_deg, fanouts):
    rng = np.random.default_rng(max_deg)
    n = 30_000
    deg = rng.integers(max_deg // 2, max_deg + 1, n)
    off = np.zeros(n + 1, np.int64)
    off[1:] = np.cumsum(deg)
    idx = rng.integers(0, n, int(off[-1])).astype(np.int32)
    feats = torch.from_numpy(rng.integers(0, 1 << 30, (n, 4)).astype(np.int32))
    order = torch.from_numpy(rng.permutation(n).astype(np.int32))
    by_rank = to_bytes(feats)[order.numpy()]
    tabs = [np.ascontiguousarray(x) for x in (by_rank[:9_000], by_rank[9_000:15_000], by_rank[15_000:])]
    rank = oracle.rank_build(order.numpy())
    h = helios.Helios(0, stream=torch.cuda.Stream())
    off_d, idx_d = torch.from_numpy(off).cuda(), torch.from_numpy(idx).cuda()
    torch.cuda.synchronize()
    h.csr_load(off_d, idx_d)
    cache = GpuCache(h, feats, order, 9_000, 6_000)  # noqa: F841
    sizes = {}
    h.reserve(700 * (1 + fanouts[0] * (1 + fanouts[1])))

    def plan_of(b):
        if b not in sizes:
            dev = h.device
            hops = helios.alloc_hops(b, fanouts, dev)
            cap = b + sum(hb.flat.numel() for hb in hops)
            ints = [torch.empty(cap, dtype=torch.int32, device=dev) for _ in range(5)]
            bufs = (hops, torch.zeros(2 * len(fanouts), dtype=torch.int64).pin_memory(), ints[0], ints[1],
                    torch.zeros(1, dtype=torch.int64).pin_memory(), torch.empty((cap, 16), dtype=torch.uint8, device=dev),
                    ints[2], ints[3], ints[4], torch.zeros(4, dtype=torch.int64).pin_memory())
            torch.cuda.synchronize()
            sizes[b] = (h.plan_create(b, fanouts, *bufs), bufs)
        return sizes[b]

    def want_of(seeds, rs):
        return oracle_path(oracle, off, idx, seeds, fanouts, rs, rank, 9_000, 6_000, *tabs, 16)

    for k, what in enumerate("direct plan plan dedup plan bad direct plan small plan small bad plan direct dedup small direct".split()):
        print(k, what, flush=True)
        b = 90 if what == "small" else 700
        seeds = rng.integers(0, n, b).astype(np.int32)
        if what == "dedup":
            ids = rng.integers(0, n, 5_000).astype(np.int32)
            t = torch.from_numpy(ids).cuda()
            uq, inv, nu = torch.empty_like(t), torch.empty_like(t), torch.zeros(1, dtype=torch.int64).pin_memory()
            torch.cuda.synchronize()
            h.dedup(t, uq, inv, nu)
            h.sync()
            wu, wi = oracle.dedup(n, ids)
            assert np.array_equal(uq[:wu.size].cpu().numpy(), wu) and np.array_equal(inv.cpu().numpy(), wi)
            continue
        if what == "bad":
            seeds[5] = n + 7
        s = torch.from_numpy(seeds).cuda()
        torch.cuda.synchronize()
        if what == "direct":
            assert_same(gpu_path(h, helios, s, fanouts, k, fused=True), want_of(seeds, k))
            continue
        plan, bufs = plan_of(b)
        plan.launch(s, k)
        if what == "bad":
            with pytest.raises(helios.HeliosError) as e:
                plan.wait()
            assert e.value.code == helios.EDATA
            continue
        plan.wait()
        want = want_of(seeds, k)
        u = want["unique"].size
        assert int(bufs[4][0]) == u and np.array_equal(bufs[2][:u].cpu().numpy(), want["unique"])
        assert np.array_equal(bufs[3][:want["inverse"].size].cpu().numpy(), want["inverse"])
        assert np.array_equal(bufs[9].numpy(), want["stats"])
        for hb, (fr, ip, fl) in zip(bufs[0], want["hops"]):
            assert np.array_equal(hb.frontier[:fr.size].cpu().numpy(), fr) and np.array_equal(hb.flat[:fl.size].cpu().numpy(), fl)
    h.close()


@pytest.mark.parametrize("recorded", [False, True])
def test_batches_queued_behind_one_whose_buffers_overlap(helios, oracle, recorded):
    """A batch whose size array lies inside one of its own indptr buffers: two nodes get places that others have, so what the list
    remembers of the samples that meet there is one of them.  It is reported, and the batches queued behind it, the third of
    which uses its table again, come out as if it had not been."""
    rng = np.random.default_rng(5)
    n, b, fanouts = 2000, 8, [30, 20]               # short lists against the worst case: emptied by list
    off = np.arange(n + 1, dtype=np.int64) * 12
    idx = rng.integers(0, n, 12 * n).astype(np.int32)
    feats = torch.from_numpy(rng.integers(0, 1 << 30, (n, 4)).astype(np.int32))
    order = torch.from_numpy(rng.permutation(n).astype(np.int32))
    by_rank = to_bytes(feats)[order.numpy()]
    tabs = [np.ascontiguousarray(x) for x in (by_rank[:100], by_rank[100:200], by_rank[200:])]
    rank = oracle.rank_build(order.numpy())
    h = helios.Helios(0, stream=torch.cuda.Stream())
    off_d, idx_d = torch.from_numpy(off).cuda(), torch.from_numpy(idx).cuda()
    torch.cuda.synchronize()
    h.csr_load(off_d, idx_d)
    cache = GpuCache(h, feats, order, 100, 100)  # noqa: F841
    h.reserve(b * (1 + fanouts[0] * (1 + fanouts[1])))

    def buffers(overlap):
        hops = helios.alloc_hops(b, fanouts, h.device)
        cap = b + sum(hb.flat.numel() for hb in hops)
        ints = [torch.empty(cap, dtype=torch.int32, device=h.device) for _ in range(5)]
        sizes = hops[1].indptr[3:7] if overlap else torch.zeros(4, dtype=torch.int64).pin_memory()
        return (hops, sizes, ints[0], ints[1], torch.zeros(1, dtype=torch.int64).pin_memory(),
                torch.full((cap, 16), 0xA5, dtype=torch.uint8, device=h.device), ints[2], ints[3], ints[4],
                torch.zeros(4, dtype=torch.int64).pin_memory())

    sets = [buffers(k == 0) for k in range(5)]
    torch.cuda.synchronize()
    plans = [h.plan_create(b, fanouts, *s) for s in sets] if recorded else []
    for k in range(6):
        print("overlap", recorded, k, flush=True)
        seeds = [rng.integers(0, n, b).astype(np.int32) for _ in sets]
        seeds_d = [torch.from_numpy(s).cuda() for s in seeds]
        torch.cuda.synchronize()
        for m in range(5):
            if recorded:
                plans[m].launch(seeds_d[m], 10 * k + m)
            else:
                h.prepare_batch(seeds_d[m], fanouts, 10 * k + m, *sets[m])
        with pytest.raises(helios.HeliosError) as e:
            plans[0].wait() if recorded else h.sync()
        assert e.value.code == helios.EDATA
        h.sync()
        for m in range(1, 5):
            hops, sizes, unique, inverse, nu, out, mp, mi, ms, stats = sets[m]
            want = oracle_path(oracle, off, idx, seeds[m], fanouts, 10 * k + m, rank, 100, 100, *tabs, 16)
            u, nm = int(nu[0]), int(stats[3])
            assert u == want["unique"].size, (k, m)
            got = dict(hops=[(hb.frontier[:fr.size].cpu().numpy(), hb.indptr[:ip.size].cpu().numpy(), hb.flat[:fl.size].cpu().numpy())
                             for hb, (fr, ip, fl) in zip(hops, want["hops"])],
                       unique=unique[:u].cpu().numpy(), inverse=inverse[:want["inverse"].size].cpu().numpy(), stats=stats.numpy().copy(),
                       miss_pos=mp[:nm].cpu().numpy(), miss_id=mi[:nm].cpu().numpy(), miss_slot=ms[:nm].cpu().numpy())
            assert_same(got, want)
            hit = np.setdiff1d(np.arange(u), got["miss_pos"])
            assert np.array_equal(out[:u].cpu().numpy()[hit], want["out_before_miss"][hit])
    h.close()


@pytest.mark.parametrize("where", ["frontier 0", "frontier 1", "indptr 1", "flat 0", "flat 1"])
@pytest.mark.parametrize("recorded", [False, True])
@pytest.mark.parametrize("bad", [False, True])
def test_inverse_in_the_memory_of_a_hop(helios, oracle, where, recorded, bad):
    """The inverse map over a buffer of the hops, whose content is lost in its favour; with a graph that holds no node IDs in
    places, what stands there meanwhile may be any number."""
    rng = np.random.default_rng(8)
    n, b, fanouts = 9_000, 600, [7, 4]
    off = np.arange(n + 1, dtype=np.int64) * 6
    idx = rng.integers(0, n, 6 * n).astype(np.int32)
    feats = torch.from_numpy(rng.integers(0, 1 << 30, (n, 4)).astype(np.int32))
    order = torch.from_numpy(rng.permutation(n).astype(np.int32))
    seeds = rng.integers(0, n, b).astype(np.int32)
    h = helios.Helios(0, stream=torch.cuda.Stream())
    graph = idx.copy()
    if bad:
        graph[::7] = rng.integers(-(1 << 31), -(1 << 30), graph[::7].size)
    off_d, graph_d, seeds_d = torch.from_numpy(off).cuda(), torch.from_numpy(graph).cuda(), torch.from_numpy(seeds).cuda()
    torch.cuda.synchronize()
    h.csr_load(off_d, graph_d)
    cache = GpuCache(h, feats, order, n, 0)  # noqa: F841
    hops = helios.alloc_hops(b, fanouts, h.device)
    cap = b + sum(hb.flat.numel() for hb in hops)
    unique, inverse, mp, mi, ms = [torch.empty(cap, dtype=torch.int32, device=h.device) for _ in range(5)]
    what, k = where.split()[0], int(where[-1])
    fr, ip, fl = hops[k].frontier, hops[k].indptr, hops[k].flat
    if what == "frontier":
        fr = inverse[:fr.numel()]
    elif what == "indptr":
        ip = inverse[:2 * ip.numel()].view(torch.int64)
    else:
        fl = inverse[:fl.numel()]
    hops[k] = helios.HopBuffers(fr, ip, fl)
    sizes, nu, stats = [torch.zeros(m, dtype=torch.int64).pin_memory() for m in (4, 1, 4)]
    bufs = (hops, sizes, unique, inverse, nu, torch.empty((cap, 16), dtype=torch.uint8, device=h.device), mp, mi, ms, stats)
    torch.cuda.synchronize()
    plan = h.plan_create(b, fanouts, *bufs) if recorded else None
    tab = np.ascontiguousarray(to_bytes(feats)[order.numpy()])
    for rs in range(3):
        print("inverse over", where, recorded, bad, rs, flush=True)
        if recorded:
            plan.launch(seeds_d, rs)
        else:
            h.prepare_batch(seeds_d, fanouts, rs, *bufs)
        if bad:
            with pytest.raises(helios.HeliosError) as e:
                h.sync()
            assert e.value.code == helios.EDATA
            continue
        h.sync()
        want = oracle_path(oracle, off, idx, seeds, fanouts, rs, oracle.rank_build(order.numpy()), n, 0, tab, tab[:0], tab[:0], 16)
        assert int(nu[0]) == want["unique"].size and np.array_equal(unique[:int(nu[0])].cpu().numpy(), want["unique"])
        assert np.array_equal(inverse[:want["inverse"].size].cpu().numpy(), want["inverse"])
        assert [int(x) for x in sizes] == [x for hop in want["hops"] for x in (hop[0].size, hop[2].size)]
    h.close()
