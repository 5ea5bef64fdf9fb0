"""GPU parity at the sizes where a kernel's tiling or a dispatch rule changes: edges of slices and blocks, remainders, the
smallest and largest of a range.  Everything compared here is integer or copied data: exact equality with the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
from gpu_common import HipBatch, assert_batch_equal, log

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module")
def B():
    from paper_2505_10806_amd import binding
    return binding


@pytest.fixture(scope="module")
def ctx(B):
    c = B.Context(0)
    yield c
    c.close()


def _i32(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.int32), device=DEV)


def _sparse_graph(n, active, degree, rng):
    """A graph of n nodes of which `active`, spread over the whole id range (both ends among them), have about `degree`
    neighbours, all active."""
    ids = np.unique(np.concatenate([[0, n - 1], rng.integers(0, n, active)]))
    deg = np.zeros(n, dtype=np.int64)
    deg[ids] = rng.integers(0, 2 * degree + 1, ids.size)
    rp = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(deg, out=rp[1:])
    return rp, ids[rng.integers(0, ids.size, rp[-1])].astype(np.int32), ids


# nodes, active nodes, mean degree, seeds per batch, fan-outs.  A slice of the marking pass covers at most 1,280,000 ids;
# above 4 Mi nodes few edges take the atomic marking; above 40,960,000 nodes there are no slices at all.
@pytest.mark.parametrize("n,active,degree,seeds,fanouts", [
    (31, 31, 3, [4], (3, 2)),                           # one launch for all hops: up to 20,480 edges (8192 above 131,072 nodes)
    (131_072, 60_000, 30, [310, 0, 1], (10, 5)),
    (131_072, 60_000, 30, [400, 300], (10, 5)),         # just too many edges for that
    (131_041, 90_000, 9, [15, 16], (16, 0, 32)),
    (524_288, 80_000, 30, [120, 64], (10, 5)),
    (524_289, 80_000, 30, [120, 64], (10, 5)),
    (1_279_999, 3000, 8, [40, 7], (5, 3)),              # one slice, last word partial
    (1_280_001, 3000, 8, [40, 7, 0], (5, 3)),           # a second slice of few words
    (20_000, 20_000, 40, [700, 900], (32, 31)),         # most ids of a tier workgroup's words are new
    (200_001, 150_000, 30, [1000, 1, 999], (25, 10)),   # the edge list split between workgroups
    (200_001, 150_000, 30, [9000, 1], (7, 2)),          # more seeds than one launch marks
    (200_001, 150_000, 30, [9000] + [40, 0, 1] * 5, (3, 2)),         # the same with the longest table of buffers
    (300_007, 250_000, 30, [1300, 600, 0], (10, 10, 40)),            # over 131,072 frontier nodes counted by a launch of their own
    (3_000_017, 400_000, 12, [900] * 8, (40, 3)),       # wavefront-per-node draw in front of the slices
    (300_007, 250_000, 30, [1500, 0, 1200, 1, 900, 1500, 1500, 1500], (25, 10)),    # over 2.2 M edges: first-seen order by rank words
    (300_007, 250_000, 30, [1500] * 4, (40, 10)),
    (2_600_021, 2_500_000, 20, [2000, 1900, 0], (15, 10, 5)),
    (2_600_021, 900_000, 12, [2000] * 4, (15, 10, 5)),
    (4_194_337, 200_000, 12, [60, 50], (5, 3)),         # atomic marking on a graph that has slices
    (4_194_337, 200_000, 30, [60, 50], (25, 20)),       # the same by a lane per draw
    (4_194_337, 200_000, 12, [3000, 2000], (15, 10)),   # slices again: the edges outweigh the bitmaps
    (41_000_033, 200_000, 12, [300, 200], (5, 3)),      # no slices
])
@pytest.mark.parametrize("first_seen", [False, True])
def test_blocks_across_the_ways_to_build_a_tier(B, ctx, n, active, degree, seeds, fanouts, first_seen):
    log(f"[tiers] N={n} active={active} seeds={seeds} fanouts={fanouts} first_seen={first_seen}")
    rng = np.random.default_rng(n % 1000 + len(seeds))
    rp, ci, ids = _sparse_graph(n, active, degree, rng)
    csr = B.CsrGraph(torch.as_tensor(rp, device=DEV).to(torch.int32), _i32(ci))
    order = oracle.ORDER_FIRST_SEEN if first_seen else oracle.ORDER_ASCENDING
    lists = [rng.permutation(ids)[:k].astype(np.int32) for k in seeds]
    outs = [B.BlockBuffers(n, ci.size, max(k, 1), fanouts, DEV) for k in seeds]
    for j, o in enumerate(outs):                        # edge lists that start at any 4-byte address
        for h in range(len(fanouts)):
            shift = lambda t: torch.full((t.numel() + 3,), -7, dtype=torch.int32, device=DEV)[(j + h) % 4:][:t.numel()]  # noqa: E731
            o.set_hop(h, shift(o.indptr[h]), shift(o.nbr[h]), shift(o.nbr_local[h]))
    for epoch in range(2):                              # the second call finds the first one's scratch
        ctx.sample_blocks_group(csr, [_i32(x) for x in lists], fanouts, 77, epoch, outs,
                                node_order=B.RG_ORDER_FIRST_SEEN if first_seen else B.RG_ORDER_ASCENDING)
        counts = torch.zeros(n, dtype=torch.int32, device=DEV)
        ctx.access_histogram_sampled(len(seeds), counts)    # the bitmaps hold the batches' input nodes
        want = np.zeros(n, dtype=np.uint32)
        for j, o in enumerate(outs):
            orc = oracle.sample_blocks(rp, ci, lists[j], fanouts, 77, epoch, order)
            assert_batch_equal(HipBatch(o, len(fanouts)), orc, len(fanouts), f"batch {j} epoch {epoch}")
            oracle.access_histogram(orc.input_nodes, want)
        assert np.array_equal(counts.cpu().numpy().view(np.uint32), want)
    if first_seen and n == 300_007:                     # without relabelling there is no room for the ranks: the same nodes
        again = [B.BlockBuffers(n, ci.size, max(k, 1), fanouts, DEV, with_local=False) for k in seeds]
        ctx.sample_blocks_group(csr, [_i32(x) for x in lists], fanouts, 77, 1, again, node_order=B.RG_ORDER_FIRST_SEEN)
        for o, w in zip(again, outs):
            k = int(o.tier_off[-1])
            assert torch.equal(o.tier_off, w.tier_off) and torch.equal(o.nodes[:k], w.nodes[:k])


# A tier workgroup of 24,576 ids has room for a third of them; more are stored and read back for the next hop's rows.
@pytest.mark.parametrize("fanouts,full_hop", [((15, 10, 5), 1), ((15, 20), 1), ((40, 10, 3), 0)])
def test_tiers_of_more_new_ids_than_a_workgroup_has_room_for(B, ctx, fanouts, full_hop):
    log(f"[dense tiers] fanouts={fanouts}")
    n, rng, per = 1_000_003, np.random.default_rng(5), 24_576
    active = np.concatenate([np.arange(4 * per - 100, 5 * per + 50), [0, 300_000, n - 1]])
    deg = np.zeros(n, dtype=np.int64)
    deg[active] = rng.integers(20, 60, active.size)
    rp = np.concatenate([[0], np.cumsum(deg)])
    ci = active[rng.integers(0, active.size, rp[-1])].astype(np.int32)
    csr = B.CsrGraph(torch.as_tensor(rp, device=DEV).to(torch.int32), _i32(ci))
    lists = [rng.permutation(active)[:k].astype(np.int32) for k in ([700] * 7 + [3])]
    outs = [B.BlockBuffers(n, ci.size, k.size, fanouts, DEV) for k in lists]
    ctx.sample_blocks_group(csr, [_i32(x) for x in lists], fanouts, 77, 1, outs)
    for j, o in enumerate(outs):
        orc = oracle.sample_blocks(rp, ci, lists[j], fanouts, 77, 1)
        tier = orc.nodes[orc.tier_off[full_hop + 1]:orc.tier_off[full_hop + 2]]
        assert j == 7 or np.bincount(tier // per).max() > per // 3
        assert_batch_equal(HipBatch(o, len(fanouts)), orc, len(fanouts), f"batch {j}")


# All neighbours of nodes that have far more of them than the average.
@pytest.mark.parametrize("first_seen", [False, True])
def test_blocks_of_hubs(B, ctx, first_seen):
    """16 batches with over twice the edges that the kernels which walk their lists are launched for."""
    log(f"[hubs] first_seen={first_seen}")
    n, hubs, rng = 400_000, 16, np.random.default_rng(9)
    ids = rng.permutation(n)[:hubs].astype(np.int32)
    deg = rng.integers(0, 3, n)
    deg[ids] = rng.integers(140_000, 160_000, hubs)
    rp = np.concatenate([[0], np.cumsum(deg)])
    ci = rng.integers(0, n, rp[-1]).astype(np.int32)
    csr = B.CsrGraph(torch.as_tensor(rp, device=DEV).to(torch.int32), _i32(ci))
    for fanouts in ((-1,), (-1, 1)):
        outs = [B.BlockBuffers(n, ci.size, 1, fanouts, DEV) for _ in range(hubs)]
        ctx.sample_blocks_group(csr, [_i32(ids[j:j + 1]) for j in range(hubs)], fanouts, 77, 1, outs,
                                node_order=B.RG_ORDER_FIRST_SEEN if first_seen else B.RG_ORDER_ASCENDING)
        for j, o in enumerate(outs):
            orc = oracle.sample_blocks(rp, ci, ids[j:j + 1], fanouts, 77, 1, oracle.ORDER_FIRST_SEEN if first_seen else oracle.ORDER_ASCENDING)
            assert_batch_equal(HipBatch(o, len(fanouts)), orc, len(fanouts), f"batch {j}")


# Count chunks of 1024 frontier nodes, 16,384 of them added up by the draw itself, more scanned by a launch of their own.
@pytest.mark.parametrize("seeds", [16_777_216, 16_777_217])
def test_blocks_of_very_large_frontiers(B, ctx, seeds):
    log(f"[very large frontiers] seeds={seeds}")
    n = 16_800_000
    deg = (np.arange(n) * 7 % 4).astype(np.int64)       # 0 to 3 neighbours, two at most drawn
    rp = np.concatenate([[0], np.cumsum(deg)])
    ci = (np.arange(rp[-1]) * 7919 % n).astype(np.int32)
    csr = B.CsrGraph(torch.as_tensor(rp, device=DEV).to(torch.int32), _i32(ci))
    ids = np.random.default_rng(1).permutation(n)[:seeds].astype(np.int32)
    out = B.BlockBuffers(n, ci.size, seeds, (2,), DEV)
    ctx.sample_blocks(csr, _i32(ids), seeds, (2,), 77, 2, out)
    assert_batch_equal(HipBatch(out, 1), oracle.sample_blocks(rp, ci, ids, (2,), 77, 2), 1)


# One launch for all hops (with its lists in LDS up to 65,536 nodes), slices, atomic marking; first-seen order by first edges and by rank words.
@pytest.mark.parametrize("n,active,degree,seeds,fanouts,first_seen", [
    (10_000, 10_000, 20, [250, 61, 0], (5, 4, 3), False),
    (65_536, 50_000, 9, [1030, 1, 1024], (2, 2, 1), False),
    (131_072, 60_000, 30, [300, 40], (10, 5), False),
    (300_007, 250_000, 30, [1500, 0, 900], (25, 10, 3), False),
    (4_194_337, 200_000, 12, [60, 50], (5, 3), False),
    (131_072, 60_000, 30, [300, 40], (10, 5), True),
    (300_007, 250_000, 30, [1500] * 8, (25, 10), True),
])
@pytest.mark.parametrize("what", ["nbr", "indptr", "all"])
def test_blocks_with_one_list_buffer_for_all_hops(B, ctx, n, active, degree, seeds, fanouts, first_seen, what):
    """A caller that keeps only the positions passes the same nbr (and indptr) buffer for every hop: each hop's positions are
    those of its own edges; what is left in the shared lists is the last hop's."""
    log(f"[shared lists] N={n} seeds={seeds} fanouts={fanouts} first_seen={first_seen} what={what}")
    rng = np.random.default_rng(n % 1000 + len(seeds))
    rp, ci, ids = _sparse_graph(n, active, degree, rng)
    csr = B.CsrGraph(torch.as_tensor(rp, device=DEV).to(torch.int32), _i32(ci))
    lists = [rng.permutation(ids)[:k].astype(np.int32) for k in seeds]
    outs, H = [B.BlockBuffers(n, ci.size, max(k, 1), fanouts, DEV) for k in seeds], len(fanouts)
    for o in outs:
        for t in o.nbr_local:
            t.fill_(-7)
        room = {k: max(getattr(o, k), key=lambda t: t.numel()) for k in ("indptr", "nbr", "nbr_local")}
        for h in range(H):
            o.set_hop(h, **({"indptr": room["indptr"]} if what in ("indptr", "all") else {}))
            if what in ("nbr", "all"):                  # set_hop wants both lists of a hop to hold the same number of edges
                o.set_hop(h, nbr=room["nbr"])
                o.set_hop(h, nbr_local=room["nbr_local"] if what == "all" else torch.full_like(room["nbr_local"], -7))
    ctx.sample_blocks_group(csr, [_i32(x) for x in lists], fanouts, 77, 3, outs,
                            node_order=B.RG_ORDER_FIRST_SEEN if first_seen else B.RG_ORDER_ASCENDING)
    order = oracle.ORDER_FIRST_SEEN if first_seen else oracle.ORDER_ASCENDING
    for j, o in enumerate(outs):
        orc = oracle.sample_blocks(rp, ci, lists[j], fanouts, 77, 3, order)
        assert o.tier_off.cpu().tolist() == orc.tier_off.tolist()
        assert np.array_equal(o.nodes[:orc.nodes.size].cpu().numpy(), orc.nodes)
        for h in range(H):
            last, e = h == H - 1, orc.nbr[h].size
            if what != "all" or last:
                assert np.array_equal(o.nbr_local[h][:e].cpu().numpy(), orc.nbr_local[h]), f"batch {j} hop {h}"
            if what == "indptr" or last:
                assert np.array_equal(o.nbr[h][:e].cpu().numpy(), orc.nbr[h]), f"batch {j} hop {h}"
            if what == "nbr" or last:
                assert np.array_equal(o.indptr[h][:orc.indptr[h].size].cpu().numpy(), orc.indptr[h]), f"batch {j} hop {h}"


# One launch with its lists in LDS and without, slices, first edges; enough edges for rank words, which need lists of their own.
@pytest.mark.parametrize("n,seeds,fanouts,first_seen", [
    (10_000, [250, 61], (5, 4, 3), False), (131_072, [250, 61], (5, 4, 3), False), (300_007, [250, 61], (5, 4, 3), False),
    (10_000, [250, 61], (5, 4, 3), True), (300_007, [1500] * 8, (25, 10), True)])
def test_blocks_whose_positions_replace_the_ids(B, ctx, n, seeds, fanouts, first_seen):
    """One list for a hop's ids and positions: the positions are what stays."""
    rng, order = np.random.default_rng(n), oracle.ORDER_FIRST_SEEN if first_seen else oracle.ORDER_ASCENDING
    rp, ci, ids = _sparse_graph(n, n // 2, 20, rng)
    csr = B.CsrGraph(torch.as_tensor(rp, device=DEV).to(torch.int32), _i32(ci))
    lists = [rng.permutation(ids)[:k].astype(np.int32) for k in seeds]
    outs = [B.BlockBuffers(n, ci.size, k, fanouts, DEV) for k in seeds]
    for o in outs:
        for h in range(len(fanouts)):
            o.set_hop(h, nbr_local=o.nbr[h])
    ctx.sample_blocks_group(csr, [_i32(x) for x in lists], fanouts, 77, 3, outs,
                            node_order=B.RG_ORDER_FIRST_SEEN if first_seen else B.RG_ORDER_ASCENDING)
    for j, o in enumerate(outs):
        orc, hip = oracle.sample_blocks(rp, ci, lists[j], fanouts, 77, 3, order), HipBatch(o, len(fanouts))
        hip.nbr = orc.nbr
        assert_batch_equal(hip, orc, len(fanouts), f"batch {j}")


def test_decoupled_misses_wait_for_the_reader_of_their_buffer(B):
    """The miss rows of batch b + 2 go into batch b's output buffer: they wait for what on_batch queued on the gather stream,
    however late it runs (here behind a long spin)."""
    import synth
    from paper_2505_10806_amd.pipeline import EpochPipeline
    wl = synth.build_workload("tiny", seed=4, device=DEV)
    pipe = EpochPipeline(wl, device=DEV)
    assert pipe.decoupled and pipe.queue_depth == 2
    nb, dim = pipe.batches_per_epoch, wl.cfg.feat_dim
    taken = []

    def on_batch(p, b):
        torch.cuda._sleep(10_000_000)                   # some milliseconds
        taken.append(p.out[:p.sizes[b], :dim].clone())

    with torch.cuda.stream(torch.cuda.Stream()):
        pipe.run_epochs(0, 2, nb, on_batch=on_batch)
        torch.cuda.synchronize()
        for b in range(nb):
            nodes = pipe.arena[b, :pipe.sizes[b]].long()
            assert torch.equal(taken[nb + b], wl.features[nodes]), f"batch {b}"
    pipe.close()


# One workgroup up to 4096 ids; buckets with LDS counters up to 8 Mi ids, with counters in HBM above.
@pytest.mark.parametrize("n", [3, 4095, 4096, 4097, 262_145, 1_000_003, 8_388_609])
def test_schedule_bucket_edges(ctx, n):
    log(f"[schedule edges] n={n}")
    ids = np.random.default_rng(n).permutation(2 * n)[:n].astype(np.int32)
    dev = _i32(ids)
    out = ctx.epoch_schedule(dev, (3 << 32) + 1, 9, dev)          # in place
    assert np.array_equal(out.cpu().numpy(), oracle.epoch_schedule(ids, (3 << 32) + 1, 9))


def test_schedule_of_ids_picked_for_one_bucket(ctx):
    """Every id's key starts with the same four bits: one of the sixteen buckets of 6000 ids holds them all, more than a workgroup
    sorts in LDS; the others are empty."""
    seed, epoch = 2025, 4
    cand = np.arange(104_000, dtype=np.uint32)
    top = np.array([oracle.philox4x32_10(np.array([v, 0xFFFFFFFF, 0, epoch]), np.array([seed, 0]))[0] >> 28 for v in cand])
    ids = cand[top == 5][:6000].astype(np.int32)
    assert ids.size == 6000
    got = ctx.epoch_schedule(_i32(ids), seed, epoch)
    assert np.array_equal(got.cpu().numpy(), oracle.epoch_schedule(ids, seed, epoch))


# A bucket has room for 2560 ids; an overfull one is sorted in tiles of 2048 that are merged.
@pytest.mark.parametrize("in_bucket", [2560, 2561, 4096, 4097, 10_001, 16_500])
def test_schedule_bucket_with_more_ids_than_room(ctx, in_bucket):
    """402,000 ids in 256 buckets, the first of which gets in_bucket of them."""
    n, seed, epoch = 402_000, 2025, 4
    order = oracle.epoch_schedule(np.arange(4_600_000, dtype=np.int32), seed, epoch)     # ascending by key: 18,000 ids or so to each of the 256
    key = lambda v: oracle.philox4x32_10(np.array([v, 0xFFFFFFFF, 0, epoch]), np.array([seed, 0]))[0] >> 24  # noqa: E731
    assert key(order[17_000]) == 0 and key(order[19_000]) == 1
    rng = np.random.default_rng(in_bucket)
    ids = rng.permutation(np.concatenate([rng.permutation(order[:17_000])[:in_bucket], rng.permutation(order[19_000:])[:n - in_bucket]]))
    got = ctx.epoch_schedule(_i32(ids), seed, epoch)
    assert np.array_equal(got.cpu().numpy(), oracle.epoch_schedule(ids, seed, epoch))


# Chunks of 1024 slots, wavefronts of 64; one key for all slots, a key per slot, keys in descending order.
@pytest.mark.parametrize("slots", [1, 63, 65, 1024, 1025, 70_001])
@pytest.mark.parametrize("pattern", ["one", "cycle", "descending", "random"])
def test_ordered_plan_chunk_edges(B, ctx, slots, pattern):
    log(f"[plan] slots={slots} pattern={pattern}")
    nb = 1023 if pattern != "random" else 192
    first = {"one": np.full(slots, 5), "cycle": np.arange(slots) % (nb + 1), "descending": nb - np.arange(slots) * (nb + 1) // slots,
             "random": np.random.default_rng(slots).integers(0, nb + 2, slots)}[pattern].astype(np.int32)
    home = _i32((2 << 30) + np.arange(slots)[::-1].astype(np.int64) - (1 << 32))       # every node remote, rows descending
    cache = B.FeatureCache(slots, slots, 4, DEV)
    ctx.build_cache(torch.ones(slots, dtype=torch.int32, device=DEV), home, None, 4, cache)
    plan = B.PrefetchPlan(slots, nb, DEV)
    ctx.plan_prefetch(cache, home, _i32(first), plan)
    key = np.minimum(first, nb)
    order = np.argsort(key, kind="stable")
    pairs = plan.list.cpu().numpy().reshape(-1, 2)
    assert np.array_equal(pairs[:, 0], order) and np.array_equal(pairs[:, 1], slots - 1 - order)
    assert np.array_equal(plan.offsets.cpu().numpy(), np.searchsorted(key[order], np.arange(nb + 2)))


# Fewer rows cached than the capacity has chunks for: none, the edges of a chunk, after a plan of all rows.
@pytest.mark.parametrize("cached", [0, 1, 1023, 1024, 1025, 300_000])
def test_ordered_plan_of_few_cached_rows(B, ctx, cached):
    log(f"[plan] cached={cached}")
    n, nb = 300_000, 7
    home, first = _i32((2 << 30) + np.arange(n, dtype=np.int64) - (1 << 32)), np.arange(n, dtype=np.int32)[::-1] % (nb + 1)
    cache, plan = B.FeatureCache(n, n, 4, DEV), B.PrefetchPlan(n, nb, DEV)
    for k in (n, cached):
        ids = np.random.default_rng(k).permutation(n)[:k]
        counts = torch.zeros(n, dtype=torch.int32, device=DEV)
        counts[torch.as_tensor(ids, device=DEV)] = 1
        ctx.build_cache(counts, home, None, 4, cache)
        ctx.plan_prefetch(cache, home, _i32(first), plan)
        ids = np.sort(ids)                              # slots in ascending id
        order = np.argsort(first[ids], kind="stable")
        pairs = plan.list.cpu().numpy().reshape(-1, 2)[:k]
        assert np.array_equal(pairs[:, 0], order) and np.array_equal(pairs[:, 1], ids[order])
        assert np.array_equal(plan.offsets.cpu().numpy(), np.searchsorted(first[ids][order], np.arange(nb + 2)))


# Ranges of 512 ids at least, two workgroups per compute unit, 2 Mi bounds per launch; runs whose ids are far from proportional.
@pytest.mark.parametrize("n,batches,hops", [(511, 3, 1), (513, 3, 2), (262_145, 9, 2), (300_000, 5000, 1), (300_000, 12_000, 1), (5_000_011, 2, 3)])
@pytest.mark.parametrize("skew", [1, 4])
def test_epoch_histogram_range_edges(B, ctx, n, batches, hops, skew):
    log(f"[histogram ranges] N={n} batches={batches} hops={hops} skew={skew}")
    rng = np.random.default_rng(n + skew)
    per = min(n // (hops + 1), 40_000 if batches < 10 else 60)
    arena = np.zeros((batches, per * hops + 2), dtype=np.int32)
    tier_offs = np.zeros((batches, hops + 2), dtype=np.int32)
    want, first = np.zeros(n, dtype=np.uint32), np.full(n, 0xFFFFFFFF, dtype=np.uint32)
    for b in range(batches):
        ids = np.unique((n * rng.random(per * hops) ** skew).astype(np.int32))       # distinct; skew 4 crowds the low ids
        ids = np.union1d(ids, [0, n - 1])[:arena.shape[1]].astype(np.int32)
        tier = rng.integers(0, hops + 1, ids.size) if b % 3 else np.full(ids.size, hops)   # every third batch: one full tier
        parts = [ids[tier == t] for t in range(hops + 1)]
        arena[b, :ids.size] = np.concatenate([rng.permutation(parts[0])] + parts[1:])
        tier_offs[b, 1:] = np.cumsum([p.size for p in parts])
        oracle.access_histogram(ids, want)
        first[ids] = np.minimum(first[ids], b)
    counts = torch.zeros(n, dtype=torch.int32, device=DEV)
    got_first = torch.full((n,), -1, dtype=torch.int32, device=DEV)
    most = int(tier_offs[:, 1].max())
    ctx.access_histogram_epoch(_i32(arena), _i32(tier_offs), batches, hops, most, counts, first_batch=got_first)
    assert np.array_equal(counts.cpu().numpy().view(np.uint32), want)
    assert np.array_equal(got_first.cpu().numpy().view(np.uint32), first)
    ctx.access_histogram_epoch(_i32(arena), _i32(tier_offs), batches, hops, most, counts)
    assert np.array_equal(counts.cpu().numpy().view(np.uint32), 2 * want)


# Seeds beside the bounds: 256 to 1024 of them to a workgroup, more of many batches and above 65,536; workgroups of one row of the grid and of
# several; batches of fewer seeds than the most.
@pytest.mark.parametrize("n,batches,most", [(90_000, 300, 256), (90_000, 300, 1025), (300_000, 300, 3073), (90_000, 200, 65_537), (300_000, 100, 9000), (3_000_000, 20, 70_000)])
def test_epoch_histogram_of_many_seeds(B, ctx, n, batches, most):
    log(f"[histogram seeds] N={n} batches={batches} most={most}")
    rng, tail = np.random.default_rng(most), 2000 if batches >= 100 else 50_000
    arena = np.zeros((batches, most + 2 * tail), dtype=np.int32)
    tier_offs = np.zeros((batches, 4), dtype=np.int32)
    want, first = np.zeros(n, dtype=np.int64), np.full(n, 0xFFFFFFFF, dtype=np.uint32)
    for b in range(batches):
        seeds = most if b in (0, batches - 1) else int(rng.integers(0, most + 1)) * (b % 4 > 0)
        parts = [rng.integers(0, n, seeds), np.sort(rng.choice(n, tail, replace=False)), np.sort(rng.choice(n, tail, replace=False))]
        tier_offs[b, 1:] = np.cumsum([p.size for p in parts])
        ids = np.concatenate(parts)
        arena[b, :ids.size] = ids
        want += np.bincount(ids, minlength=n)
        first[ids] = np.minimum(first[ids], b)
    counts = torch.zeros(n, dtype=torch.int32, device=DEV)
    got_first = torch.full((n,), -1, dtype=torch.int32, device=DEV)
    ctx.access_histogram_epoch(_i32(arena), _i32(tier_offs), batches, 2, most, counts, first_batch=got_first)
    assert np.array_equal(counts.cpu().numpy(), want)
    assert np.array_equal(got_first.cpu().numpy().view(np.uint32), first)


# Segments of one wavefront's lanes, one more, one round of loads and one more, with and without bounds found first.
@pytest.mark.parametrize("batches", [1, 10_000])
def test_epoch_histogram_segment_lengths(B, ctx, batches):
    log(f"[histogram segments] batches={batches}")
    lengths = [0, 1, 63, 64, 65, 255, 256, 257, 400]
    runs = [np.sort(np.random.default_rng(k).permutation(400)[:k]) for k in lengths]
    arena, tier_offs = np.zeros((batches, 1370), dtype=np.int32), np.zeros((batches, 10), dtype=np.int32)
    arena[:, :1361] = np.concatenate(runs)
    tier_offs[:, 2:] = np.cumsum(lengths[1:])
    want = np.bincount(arena[0, :1361], minlength=1024).astype(np.uint32)
    first = np.where(want > 0, 0, 0xFFFFFFFF).astype(np.uint32)
    counts, got = torch.zeros(1024, dtype=torch.int32, device=DEV), torch.full((1024,), -1, dtype=torch.int32, device=DEV)
    ctx.access_histogram_epoch(_i32(arena), _i32(tier_offs), batches, 8, 0, counts, first_batch=got)
    assert np.array_equal(counts.cpu().numpy().view(np.uint32), batches * want)
    assert np.array_equal(got.cpu().numpy().view(np.uint32), first)
    ctx.access_histogram_epoch(_i32(arena), _i32(tier_offs), batches, 8, 0, counts)
    assert np.array_equal(counts.cpu().numpy().view(np.uint32), 2 * batches * want)


# Every capacity of a small curve against sorted counts: bins at both ends of a thread's share, the clamped bin and sums above 2^32.
@pytest.mark.parametrize("values", [[1], [7, 8, 9], [2040, 2046, 2047, 2048], [1, 15, 16, 2039, 2040, 3_000_000_000]])
def test_hit_curve_bins(B, ctx, values):
    log(f"[hit curve bins] {values}")
    n = 37
    counts = np.random.default_rng(len(values)).choice(np.array(values + [0], dtype=np.uint32), n)
    home = np.where(np.arange(n) % 5 == 0, np.arange(n), (2 << 30) + np.arange(n)).astype(np.uint32).view(np.int32)
    best = np.sort(np.where(np.arange(n) % 5 == 0, 0, counts).astype(np.uint64))[::-1]
    caps = list(range(n + 2))
    hits, total = ctx.cache_hit_curve(torch.as_tensor(counts.view(np.int32), device=DEV), torch.as_tensor(home, device=DEV), caps)
    assert hits.tolist() == [int(best[:k].sum()) for k in caps] and int(total) == int(best.sum())


def _captured(call):
    """The call recorded into a graph on a side stream."""
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        graph.capture_begin(capture_error_mode="global")
        call()
        graph.capture_end()
    torch.cuda.synchronize()
    return graph


# The first histogram of a context inside a captured graph, where no scratch can be allocated: runs searched by the counting kernel.
@pytest.mark.parametrize("n,batches,hops", [(700, 3, 1), (300_007, 200, 3), (4_300_001, 5, 8)])
def test_epoch_histogram_without_scratch(B, n, batches, hops):
    log(f"[captured histogram] N={n} batches={batches} hops={hops}")
    rng = np.random.default_rng(n)
    per = min(n // 2, 300 * hops)
    arena, tier_offs = np.zeros((batches, per + 2), dtype=np.int32), np.zeros((batches, hops + 2), dtype=np.int32)
    want, first = np.zeros(n, dtype=np.uint32), np.full(n, 0xFFFFFFFF, dtype=np.uint32)
    for b in range(batches):
        ids = np.union1d(rng.integers(0, n, per), [0, n - 1])[:per + 2].astype(np.int32)
        tier = rng.integers(0, hops + 1, ids.size)
        parts = [ids[tier == t] for t in range(hops + 1)]
        arena[b, :ids.size] = np.concatenate(parts)
        tier_offs[b, 1:] = np.cumsum([p.size for p in parts])
        oracle.access_histogram(ids, want)
        first[ids] = np.minimum(first[ids], b)
    arena_d, tiers_d, most = _i32(arena), _i32(tier_offs), int(tier_offs[:, 1].max())
    counts, got_first = torch.zeros(n, dtype=torch.int32, device=DEV), torch.full((n,), -1, dtype=torch.int32, device=DEV)
    ctx = B.Context(0)
    graph = _captured(lambda: ctx.access_histogram_epoch(arena_d, tiers_d, batches, hops, most, counts, first_batch=got_first))
    plain = _captured(lambda: ctx.access_histogram_epoch(arena_d, tiers_d, batches, hops, most, counts))
    for replay in range(3):
        counts.zero_()
        got_first.fill_(-1)
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(counts.cpu().numpy().view(np.uint32), want)
        assert np.array_equal(got_first.cpu().numpy().view(np.uint32), first)
        plain.replay()
        torch.cuda.synchronize()
        assert np.array_equal(counts.cpu().numpy().view(np.uint32), 2 * want)
    del graph, plain
    ctx.close()


# Calls whose tier kernels want scratch that the context's earlier calls had no use for, captured: ascending order after first-seen
# order, small first-seen calls after calls of over 2.2 M edges, more hops, and the other ways round.
@pytest.mark.parametrize("warm_seeds,warm_fanouts,warm_seen,seeds,fanouts,seen", [
    ([600, 500], (25, 10), True, [600, 500], (25, 10), False),
    ([600, 500], (25, 10), False, [600, 500], (24, 2, 2), False),
    ([1500] * 8, (25, 10), True, [40] * 8, (5, 3), True),
    ([1500] * 8, (25, 10), True, [1500] * 8, (25, 10), True),
])
def test_captured_call_after_another_kind(B, warm_seeds, warm_fanouts, warm_seen, seeds, fanouts, seen):
    log(f"[captured sampler] {warm_seeds} {warm_fanouts} {warm_seen} -> {seeds} {fanouts} {seen}")
    n = 300_007
    rng = np.random.default_rng(len(seeds) + sum(fanouts))
    rp, ci, ids = _sparse_graph(n, 250_000, 30, rng)
    csr = B.CsrGraph(torch.as_tensor(rp, device=DEV).to(torch.int32), _i32(ci))
    kind = lambda first: B.RG_ORDER_FIRST_SEEN if first else B.RG_ORDER_ASCENDING  # noqa: E731
    warm = [rng.permutation(ids)[:k].astype(np.int32) for k in warm_seeds]
    lists = [rng.permutation(ids)[:k].astype(np.int32) for k in seeds]
    lists_d = [_i32(x) for x in lists]
    outs = [B.BlockBuffers(n, ci.size, k, fanouts, DEV) for k in seeds]
    warm_d, warm_outs = [_i32(x) for x in warm], [B.BlockBuffers(n, ci.size, k, warm_fanouts, DEV) for k in warm_seeds]
    ctx = B.Context(0)
    ctx.sample_blocks_group(csr, warm_d, warm_fanouts, 77, 0, warm_outs, node_order=kind(warm_seen))
    graph = _captured(lambda: ctx.sample_blocks_group(csr, lists_d, fanouts, 77, 1, outs, node_order=kind(seen)))
    order = oracle.ORDER_FIRST_SEEN if seen else oracle.ORDER_ASCENDING
    want = [oracle.sample_blocks(rp, ci, x, fanouts, 77, 1, order) for x in lists]
    for replay in range(3):
        for o in outs:
            o.nodes.fill_(-7)
            o.tier_off.fill_(0)
        graph.replay()
        for j, o in enumerate(outs):
            assert_batch_equal(HipBatch(o, len(fanouts)), want[j], len(fanouts), f"batch {j} replay {replay}")
        # calls of either kind between the replays make the scratch that the captured one did without, and free none of its own
        ctx.sample_blocks_group(csr, lists_d, fanouts, 77, 1, outs, node_order=kind(seen))
        ctx.sample_blocks_group(csr, warm_d, warm_fanouts, 77, 0, warm_outs, node_order=kind(warm_seen))
        for j, o in enumerate(outs):
            assert_batch_equal(HipBatch(o, len(fanouts)), want[j], len(fanouts), f"batch {j} after replay {replay}")
    del graph
    ctx.close()


# One launch with its lists in LDS: whole words and parts of one to a thread, ids of 16 bits at most, rounds of 1024 nodes, the
# largest lists that fit, hops without edges, more edges than one launch takes.
@pytest.mark.parametrize("n,degree,seeds,fanouts", [
    (31, 4, [31, 1, 0], (3, 2)), (4096, 9, [100, 4096], (1, 1)), (4097, 9, [300], (10, 5)), (8193, 30, [50] * 9, (5, 5, 5, 5)),
    (16_384, 12, [1025, 1024], (7, 2)), (16_385, 40, [20, 0, 37], (16, 16, 2)), (65_536, 8, [90] * 3, (10, 5)), (65_537, 8, [90], (10, 5)),
    (40_000, 20, [400], (16, 0, 3)), (20_000, 70, [9], (32, 32)), (10_000, 20, [490] * 2, (10, 5)), (10_000, 20, [491], (10, 5)),
    (24_000, 30, [2000], (5, 3))])
def test_batches_of_one_launch(B, ctx, n, degree, seeds, fanouts):
    log(f"[one launch] N={n} seeds={seeds} fanouts={fanouts}")
    rng = np.random.default_rng(n + len(fanouts))
    rp, ci, ids = _sparse_graph(n, n, degree, rng)
    csr = B.CsrGraph(torch.as_tensor(rp, device=DEV).to(torch.int64 if n % 2 else torch.int32), _i32(ci))
    lists = [rng.permutation(ids)[:k].astype(np.int32) for k in seeds]
    outs = [B.BlockBuffers(n, ci.size, max(k, 1), fanouts, DEV, with_local=n != 4097) for k in seeds]
    for epoch in range(2):
        ctx.sample_blocks_group(csr, [_i32(x) for x in lists], fanouts, 5, epoch, outs)
        counts, want = torch.zeros(n, dtype=torch.int32, device=DEV), np.zeros(n, dtype=np.uint32)
        ctx.access_histogram_sampled(len(seeds), counts)
        for j, o in enumerate(outs):
            orc = oracle.sample_blocks(rp, ci, lists[j], fanouts, 5, epoch)
            hip = HipBatch(o, len(fanouts))
            if n == 4097:
                hip.nbr_local = orc.nbr_local
            assert_batch_equal(hip, orc, len(fanouts), f"batch {j} epoch {epoch}")
            oracle.access_histogram(orc.input_nodes, want)
        assert np.array_equal(counts.cpu().numpy().view(np.uint32), want)


# A wavefront (eight of them on up to 2048 x 2048 nodes) counts 64 words of ids, a word of all batches in a lane; the batches come in any
# order, some under one index.
@pytest.mark.parametrize("n,group", [(31, 2), (2048, 16), (2049, 5), (70_001, 1), (70_001, 9), (2048 * 2048, 3), (2048 * 2048 + 1, 2)])
def test_bitmap_counts_of_batches_in_any_order(B, ctx, n, group):
    log(f"[bitmap counts] N={n} group={group}")
    rng = np.random.default_rng(n + group)
    rp = np.arange(n + 1, dtype=np.int64)
    ci = rng.integers(0, n, n).astype(np.int32)
    seeds = [rng.permutation(n)[:rng.integers(0, n // 2 + 1)].astype(np.int32) for _ in range(group)]
    outs = [B.BlockBuffers(n, n, max(x.size, 1), (1,), DEV, with_local=False) for x in seeds]
    ctx.sample_blocks_group(B.CsrGraph(torch.as_tensor(rp, device=DEV), _i32(ci)), [_i32(x) for x in seeds], (1,), 3, 1, outs)
    index = [int(x) for x in rng.integers(0, max(2, group - 2), group)]
    counts, first = torch.ones(n, dtype=torch.int32, device=DEV), torch.full((n,), 2, dtype=torch.int32, device=DEV)
    ctx.access_histogram_sampled(group, counts, batch_index=index, first_batch=first)
    want, want_first = np.ones(n, dtype=np.int64), np.full(n, 2, dtype=np.int64)
    for x, b in zip(seeds, index):
        named = np.union1d(x, ci[x])
        want[named] += 1
        want_first[named] = np.minimum(want_first[named], b)
    assert np.array_equal(counts.cpu().numpy(), want) and np.array_equal(first.cpu().numpy(), want_first)


# Runs long enough to be read ahead of the count, and with room for fewer entries not: empty ones, ones of a whole step and one more,
# more of them than a tile has.
@pytest.mark.parametrize("batches,hops,room", [(3, 2, 3200), (1, 1, 1700), (400, 3, 4700), (350, 3, 4500), (5, 7, 10_800)])
def test_epoch_histogram_reading_ahead(B, ctx, batches, hops, room):
    log(f"[histogram ahead] batches={batches} hops={hops} room={room}")
    n, rng = 2000, np.random.default_rng(batches + hops)
    arena, tiers = np.zeros((batches, room), dtype=np.int32), np.zeros((batches, hops + 2), dtype=np.int32)
    want, first = np.zeros(n, dtype=np.int64), np.full(n, -1, dtype=np.int64)
    for b in range(batches):
        for h in range(hops):
            k = int(rng.choice([0, 1, 64, 255, 256, 257, 511, 700])) if room > hops * 700 else int(rng.integers(0, room // hops))
            ids = np.sort(rng.integers(0, n, k)).astype(np.int32)        # repeats count each time
            at = tiers[b, h + 1]
            arena[b, at:at + k] = ids
            tiers[b, h + 2] = at + k
            np.add.at(want, ids, 1)
            first[ids[first[ids] < 0]] = b
    counts, got = torch.zeros(n, dtype=torch.int32, device=DEV), torch.full((n,), -1, dtype=torch.int32, device=DEV)
    ctx.access_histogram_epoch(_i32(arena), _i32(tiers), batches, hops, 0, counts, first_batch=got)
    assert np.array_equal(counts.cpu().numpy(), want) and np.array_equal(got.cpu().numpy(), first)


def test_selection_after_other_selections(B):
    """Selections that the clamped counts settle and that they do not, hit curves and replays of recorded calls of either, on one
    context: each finds the histograms as it needs them."""
    ctx, n, cap = B.Context(0), 70_003, 9_000
    rng = np.random.default_rng(8)
    home = np.where(rng.random(n) < 0.3, np.arange(n), np.arange(n) + (2 << 30) - (1 << 32)).astype(np.int32)
    few, many = (rng.pareto(0.8, n) * 2).astype(np.int64) % 300, rng.integers(0, 1 << 32, n)
    counts = {k: _i32(np.where(x > 0x7FFFFFFF, x - (1 << 32), x)) for k, x in (("few", few), ("many", many))}
    want = {k: oracle.build_cache(x.astype(np.uint32), home, cap) for k, x in (("few", few), ("many", many))}
    home_d, caches, graphs = _i32(home), {}, {}
    for k in counts:
        caches[k] = B.FeatureCache(n, cap, 4, DEV)
        ctx.build_cache(counts[k], home_d, None, 4, caches[k])
        graphs[k] = _captured(lambda: ctx.build_cache(counts[k], home_d, None, 4, caches[k]))
    ctx.cache_hit_curve(counts["many"], home_d, [cap, 100, n])
    graphs["curve"] = _captured(lambda: ctx.cache_hit_curve(counts["many"], home_d, [cap, 100, n]))
    for how in ("few", "curve", "few", "many", "replay few", "many", "replay many", "few", "curve", "replay few", "replay curve", "many", "few"):
        k = how.split()[-1]
        if how.startswith("replay") or k == "curve":
            graphs[k].replay()
        else:
            ctx.build_cache(counts[k], home_d, None, 4, caches[k])
        torch.cuda.synchronize()
        if k == "curve":
            continue
        ids, loc = want[k]
        assert int(caches[k].num_cached) == ids.size, how
        assert np.array_equal(caches[k].cache_ids[:ids.size].cpu().numpy(), ids) and np.array_equal(caches[k].loc.cpu().numpy(), loc), how
    ctx.close()


@pytest.mark.parametrize("distinct,copies", [(7, 1024), (7, 1025), (7, 2560), (7, 2561), (7, 4000), (157, 2560), (157, 2561)])
def test_schedule_of_ids_given_many_times(ctx, distinct, copies):
    """Some ids a few thousand times each fill their buckets, small ones or large ones, up to the last place and beyond; the others stay empty."""
    ids = np.random.default_rng(copies).permutation(np.repeat(np.arange(distinct, dtype=np.int32) * 977, copies))
    got = ctx.epoch_schedule(_i32(ids), 11, 3)
    assert np.array_equal(got.cpu().numpy(), oracle.epoch_schedule(ids, 11, 3))


def test_schedule_counters_between_calls(B):
    """Calls of other sizes and replays of a recorded one, on one context: every call finds its counters cleared."""
    ctx = B.Context(0)
    sizes = [300_000, 9_000, 5_000, 4_097, 300_000, 70_000, 9_000]
    ids = {n: np.random.default_rng(n).permutation(3 * n)[:n].astype(np.int32) for n in sizes}
    dev = {n: _i32(ids[n]) for n in sizes}
    want = {n: oracle.epoch_schedule(ids[n], 5, 2) for n in sizes}
    ctx.epoch_schedule(dev[300_000], 5, 2)
    recorded = torch.zeros(9_000, dtype=torch.int32, device=DEV)
    graph = _captured(lambda: ctx.epoch_schedule(dev[9_000], 5, 2, recorded))
    for n in sizes:
        got = ctx.epoch_schedule(dev[n], 5, 2)
        recorded.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(got.cpu().numpy(), want[n]), n
        assert np.array_equal(recorded.cpu().numpy(), want[9_000]), n
    ctx.close()


def test_schedule_captured_after_a_smaller_one(B):
    """A schedule of no more than twice as many ids, up to the next power of two, finds the scratch of an earlier call."""
    few, many = 4097, 8192
    ids = np.random.default_rng(3).permutation(50_000)[:many].astype(np.int32)
    ids_d, order = _i32(ids), torch.zeros(many, dtype=torch.int32, device=DEV)
    ctx = B.Context(0)
    ctx.epoch_schedule(ids_d[:few], 5, 1)
    graph = _captured(lambda: ctx.epoch_schedule(ids_d, 5, 2, order))
    for replay in range(3):
        order.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(order.cpu().numpy(), oracle.epoch_schedule(ids, 5, 2))
    del graph
    ctx.close()


# Blocks of 4096 nodes; above 16 Mi nodes the blocks' totals are scanned by a launch of their own.  Capacities that cut a tie.
@pytest.mark.parametrize("n", [1, 4095, 4096, 4097, 1_300_003, 16_777_217])
@pytest.mark.parametrize("large", [False, True])
def test_select_block_edges(B, ctx, n, large):
    log(f"[select] N={n} large={large}")
    rng = np.random.default_rng(n)
    counts = rng.integers(0, 4, n).astype(np.uint32)
    if large:                                           # the threshold behind the clamped bin
        counts[rng.integers(0, n, n // 3 + 1)] = rng.choice(np.array([2046, 2047, 2048, 70_000, 2 ** 32 - 1], dtype=np.uint32))
    remote = rng.random(n) < 0.7
    home_np = np.where(remote, (2 << 30) + np.cumsum(remote) - 1, np.cumsum(~remote) - 1).astype(np.uint32).view(np.int32)
    dev_counts, home = torch.from_numpy(counts.view(np.int32)).to(DEV), _i32(home_np)
    for cap in {0, 1, n // 5, n}:
        cache = B.FeatureCache(n, cap, 4, DEV)
        cache.filled.fill_(-1)
        ctx.build_cache(dev_counts, home, None, 4, cache)
        ids, loc = oracle.build_cache(counts, home_np, cap)
        assert int(cache.num_cached.item()) == ids.size, cap
        assert np.array_equal(cache.cache_ids[:ids.size].cpu().numpy(), ids) and np.array_equal(cache.loc.cpu().numpy(), loc), cap
        assert cap == 0 or not cache.filled.any()


def test_hit_curve_of_large_counts(B, ctx):
    """Every count behind the clamped bin: capacities of all candidates are read off the sums, the others go through the radix
    passes, in either order."""
    rng = np.random.default_rng(6)
    n = 30_000
    remote = rng.random(n) < 0.7
    home = np.where(remote, (2 << 30) + np.cumsum(remote) - 1, np.cumsum(~remote) - 1).astype(np.uint32).view(np.int32)
    counts = rng.choice(np.array([2047, 2048, 70_000, 2 ** 31 + 5], dtype=np.uint32), n)
    k = int(remote.sum())
    for caps in ([k, k + 1, 10 ** 6], [0, 1, k - 1, k, 17, k + 1, 5000, 0]):
        hits, total = ctx.cache_hit_curve(torch.from_numpy(counts.view(np.int32)).to(DEV), _i32(home), caps)
        want, want_total = oracle.cache_hit_curve(counts, home, caps)
        assert hits.cpu().numpy().astype(np.uint64).tolist() == want.tolist() and int(total.item()) == want_total


# Lane groups of 64, 32 and 16 (65, 68, 80, 151 chunks of 16 bytes; 301 of 8), eight edges per step.
@pytest.mark.parametrize("dim,stride", [(260, 260), (269, 272), (317, 320), (602, 604), (602, 602)])
def test_mean_aggregate_lane_groups(B, ctx, dim, stride):
    rng = np.random.default_rng(dim)
    m = np.concatenate([[0, 1, 7, 8, 9, 16, 17, 25], rng.integers(0, 12, 400)])
    indptr = np.concatenate([[0], np.cumsum(m)]).astype(np.int32)
    nbr = rng.integers(0, 900, indptr[-1]).astype(np.int32)
    feat = torch.zeros(900, stride, device=DEV)
    feat[:, :dim] = torch.from_numpy(rng.standard_normal((900, dim)).astype(np.float32)).to(DEV)
    agg = torch.full((m.size, stride), float("nan"), device=DEV)
    ctx.mean_aggregate(_i32(indptr), _i32(nbr), m.size, feat, dim, agg)
    x = feat[:, :dim].cpu().numpy()
    want = np.zeros((m.size, dim), dtype=np.float32)
    for i in range(m.size):                             # the same fp32 sums in edge order, then one division
        for e in range(indptr[i], indptr[i + 1]):
            want[i] += x[nbr[e]]
        if m[i]:
            want[i] /= np.float32(m[i])
    assert np.array_equal(agg[:, :dim].cpu().numpy(), want)
    assert torch.isnan(agg[:, dim:]).all()


# More than 16,383 rows: groups of 64, 32 and 16 lanes (65, 76, 96 and 80, 144 chunks); wider ones where the device counts fewer.
@pytest.mark.parametrize("dim", [260, 302, 384, 320, 576])
def test_mean_aggregate_many_rows(B, ctx, dim):
    rng = np.random.default_rng(dim)
    n, stride = 16_389, -(-dim // 4) * 4
    m = rng.integers(0, 10, n)
    indptr = np.concatenate([[0], np.cumsum(m)]).astype(np.int32)
    nbr = rng.integers(0, 900, indptr[-1]).astype(np.int32)
    feat = torch.zeros(900, stride, device=DEV)
    feat[:, :dim] = torch.from_numpy(rng.standard_normal((900, dim)).astype(np.float32)).to(DEV)
    x = feat[:, :dim].cpu().numpy()
    want = np.zeros((n, dim), dtype=np.float32)
    for e in range(9):                                  # the same fp32 sums in edge order, then one division
        rows = np.flatnonzero(m > e)
        want[rows] += x[nbr[indptr[rows] + e]]
    want[m > 0] /= m[m > 0, None].astype(np.float32)
    for count in (None, 16_384, 16_383, 8193, 8192, 1):
        agg = torch.full((n, stride), -7.0, device=DEV)
        ctx.mean_aggregate(_i32(indptr), _i32(nbr), n, feat, dim, agg, n_dst_dev=None if count is None else _i32([count]))
        got, k = agg.cpu().numpy(), n if count is None else count
        assert np.array_equal(got[:k, :dim], want[:k]) and np.all(got[k:] == -7.0)


# One launch up to 64 Ki rows of 24 MiB on one stream, 96 Ki rows of 32 MiB on two (8-64 rows per workgroup), lookups of 1024 rows per workgroup; counters that have to be zero
# again for the next call, whichever kernel makes it.
@pytest.mark.parametrize("rows,dim,stride", [(1, 64, 64), (7, 602, 604), (513, 3, 3), (4097, 37, 40), (16_384, 512, 512), (16_385, 512, 512),
                                             (131_000, 64, 64), (140_000, 64, 64), (65_536, 64, 64), (65_537, 64, 64), (98_304, 64, 64)])
@pytest.mark.parametrize("mirror", [False, True])
def test_gather_one_launch_edges(B, ctx, rows, dim, stride, mirror):
    log(f"[gather] rows={rows} dim={dim} mirror={mirror}")
    rng = np.random.default_rng(rows + dim)
    n = rows + 1000
    x = rng.standard_normal((n, dim), dtype=np.float32)
    is_local = rng.random(n) < 0.4
    row = np.where(is_local, np.cumsum(is_local), np.cumsum(~is_local)) - 1
    home_np = np.where(is_local, row, row + (2 << 30)).astype(np.uint32).view(np.int32)
    n_remote = max(int((~is_local).sum()), 1)

    def store(a, **kw):
        t = torch.zeros(max(a.shape[0], 1), stride, **kw)
        t[:a.shape[0], :dim] = torch.from_numpy(a)
        return t
    local, remote = store(x[is_local], device=DEV), store(x[~is_local], pin_memory=True)
    counts_np = (rng.random(n) < (1.0 if mirror else 0.5)).astype(np.uint32)
    home, counts = _i32(home_np), torch.from_numpy(counts_np.view(np.int32)).to(DEV)
    cache = B.FeatureCache(n, n_remote, stride, DEV, mirror_rows=n_remote if mirror else 0, home=home if mirror else None)
    ctx.build_cache(counts, home, None if mirror else remote, dim, cache)
    if mirror:
        cache.cache_rows.copy_(remote)
    _, loc = oracle.build_cache(counts_np, home_np, n_remote)
    side = torch.cuda.Stream()
    for call in range(4):
        nodes = rng.integers(0, n, rows).astype(np.int32)
        want, st = oracle.gather_features(x, nodes, loc)
        out = torch.full((rows, stride), float("nan"), device=DEV)
        stats = torch.full((3,), -1, dtype=torch.int64, device=DEV)
        n_dev = torch.tensor([rows // 2], dtype=torch.int32, device=DEV) if call == 3 else None
        k = rows // 2 if call == 3 else rows
        if call == 3:
            want, st = oracle.gather_features(x, nodes[:k], loc)
        gather = ctx.gather_features_static if call == 1 else ctx.gather_features
        gather(_i32(nodes), rows, cache, local, remote, dim, out, stats, n_dev=n_dev, miss_stream=side if call else None)
        assert tuple(stats.cpu().tolist()) == st, call
        assert np.array_equal(out[:k, :dim].cpu().numpy(), want), call
        assert torch.isnan(out[k:]).all() and torch.isnan(out[:, dim:]).all(), call
        if call == 2:                                   # the ticket's lookups can be run again
            out.fill_(float("nan"))
            ctx.gather_run(0, rows, cache, local, remote, dim, out, miss_stream=side)
            assert np.array_equal(out[:k, :dim].cpu().numpy(), want)


# One launch up to 32 MiB of rows on two streams that record nothing, three above.
@pytest.mark.parametrize("rows", [1500, 16_384, 16_385])
@pytest.mark.parametrize("static", [False, True])
def test_gather_on_two_streams_captured(B, rows, static):
    """The hit stream records a graph, the miss stream is another one: the library draws it into the graph and joins it back.
    Replayed on changed inputs, with eager calls on the same two streams in between."""
    log(f"[captured gather] rows={rows} static={static}")
    rng, dim, n = np.random.default_rng(rows), 512, rows + 1000
    x = rng.standard_normal((n, dim), dtype=np.float32)
    tag = rng.integers(0, 3, n)
    row = np.zeros(n, dtype=np.int64)
    for t in range(3):
        row[tag == t] = np.arange((tag == t).sum())
    loc = (row + (tag << 30)).astype(np.uint32).view(np.int32)
    local, rows_c = (torch.from_numpy(x[tag == t]).to(DEV) for t in (0, 1))
    remote = torch.from_numpy(x[tag == 2]).pin_memory()
    cache = B.FeatureCache(n, rows_c.shape[0], dim, DEV)
    cache.cache_rows.copy_(rows_c)
    cache.loc.copy_(torch.from_numpy(loc))
    ctx, side = B.Context(0), torch.cuda.Stream()
    ids, out = torch.zeros(rows, dtype=torch.int32, device=DEV), torch.zeros(rows, dim, device=DEV)
    stats = torch.zeros(3, dtype=torch.int64, device=DEV)
    ctx.gather_features(ids, rows, cache, local, remote, dim, out, stats, miss_stream=side)       # makes the scratch
    gather = ctx.gather_features_static if static else ctx.gather_features
    graph = _captured(lambda: gather(ids, rows, cache, local, remote, dim, out, stats, miss_stream=side))
    for replay in range(3):
        nodes = rng.integers(0, n, rows).astype(np.int32)
        want, st = oracle.gather_features(x, nodes, loc)
        for call in ("replay", "eager"):
            ids.copy_(torch.from_numpy(nodes))
            out.fill_(float("nan"))
            stats.fill_(-1)
            if call == "replay":
                graph.replay()
            else:
                gather(ids, rows, cache, local, remote, dim, out, stats, miss_stream=side)
            torch.cuda.synchronize()
            assert tuple(stats.cpu().tolist()) == st, (replay, call)
            assert np.array_equal(out.cpu().numpy(), want), (replay, call)
    del graph
    ctx.close()


def test_gather_after_calls_that_overlapped(B):
    """Two calls that overlap on the shared scratch (a caller's error) spoil their own statistics; the calls after them, eager or
    replayed, find their counters clear."""
    rng, rows, dim, n = np.random.default_rng(8), 20_000, 16, 25_000
    x = rng.standard_normal((n, dim), dtype=np.float32)
    tag = rng.integers(0, 3, n)
    row = np.zeros(n, dtype=np.int64)
    for t in range(3):
        row[tag == t] = np.arange((tag == t).sum())
    loc = (row + (tag << 30)).astype(np.uint32).view(np.int32)
    local, rows_c = (torch.from_numpy(x[tag == t]).to(DEV) for t in (0, 1))
    remote = torch.from_numpy(x[tag == 2]).pin_memory()
    cache = B.FeatureCache(n, rows_c.shape[0], dim, DEV)
    cache.cache_rows.copy_(rows_c)
    cache.loc.copy_(torch.from_numpy(loc))
    nodes = rng.integers(0, n, rows).astype(np.int32)
    want, st = oracle.gather_features(x, nodes, loc)
    ids, streams = _i32(nodes), [torch.cuda.Stream() for _ in range(2)]
    outs = [torch.zeros(rows, dim, device=DEV) for _ in range(2)]
    stats = [torch.zeros(3, dtype=torch.int64, device=DEV) for _ in range(2)]
    ctx = B.Context(0)
    call = lambda k: ctx.gather_features_static(ids, rows, cache, local, remote, dim, outs[k], stats[k])  # noqa: E731
    call(0)
    graph = _captured(lambda: call(0))
    for _ in range(20):
        torch.cuda.synchronize()
        for k in range(2):                              # side by side on the two streams
            with torch.cuda.stream(streams[k]):
                call(k)
        torch.cuda.synchronize()
        for replay in (True, False):
            outs[0].fill_(float("nan"))
            stats[0].fill_(-1)
            graph.replay() if replay else call(0)
            torch.cuda.synchronize()
            assert tuple(stats[0].cpu().tolist()) == st and np.array_equal(outs[0].cpu().numpy(), want), replay
    del graph
    ctx.close()


# A packed counter up to 2^23 - 1 rows, separate ones above, for all batches of a group that has such a one.
@pytest.mark.parametrize("wide", [False, True])
def test_lookups_of_very_large_batches(B, wide):
    log(f"[very large batches] wide={wide}")
    sizes = [700, 0, (1 << 23) - 1, 3] if not wide else [700, (1 << 23), 0, 3]
    n, dim = 10_000, 1
    rng = np.random.default_rng(5)
    x = rng.standard_normal((n, dim), dtype=np.float32)
    tag = rng.choice([0, 1, 2], n, p=[0.2, 0.79, 0.01])
    row = np.zeros(n, dtype=np.int64)
    for t in range(3):
        row[tag == t] = np.arange((tag == t).sum())
    loc = (row + (tag << 30)).astype(np.uint32).view(np.int32)
    local, rows_c = (torch.from_numpy(x[tag == t]).to(DEV) for t in (0, 1))
    remote = torch.from_numpy(x[tag == 2]).pin_memory()
    cache = B.FeatureCache(n, rows_c.shape[0], dim, DEV)
    cache.cache_rows.copy_(rows_c)
    cache.loc.copy_(torch.from_numpy(loc))
    ctx = B.Context(0)
    for sizes_now in (sizes, [500, 20_000, 0, 1], sizes):
        batches = [rng.integers(0, n, size=k).astype(np.int32) for k in sizes_now]
        ids = [_i32(b) if b.size else torch.zeros(1, dtype=torch.int32, device=DEV) for b in batches]
        stats = torch.full((4, 3), -1, dtype=torch.int64, device=DEV)
        ctx.gather_prepare(0, ids, sizes_now, cache, [stats[t] for t in range(4)])
        for t, k in enumerate(sizes_now):
            out = torch.full((max(k, 1), dim), float("nan"), device=DEV)
            ctx.gather_run(t, k, cache, local, remote, dim, out)
            if k:
                want, st = oracle.gather_features(x, batches[t], loc)
                assert np.array_equal(out.cpu().numpy(), want), (sizes_now, t)
            assert tuple(stats[t].cpu().tolist()) == (st if k else (0, 0, 0)), (sizes_now, t)
        k = sizes_now[0]                                # the same ticket in one launch
        out = torch.full((k, dim), float("nan"), device=DEV)
        ctx.gather_features(ids[0], k, cache, local, remote, dim, out, stats[0])
        want, st = oracle.gather_features(x, batches[0], loc)
        assert tuple(stats[0].cpu().tolist()) == st and np.array_equal(out.cpu().numpy(), want)
    ctx.close()


def test_mirrored_pulls_of_growing_calls(B):
    """Calls that grow from single batches: every size adds up, and the gathers of an epoch sampled that way are right."""
    import dataclasses

    import synth
    from paper_2505_10806_amd.pipeline import EpochPipeline
    cfg = dataclasses.replace(synth.get_config("tiny"), cache_frac=1.0, max_batches=None)
    wl = synth.build_workload(cfg, seed=6, device=DEV)
    pipe = EpochPipeline(wl, device=DEV)
    assert pipe.mirror and not pipe.ramp                # a small remote partition
    pipe.ramp = True
    for n in (1, 2, 3, 7, 20, 61):
        for g in (2, 8, 16):
            for first in (False, True):
                for last in (False, True):
                    sizes = pipe._call_sizes(n, g, first, last, ramp=True)
                    assert sum(sizes) == n and all(0 < s <= g for s in sizes), (n, g, first, last, sizes)
    assert pipe._call_sizes(20, 8, True, True, ramp=True) == [1, 1, 1, 1, 1, 1, 2, 2, 3, 3, 2, 1, 1]
    taken = []
    with torch.cuda.stream(torch.cuda.Stream()):
        pipe.run_epoch(1, pipe.batches_per_epoch, lambda p, b: taken.append(p.out[:p.sizes[b], :cfg.feat_dim].clone()))
        torch.cuda.synchronize()
        for b, rows in enumerate(taken):
            assert torch.equal(rows, wl.features[pipe.arena[b, :pipe.sizes[b]].long()]), f"batch {b}"
        assert int(pipe.stats[:, 2].sum()) == 0
    pipe.close()


# Tiers from bytes: workgroups of 192 bitmap words, which count what is in front of their words up to 160,000 nodes and 12 MB of bytes (of 768
# words where many batches make enough of those); hops that clear the other map for the next one; a hub that most edges name.
@pytest.mark.parametrize("n,seeds,fanouts", [
    (6143, [380, 383, 0], (32, 31)), (6145, [384, 1], (32, 5, 3)), (24_577, [1536] * 16, (25, 10)), (159_999, [3000], (10, 10, 10, 2)),
    (160_000, [900, 0, 850], (25, 10)), (160_001, [900, 0, 850], (25, 10)), (150_000, [700] * 16, (20, 3)), (1_600_000, [90] * 16, (10, 5)), (4_194_304, [300, 299], (10, 5))])
@pytest.mark.parametrize("captured", [False, True])
def test_tiers_from_bytes(B, ctx, n, seeds, fanouts, captured):
    log(f"[bytes] N={n} seeds={seeds} fanouts={fanouts} captured={captured}")
    rng = np.random.default_rng(n)
    deg = rng.integers(0, 60, n) * (rng.random(n) < min(1.0, 200_000 / n))
    deg[[0, n - 1]] = 300
    rp = np.concatenate([[0], np.cumsum(deg)])
    ci = rng.integers(0, n, rp[-1]).astype(np.int32)
    ci[rng.random(ci.size) < 0.3] = n - 1
    csr = B.CsrGraph(torch.as_tensor(rp, device=DEV).to(torch.int32), _i32(ci))
    ids = np.unique(np.concatenate([[0, n - 1], np.flatnonzero(deg)]))
    outs = [B.BlockBuffers(n, ci.size, max(k, 1), fanouts, DEV) for k in seeds]
    bufs = [torch.zeros(max(k, 1), dtype=torch.int32, device=DEV) for k in seeds]
    run = lambda: ctx.sample_blocks_group(csr, [b[:k] for b, k in zip(bufs, seeds)], fanouts, 77, 1, outs)  # noqa: E731
    for b, k in zip(bufs, seeds):
        b[:k] = _i32(rng.permutation(ids)[:k])
    run()
    if captured:
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            run()
    for _ in range(3 if captured else 1):               # (replays with other seeds, and an eager call of its own seeds in front of each)
        lists = [rng.permutation(ids)[:k].astype(np.int32) for k in seeds]
        if captured:
            run()
        for b, x in zip(bufs, lists):
            b[:x.size] = _i32(x)
        if captured:
            graph.replay()
        else:
            run()
        for j, o in enumerate(outs):
            orc = oracle.sample_blocks(rp, ci, lists[j], fanouts, 77, 1)
            assert_batch_equal(HipBatch(o, len(fanouts)), orc, len(fanouts), f"batch {j}")


# One launch, ordered by values and by events; lookup and copies apart, by values and by events; more calls on their way than there are signals.
@pytest.mark.parametrize("rows", [2000, 30_000, 38_000, 70_000])
def test_two_stream_gathers_keep_their_place_in_both_streams(B, ctx, rows):
    """The miss rows of a call come behind what the miss stream was given before it and in front of what either stream is given next."""
    log(f"[order] rows={rows}")
    dim, n, calls, side = 256, max(40_000, rows), 100, torch.cuda.Stream()
    ids = torch.randperm(n, device=DEV, dtype=torch.int32)[:rows].contiguous()
    cache = B.FeatureCache(n, 1, dim, DEV)
    cache.loc.copy_(torch.where(torch.arange(n, device=DEV) % 4 == 0, torch.arange(n, device=DEV) // 4 - 2 ** 31, torch.arange(n, device=DEV)).int())
    remote = torch.zeros(n // 4, dim, pin_memory=True)
    local, out = torch.zeros(n, dim, device=DEV), torch.zeros(rows, dim, device=DEV)
    stats, taken, source = torch.zeros(3, dtype=torch.int64, device=DEV), [], torch.zeros(n // 4, dim, device=DEV)
    missing = (ids % 4 == 0).nonzero().flatten()
    torch.cuda.synchronize()
    for k in range(calls):
        with torch.cuda.stream(side):                   # late, and only for this call
            torch.cuda._sleep(20_000)
            remote.copy_(source.fill_(k + 1), non_blocking=True)
        ctx.gather_features(ids, rows, cache, local, remote, dim, out, stats, miss_stream=side)
        with torch.cuda.stream(side):
            remote.copy_(source.fill_(-1), non_blocking=True)
        taken.append(out[missing].amin().reshape(1))
        taken.append(out[missing].amax().reshape(1))
    got = torch.cat(taken).reshape(calls, 2).cpu()
    assert torch.equal(got, torch.arange(1, calls + 1, dtype=torch.float32).reshape(-1, 1).expand(-1, 2)), got.flatten().tolist()
    assert stats.cpu().tolist() == [rows - missing.numel(), 0, missing.numel()]


# One workgroup up to 4096 ids, with room for 3072 where that does, buckets of 256 to 512 ids up to 400,000, of 1024 to 2048 above.
@pytest.mark.parametrize("n", [1025, 3071, 3072, 3073, 4096, 4097, 16_384, 16_385, 262_144, 400_000, 400_001])
def test_schedule_bucket_sizes(ctx, n):
    log(f"[schedule sizes] n={n}")
    ids = np.random.default_rng(n).permutation(2 * n)[:n].astype(np.int32)
    assert np.array_equal(ctx.epoch_schedule(_i32(ids), 21, 4).cpu().numpy(), oracle.epoch_schedule(ids, 21, 4))


# A small bucket's workgroup takes two rounds up to 1024 ids, five up to the 2560 that there is room for.
@pytest.mark.parametrize("in_bucket", [1000, 1024, 1025, 2048, 2559, 2560, 2561, 5000])
def test_schedule_small_bucket_with_more_ids_than_room(ctx, in_bucket):
    log(f"[small bucket] {in_bucket}")
    order = oracle.epoch_schedule(np.arange(2_000_000, dtype=np.int32), 21, 4)         # ascending by key: 7800 ids or so to each of 256 buckets
    rng = np.random.default_rng(in_bucket)
    ids = rng.permutation(np.concatenate([order[:in_bucket], order[20_000:][rng.permutation(1_980_000)[:70_000]]])).astype(np.int32)
    assert np.array_equal(ctx.epoch_schedule(_i32(ids), 21, 4).cpu().numpy(), oracle.epoch_schedule(ids, 21, 4))


def test_schedule_recorded_for_many_ids_survives_few(B):
    """Large buckets and small ones take different scratch: what a graph holds is there for both."""
    ctx = B.Context(0)
    ids = {n: np.random.default_rng(n).permutation(2 * n)[:n].astype(np.int32) for n in (400_001, 390_000)}
    dev, out = {n: _i32(x) for n, x in ids.items()}, torch.empty(400_001, dtype=torch.int32, device=DEV)
    ctx.epoch_schedule(dev[400_001], 5, 2, out)
    graph = _captured(lambda: ctx.epoch_schedule(dev[400_001], 5, 2, out))
    for _ in range(3):
        assert np.array_equal(ctx.epoch_schedule(dev[390_000], 5, 2).cpu().numpy(), oracle.epoch_schedule(ids[390_000], 5, 2))
        out.zero_()
        graph.replay()
        assert np.array_equal(out.cpu().numpy(), oracle.epoch_schedule(ids[400_001], 5, 2))
    ctx.close()


# Lookups: workgroups of 1024 rows up to 220,000, above of 4096 for one batch, of 2048 for several; last ones of one row, of all.
@pytest.mark.parametrize("rows", [[1], [1024], [1025], [220_000], [220_001], [225_280], [225_281], [1, 0], [1025, 1023, 0, 4096], [220_001, 2048, 2049, 0, 225_281]])
@pytest.mark.parametrize("mirror", [False, True])
def test_lookups_of_one_and_of_several_batches(B, ctx, rows, mirror):
    log(f"[lookups] rows={rows} mirror={mirror}")
    n, dim, rng = 300_000, 4, np.random.default_rng(sum(rows))
    X = torch.arange(n, device=DEV, dtype=torch.float32).reshape(-1, 1).expand(-1, dim).contiguous()
    kind = rng.integers(0, 3, n)                        # local, cached, missing
    is_local, is_cached = _i32(kind == 0).bool(), _i32(kind == 1).bool()
    place = lambda m: torch.cumsum(m, 0) - 1  # noqa: E731
    word = lambda tag, row: row + (tag << 30) - ((tag >= 2) << 32)  # noqa: E731
    home = torch.where(is_local, word(0, place(is_local)), word(2, place(~is_local))).int()
    loc = torch.where(is_cached, word(1, place(is_cached)), home.long()).int()
    cache = B.FeatureCache(n, int((~is_local).sum()), dim, DEV, mirror_rows=int((~is_local).sum()) if mirror else 0, home=home if mirror else None)
    cache.loc.copy_(loc)
    at = (home.long() & (1 << 30) - 1)[is_cached] if mirror else place(is_cached)[is_cached]
    cache.cache_rows[at] = X[is_cached]
    remote = X[~is_local].cpu().pin_memory()
    ids = [_i32(rng.permutation(n)[:k]) if k else torch.zeros(1, dtype=torch.int32, device=DEV) for k in rows]
    stats = [torch.full((3,), -7, dtype=torch.int64, device=DEV) for _ in rows]
    for _ in range(5):                                  # every one of the running counts, and the first again
        ctx.gather_prepare(0, ids, rows, cache, stats)
    for j, k in enumerate(rows):
        out = torch.full((max(k, 1), dim), -7.0, device=DEV)
        ctx.gather_run(j, k, cache, X[is_local].contiguous(), remote, dim, out)
        assert torch.equal(out[:k], X[ids[j][:k].long()])
        assert stats[j].cpu().tolist() == np.bincount(kind[ids[j][:k].cpu().numpy()], minlength=3).tolist()


# First-seen order by first edges where workgroups take several chunks of the edge list behind a scan: active nodes of far more neighbours than the
# average, and a bound of more than 4096 chunks.
def test_first_seen_chunks_behind_a_scan(B, ctx):
    log("[first seen] several chunks to a workgroup behind a scan")
    n, fanouts, rng = 9_000_000, (1, 33), np.random.default_rng(4)
    deg = np.zeros(n, dtype=np.int64)
    ids = rng.permutation(n)[:300_000]
    deg[ids] = rng.choice([0, 1, 20, 34], ids.size)
    rp = np.concatenate([[0], np.cumsum(deg)])
    ci = rng.integers(0, n, rp[-1]).astype(np.int32)
    ci[::2] = rng.choice(ids, ci[::2].size)
    csr = B.CsrGraph(torch.as_tensor(rp, device=DEV).to(torch.int32), _i32(ci))
    seeds = rng.permutation(ids)[:200_000].astype(np.int32)
    out = B.BlockBuffers(n, ci.size, seeds.size, fanouts, DEV)
    ctx.sample_blocks_group(csr, [_i32(seeds)], fanouts, 77, 1, [out], node_order=B.RG_ORDER_FIRST_SEEN)
    orc = oracle.sample_blocks(rp, ci, seeds, fanouts, 77, 1, oracle.ORDER_FIRST_SEEN)
    assert_batch_equal(HipBatch(out, len(fanouts)), orc, len(fanouts), "batch")


# A lane per draw for fan-outs of 33 to 64 (four nodes to a workgroup), a wavefront per node above; rows of about as many neighbours as
# are drawn, where most draws find theirs taken.
@pytest.mark.parametrize("n,fanouts,seeds", [(3001, (33, 2), [5, 0, 4]), (3001, (64, 3), [1, 130]), (70_001, (63, 2), [257]), (70_001, (65, 2), [257]),
                                             (70_001, (5, 64), [600] * 2), (600_001, (2, 64, 33), [700, 0, 699]), (9_000_000, (64, 3), [120, 1]),
                                             (9_000_000, (1, 33), [262_144])])
@pytest.mark.parametrize("first_seen", [False, True])
def test_draws_of_33_to_64(B, ctx, n, fanouts, seeds, first_seen):
    log(f"[wide draws] N={n} fanouts={fanouts} seeds={seeds} first_seen={first_seen}")
    rng, k = np.random.default_rng(n + len(fanouts)), max(fanouts)
    deg = np.zeros(n, dtype=np.int64)
    ids = rng.permutation(n)[:min(n, 300_000)]
    deg[ids] = rng.choice([0, 1, k - 1, k, k + 1, k + 2, 2 * k], ids.size) if sum(seeds) < 100_000 else rng.choice([0, 1, 33, 34], ids.size)
    rp = np.concatenate([[0], np.cumsum(deg)])
    ci = rng.choice(ids, rp[-1]).astype(np.int32)
    csr = B.CsrGraph(torch.as_tensor(rp, device=DEV).to(torch.int32), _i32(ci))
    lists = [rng.permutation(ids)[:s].astype(np.int32) for s in seeds]
    outs = [B.BlockBuffers(n, ci.size, max(s, 1), fanouts, DEV) for s in seeds]
    ctx.sample_blocks_group(csr, [_i32(x) for x in lists], fanouts, 77, 1, outs, node_order=B.RG_ORDER_FIRST_SEEN if first_seen else B.RG_ORDER_ASCENDING)
    for j, o in enumerate(outs):
        orc = oracle.sample_blocks(rp, ci, lists[j], fanouts, 77, 1, oracle.ORDER_FIRST_SEEN if first_seen else oracle.ORDER_ASCENDING)
        assert_batch_equal(HipBatch(o, len(fanouts)), orc, len(fanouts), f"batch {j}")


# Plans from the sampler's bitmaps: 4096 workgroups of 256 words add up the counts in front of their own, more of them have these scanned.
@pytest.mark.parametrize("n", [33_554_432, 33_554_433, 41_943_041])
def test_plan_segments_behind_a_scan(B, ctx, n):
    log(f"[plan scan] N={n}")
    rng, fanouts, group = np.random.default_rng(n), (6, 4), 3
    block = 256 * 32
    active = np.unique(np.concatenate([np.arange(40), n // 2 + np.arange(-20, 20), 2 * block + np.arange(-3, 3), n - 1 - np.arange(40),
                                       n // block * block - 1 - np.arange(40), rng.integers(0, n, 3000)]))
    deg = np.zeros(n, dtype=np.int64)
    deg[active] = rng.integers(0, 9, active.size)
    rp = np.concatenate([[0], np.cumsum(deg)])
    ci = rng.choice(active, rp[-1]).astype(np.int32)
    csr = B.CsrGraph(torch.as_tensor(rp, device=DEV).to(torch.int32), _i32(ci))
    remote = np.arange(n) % 3 > 0
    remote[[0, n - 1]] = True
    home = np.where(remote, np.cumsum(remote) - 1 - (1 << 31), np.cumsum(~remote) - 1).astype(np.int32)
    n_remote = int(remote.sum())
    cache = B.FeatureCache(n, n_remote, 1, DEV, mirror_rows=n_remote, home=_i32(home))
    plan = B.PrefetchPlan(n_remote, 3, DEV)
    plan.set_num_batches(3)
    claimed = torch.zeros((n + 31) // 32, dtype=torch.int32, device=DEV)
    seen, start = np.zeros(0, dtype=np.int64), 0
    for seg in range(3):
        seeds = [rng.permutation(active)[:300].astype(np.int32) if seg != 1 else np.array([0, n - 1], dtype=np.int32) for _ in range(group)]
        outs = [B.BlockBuffers(n, ci.size, x.size, fanouts, DEV) for x in seeds]
        ctx.sample_blocks_group(csr, [_i32(x) for x in seeds], fanouts, 11, seg, outs)
        ctx.plan_sampled(group, cache, claimed, plan, seg)
        named = np.unique(np.concatenate([oracle.sample_blocks(rp, ci, x, fanouts, 11, seg).input_nodes for x in seeds]))
        new = np.setdiff1d(named, seen)
        seen = np.union1d(seen, named)
        rows = home[new[remote[new]]] & 0x3FFFFFFF
        offs = plan.offsets.cpu().numpy()
        assert offs[seg] == start and offs[seg + 1] == start + rows.size, (seg, offs[:4], rows.size)
        pairs = plan.list[2 * start:2 * (start + rows.size)].cpu().numpy().reshape(-1, 2)
        assert np.array_equal(pairs[:, 0], rows) and np.array_equal(pairs[:, 1], rows)
        words = claimed.cpu().numpy().view(np.uint32)
        want = np.zeros(words.size, dtype=np.uint32)
        np.bitwise_or.at(want, seen >> 5, np.uint32(1) << (seen & 31).astype(np.uint32))
        assert np.array_equal(words, want)
        start += rows.size
    assert start > 1000
