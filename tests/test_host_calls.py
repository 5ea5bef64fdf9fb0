"""What the library's host code asks of the HIP runtime, call by call, without a GPU: order of streams, scratch, choice of kernels."""
import pytest

import host_calls


# One launch up to 32 MiB of rows (24 on one stream), more above.
@pytest.mark.parametrize("rows", [1500, 16_384, 16_385])
@pytest.mark.parametrize("static", [False, True])
def test_two_stream_gather_stays_inside_the_graph_it_is_recorded_into(rows, static):
    """The hit stream records a graph: it waits for nothing outside the graph, and the miss stream, which the library draws into
    the graph, is joined back."""
    host_calls.run(f"""
c = context()
assert gather(c, {rows}, 512, hit=0x51, miss=0x52, static={static}) == OK
eager = kernels()
rt.begin_capture(0x51)
assert gather(c, {rows}, 512, hit=0x51, miss=0x52, static={static}) == OK, lib.rg_last_error(c)
assert rt.end_capture() == 0
assert [k.split("<")[0] for k in kernels()] == ["k_clear_counters", "k_classify", "k_gather_hbm", "k_gather_miss"]
assert (len(eager) == 1) == ({rows} <= 16384), eager
assert gather(c, {rows}, 512, hit=0x51, static={static}) == OK
eager = kernels()
rt.begin_capture(0x51)
assert gather(c, {rows}, 512, hit=0x51, static={static}) == OK
assert rt.end_capture() == 0 and kernels() == ["k_clear_counters"] + eager         # a replay starts from clear counters
""")


# (nodes, edges, seeds, fan-outs, order) of a call that may have been captured, then of one that needs no more of what every call
# uses (members, positions, frontier): another order, more hops, more edges per hop, another number of slices, fewer but larger batches.
_CALLS = {
    "order": [(300_007, 9_000_000, [13_000] * 2, (5, 3), "FIRST_SEEN"), (300_007, 9_000_000, [1500] * 2, (25, 10), "ASCENDING"),
              (300_007, 9_000_000, [1500] * 2, (25, 10), "FIRST_SEEN"), (300_007, 9_000_000, [1500] * 2, (25, 10), "ASCENDING")],
    "hops": [(300_007, 9_000_000, [2000] * 4, (25, 10), "ASCENDING"), (300_007, 9_000_000, [200] * 4, (10, 3, 2, 2), "ASCENDING"),
             (300_007, 9_000_000, [50] * 4, (10, 3, 2, 2, 1, 1), "ASCENDING")],
    "edges": [(200_000, 9_000_000, [2000] * 4, (25, 10), "ASCENDING"), (200_000, 9_000_000, [2000] * 4, (25, 13), "FIRST_SEEN")],
    "slices": [(1_300_000, 9_000_000, [2000] * 2, (25, 10), "ASCENDING"), (1_270_000, 9_000_000, [2000] * 2, (25, 10), "ASCENDING")],
    "group": [(100_000, 9_000_000, [3000] * 8, (25, 10), "ASCENDING"), (700_000, 9_000_000, [2000], (25, 10), "ASCENDING")],
    "reserved": [(300_007, 9_000_000, [600] * 8, (25, 5), "FIRST_SEEN"), (300_007, 9_000_000, [900] * 8, (25, 5), "FIRST_SEEN")],
    "small": [(131_000, 9_000_000, [300] * 8, (10, 5), "ASCENDING"), (131_000, 9_000_000, [300] * 8, (10, 5), "FIRST_SEEN"),
              (131_000, 9_000_000, [400] * 2, (10, 5), "ASCENDING")],
}


@pytest.mark.parametrize("name", list(_CALLS))
@pytest.mark.parametrize("captured", [False, True])
def test_sampler_scratch_outlives_calls_of_another_kind(name, captured):
    """A graph holds the addresses of the scratch it was recorded with: calls that are no larger than the earlier ones free none."""
    calls = ", ".join(f"({n}, {e}, {s}, {f}, {o})" for n, e, s, f, o in _CALLS[name])
    host_calls.run(f"""
c, calls = context(), [{calls}]
if "{name}" == "reserved":
    assert lib.rg_reserve(c, i64(300_007), i64(300_007), i64(0), i32(8)) == OK
assert sample(c, *calls[0]) == OK
if {captured}:                                            # what the second call records into a graph is there to stay
    rt.begin_capture(0x51)
    if sample(c, *calls[-1], stream=0x51) != OK:
        assert any("in a graph" in x for x in log()), lib.rg_last_error(c)      # the call wants more than there is
    rt.end_capture()
for call in calls + calls:
    assert sample(c, *call) == OK, lib.rg_last_error(c)
    assert not log("free"), call
""")


def test_histogram_scratch_outlives_larger_calls():
    """A graph that holds the address of the histogram's scratch is safe whatever is counted later: outgrown scratch stays."""
    host_calls.run("""
c = context()
assert histogram(c, 100_000, 100, 2) == OK
log()
rt.begin_capture(0x51)
assert histogram(c, 100_000, 100, 2, stream=0x51) == OK
rt.end_capture()
for n, batches, hops in ((100_000, 300, 2), (100_000, 5000, 3), (10_000_000, 245, 3), (1 << 30, 3, 8), (1 << 30, 300, 8)):
    assert histogram(c, n, batches, hops) == OK and not log("free"), n
assert lib.rg_reserve(c, i64(1 << 20), i64(100), i64(100), i32(2)) == OK
assert not log("free")
assert rt.memory_held() < 200 << 20
lib.rg_destroy(c)
assert rt.memory_held() == 0
c = context()                                             # rg_reserve makes room for any histogram of such a graph
assert lib.rg_reserve(c, i64(3_000_000), i64(100), i64(100), i32(1)) == OK
log()
for batches, hops in ((5, 8), (64, 8), (2000, 8), (2000, 1)):
    assert histogram(c, 3_000_000, batches, hops) == OK and not log("malloc"), batches
d = context()                                             # none there, and none to be had while the graph is recorded
log()
rt.begin_capture(0x51)
assert histogram(d, 10_000_000, 245, 3, stream=0x51) == OK
rt.end_capture()
assert [k.split("<")[0] for k in kernels()] == ["k_histogram_seeds", "k_histogram_runs"]
e = context()                                             # some there: as many batches to a launch as fit, if that pays
assert histogram(e, 10_000_000, 60, 3) == OK
log()
rt.begin_capture(0x51)
assert histogram(e, 10_000_000, 180, 3, stream=0x51) == OK
rt.end_capture()
assert [k.split("<")[0] for k in kernels()] == ["k_histogram_seeds"] + 3 * ["k_hist_bounds", "k_histogram_runs"]
f = context()                                             # room for half of the batches: more room, where none was reserved
assert histogram(f, 300_000, 130, 1) == OK
log()
assert histogram(f, 300_000, 260, 1) == OK
assert [k.split("<")[0] for k in kernels()] == ["k_histogram_seeds", "k_hist_bounds", "k_histogram_runs"]
""")


# No more ranges than 136 or sqrt(4.4 entries) of a run, of 512 to 8192 ids; whole rounds of the device where the runs are long.
@pytest.mark.parametrize("n,stride,ranges", [(1000, 1 << 24, 2), (20_000, 3, 40), (334_000, 3, 136), (334_000, 3000, 136), (334_000, 30_000, 363), (334_000, 300_000, 512),
                                             (10_000_000, 30_000, 1221), (10_000_000, 1 << 24, 1536)])
def test_histogram_ranges(n, stride, ranges):
    host_calls.run(f"""
c = context()
assert histogram(c, {n}, 60, 1, stride={stride}) == OK
assert [int(x.split()[2]) for x in log("launch k_histogram_runs")] == [{ranges}]
""")


# Few or short runs; the most batches that one launch's scratch holds (28 on 200 M nodes), two launches, more than two.
@pytest.mark.parametrize("n,batches,hops,stride,search,launches", [
    (1000, 5, 2, 1 << 24, True, 1), (300_000, 100, 2, 1000, True, 1), (1 << 20, 25, 1, 30_000, True, 1), (1 << 20, 26, 1, 30_000, False, 1),
    (1 << 22, 17, 1, 30_000, True, 1), (1 << 22, 18, 1, 30_000, False, 1), (10_000_000, 122, 1, 64, True, 1), (10_000_000, 123, 1, 64, False, 1),
    (10_000_000, 1, 1, 65, False, 1), (10_000_000, 454, 3, 1 << 24, False, 1), (10_000_000, 2000, 3, 1 << 24, False, 5),
    (200_000_000, 28, 3, 1 << 24, False, 1), (200_000_000, 56, 3, 1 << 24, False, 2), (200_000_000, 57, 3, 1 << 24, True, 1),
    (1 << 30, 1, 8, 1 << 24, False, 1), (1 << 30, 245, 8, 1 << 24, True, 1)])
def test_histogram_searches_where_bounds_do_not_pay(n, batches, hops, stride, search, launches):
    host_calls.run(f"""
c = context()
assert histogram(c, {n}, {batches}, {hops}, stride={stride}) == OK
names = [k.split("<")[0] for k in kernels()]
assert names.count("k_histogram_runs") == {launches}, names
assert names.count("k_hist_bounds") == (0 if {search} else {launches}), names
""")


def test_reserve_and_sampler_without_memory_for_what_they_can_do_without():
    """Rank words, slices' bitmaps and range bounds that cannot be allocated: rg_reserve succeeds all the same, gives back what it
    got of them, and the calls behind it neither ask again nor wait for the device."""
    host_calls.run("""
N, FRONTIER, GROUP, FANOUTS = 10_000_000, 4_000_000, 8, (15, 10, 5)
RANK, MARKS = 8 * GROUP * (N // 32) * 8, 256 * 40_000 * 4
reserve = lambda c: lib.rg_reserve(c, i64(N), i64(FRONTIER), i64(1000), i32(GROUP))
call = lambda c, **kw: sample(c, N, 500_000_000, [2000] * GROUP, FANOUTS, **kw)
full = context()
assert reserve(full) == OK
total = rt.memory_held()
lib.rg_destroy(full)
assert rt.memory_held() == 0
for short in (1, RANK // 2, RANK, RANK + MARKS // 2):     # the bounds, the rank words, the bitmaps cannot be had
    rt.limit_memory(total - short)
    c = context()
    assert reserve(c) == OK, lib.rg_last_error(c)
    sliced = short < RANK // 2
    assert rt.memory_held() < total - (0 if sliced else RANK + MARKS), (short, rt.memory_held())
    rt.limit_memory(rt.memory_held())
    log()
    for _ in range(2):
        assert call(c) == OK and histogram(c, N, 20, 3) == OK
        lines = log()
        assert all(x.startswith("launch") for x in lines), lines
        assert any("k_slice_emit" in x for x in lines) == sliced
        assert any("k_tier_emit" in x for x in lines) == (not sliced)
    rt.limit_memory(1 << 40)
    assert reserve(c) == OK and call(c) == OK and "k_slice_mark" in kernels()
    lib.rg_destroy(c)
# without rg_reserve: one failed try, then none until less is wanted
rt.limit_memory(1 << 40)
c = context()
assert call(c) == OK
base = rt.memory_held()
lib.rg_destroy(c)
rt.limit_memory(base - RANK // 4)
c = context()
log()
assert call(c) == OK
first = log()
assert any(x.startswith("no memory") for x in first) and any("k_tier_emit" in x for x in first)
assert call(c) == OK and all(x.startswith("launch") for x in log())
""")


@pytest.mark.parametrize("n,edges,seeds,fanouts,small", [
    (131_072, 9_000_000, [315], (10, 5), True), (131_072, 9_000_000, [316], (10, 5), False), (131_073, 9_000_000, [126], (10, 5), True),
    (131_073, 9_000_000, [127], (10, 5), False), (524_289, 9_000_000, [10], (10, 5), False), (10_000, 9_000_000, [10], (33,), False),
    (131_072, 9_000_000, [20_480], (0,), True), (131_072, 9_000_000, [20_481], (0,), False),            # frontiers without edges
    (500_000, 9_000_000, [2048] * 2, (0, 1, 1), True), (500_000, 9_000_000, [2049] * 2, (0, 1, 1), False), (500_000, 4000, [500_000], (5,), False)])
def test_batches_that_one_launch_takes(n, edges, seeds, fanouts, small):
    host_calls.run(f"""
c = context()
assert sample(c, {n}, {edges}, {seeds}, {fanouts}) == OK, lib.rg_last_error(c)
names = kernels()
assert ([k.split("<")[0] for k in names] == ["k_sample_small"]) == {small}, names
""")


@pytest.mark.parametrize("n,seeds,one", [(1_000_000, [8192], True), (1_000_000, [8193, 5], False), (4_000_000, [50_000] * 8, True),
                                         (4_000_000, [50_000] * 7, False), (41_000_000, [10], False)])
def test_seeds_that_one_launch_takes(n, seeds, one):
    host_calls.run(f"""
c = context()
assert sample(c, {n}, 90_000_000, {seeds}, (10,)) == OK, lib.rg_last_error(c)
names = kernels()
assert ("k_sample_init" in names) == {one} and ("k_mark_seeds" in names) == (not {one}), names
""")


@pytest.mark.parametrize("n,edges,seeds,fanouts,order,tier", [
    (10_000_000, 200_000_000, [16], (-1, -1), "ASCENDING", "k_tier_emit"), (10_000_000, 200_000_000, [16], (1024, 64), "ASCENDING", "k_tier_emit"),
    (10_000_000, 200_000_000, [1024], (-1, -1, -1), "ASCENDING", "k_slice_emit<false>"),
    (10_000_000, 490_000_000, [4096] * 8, (15, 10, 5), "ASCENDING", "k_slice_emit<false>"),
    (10_000_000, 490_000_000, [700], (15, 10, 5), "ASCENDING", "k_slice_emit<false>"),           # 16 N edges of average nodes
    (10_000_000, 490_000_000, [500], (15, 10, 5), "ASCENDING", "k_tier_emit"),
    (1_000_000, 16_000_000, [16] * 8, (-1, -1), "FIRST_SEEN", "k_first_seen_emit")])
def test_tiers_by_the_edges_that_average_nodes_have(n, edges, seeds, fanouts, order, tier):
    host_calls.run(f"""
c = context()
assert sample(c, {n}, {edges}, {seeds}, {fanouts}, {order}) == OK, lib.rg_last_error(c)
names = kernels()
assert "{tier}" in names, names
""")


def test_few_edges_are_not_split_between_many_workgroups():
    """All neighbours of one seed: the marking pass is not cut up for every edge of the graph."""
    host_calls.run("""
c = context()
for seeds, fanouts, most in (([1], (-1,), 1), ([16], (-1, -1), 1), ([1500] * 2, (25, 10), 12)):
    assert sample(c, 1_000_000, 16_000_000, seeds, fanouts) == OK
    grids = [int(x.split()[2]) for x in log("launch k_slice_mark")]
    assert grids and max(grids) == most, grids
""")


@pytest.mark.parametrize("group", [1, 2, 16])
def test_few_edges_are_not_walked_by_workgroups_for_the_whole_graph(group):
    """All neighbours of a few seeds: the kernels that walk the hops' edges are launched for those of average nodes, eightfold, four
    workgroups per compute unit (of the 256 the recording runtime's device counts as) at least."""
    host_calls.run(f"""
c = context()
for order, names in ((ASCENDING, ["k_relabel"]), (FIRST_SEEN, ["k_first_seen_count", "k_first_seen_emit", "k_relabel"])):
    for local in (True, False):
        assert sample(c, 190_610, 35_400_000, [6] * {group}, (-1, 5), order, local=local) == OK, lib.rg_last_error(c)
        launches = log("launch")
        for name in names:
            grids = [int(x.split()[2]) for x in launches if x.split()[1].startswith(name)]
            assert max(grids, default=0) <= 1024 and (grids or not local and name == "k_relabel"), (name, grids)
    assert sample(c, 190_610, 35_400_000, [1024] * {group}, (25, 10), order) == OK              # nodes have them all: as many as the bound
    grids = [int(x.split()[2]) for x in log("launch") if x.split()[1].startswith("k_relabel") or x.split()[1].startswith("k_seen_relabel")]
    assert grids == [min(1024 * 26 * 10 // 1024, 8192 // {group}) * {group}], grids
""")


# 2.2 M edges in all, nodes times batches squared, a hop's and all edges above.
@pytest.mark.parametrize("n,edges,seeds,fanouts,ranked", [
    (10_000_000, 490_000_000, [4096], (15, 10, 5), False), (10_000_000, 490_000_000, [1100] * 2, (15, 10, 5), True),
    (10_000_000, 490_000_000, [1000] * 2, (15, 10, 5), False), (2_250_000, 112_000_000, [4096] * 2, (15, 10, 5), True),
    (2_240_000, 112_000_000, [4096] * 2, (15, 10, 5), False), (1_000_000, 49_000_000, [1024] * 3, (15, 10, 5), True),
    (232_965, 114_000_000, [4096] * 4, (25, 10), False), (300_000, 6_000_000, [1500] * 8, (25, 10), True),
    (150_000, 60_000_000, [1024] * 8, (15, 10, 5), True), (150_000, 60_000_000, [4000] * 8, (15, 10, 20), False),
    (10_000_000, 490_000_000, [500_000] * 2, (16,), True), (10_000_000, 490_000_000, [600_000] * 2, (16,), False)])
def test_first_seen_calls_that_rank_words_take(n, edges, seeds, fanouts, ranked):
    host_calls.run(f"""
c = context()
assert sample(c, {n}, {edges}, {seeds}, {fanouts}, FIRST_SEEN) == OK, lib.rg_last_error(c)
names = kernels()
assert ("k_seen_emit" in names) == {ranked} and ("k_first_seen_emit" in names) == (not {ranked}), names
""")


@pytest.mark.parametrize("seeds,scan", [(16_384 * 1024, False), (16_384 * 1024 + 1, True)])
def test_frontiers_whose_chunks_are_scanned(seeds, scan):
    host_calls.run(f"""
c = context()
assert sample(c, 20_000_000, 90_000_000, [{seeds}], (3,)) == OK
assert ("k_scan_hop" in kernels()) == {scan}
""")


# Rows, bytes of rows, bytes of rows in chunks of 8 or 4; on one stream and on two.
@pytest.mark.parametrize("rows,dim,one,two", [
    (65_536, 1, True, True), (65_537, 1, False, True), (98_304, 16, False, True), (98_305, 16, False, False), (8_000_000, 1, False, False),
    (12_288, 512, True, True), (12_289, 512, False, True), (16_384, 512, False, True), (16_385, 512, False, False),
    (8709, 602, True, True), (8710, 602, False, True), (13_934, 602, False, True), (13_935, 602, False, False), (19_878, 211, True, True), (19_879, 211, False, False)])
def test_gathers_that_one_launch_takes(rows, dim, one, two):
    host_calls.run(f"""
c = context()
for miss, expected in ((None, {one}), (0x52, {two})):
    for static in (False, True):
        if static and {rows} > 1 << 20:
            continue
        assert gather(c, {rows}, {dim}, hit=0x51, miss=miss, static=static) == OK, lib.rg_last_error(c)
        names = [k.split("<")[0] for k in kernels()]
        assert names == (["k_gather_fused"] if expected else ["k_classify", "k_gather_hbm", "k_gather_miss"]), (miss, static, names)
""")


def test_mean_aggregate_grid():
    """Up to 32 workgroups per compute unit (of the 256 the recording runtime's device counts as)."""
    host_calls.run("""
c = context()
for dst, grid in ((1, 1), (4 * 8192, 8192), (200_000, 8192)):
    assert lib.rg_mean_aggregate(c, p(address()), p(address()), i64(dst), None, p(address()), i64(256), i32(256), p(address()), i64(256), None) == OK
    assert [int(x.split()[2]) for x in log("launch k_mean_aggregate")] == [grid]
""")


# Rows of 80 chunks take 16 lanes each, of 76 chunks 32, of 65 a wavefront; up to 8192 rows all do, up to 16,384 at least 32 lanes: workgroups
# for as many whatever the device counts.
@pytest.mark.parametrize("dim,dst,grid", [(320, 2, 1), (320, 1000, 250), (320, 8192, 2048), (320, 8193, 2048), (320, 40_000, 2500),
                                          (304, 8192, 2048), (304, 40_000, 5000), (260, 20_000, 5000)])
def test_mean_aggregate_lanes_per_row(dim, dst, grid):
    host_calls.run(f"""
c = context()
assert lib.rg_mean_aggregate(c, p(address()), p(address()), i64({dst}), None, p(address()), i64({dim}), i32({dim}), p(address()), i64({dim}), None) == OK
assert [int(x.split()[2]) for x in log("launch k_mean_aggregate")] == [{grid}]
""")


def test_selection_grid():
    """The counts' histogram: one workgroup per compute unit, two above 8 Mi nodes."""
    host_calls.run("""
c = context()
for n, grid in ((1, 1), (4097, 2), (8 << 20, 256), ((8 << 20) + 1, 512)):
    cache = Cache(address(), address(), 1000, 4, address(), address(), address(), 0, None)
    assert lib.rg_build_cache(c, p(address()), p(address()), i64(n), None, i64(0), i32(4), byref(cache), None) == OK
    assert [int(x.split()[2]) for x in log("launch k_topk_hist_low")] == [grid]
    log()
""")


# Tiers from bytes by edges times nodes of all batches, up to 4 Mi nodes and two byte maps of 41 MB; counted by the emit up to 160,000 nodes.
# Beyond that the atomic marking for less than a 16th of the nodes' number of edges and 256 Ki in all.
@pytest.mark.parametrize("n,edges,seeds,fanouts,tier", [
    (232_965, 114_000_000, [1024], (25, 10), ["k_bytes_count", "k_tier_emit_small"]), (160_000, 9_000_000, [1024], (25, 10), ["k_bytes_emit_small"]),
    (160_001, 9_000_000, [1024], (25, 10), ["k_bytes_count", "k_tier_emit_small"]), (1_600_000, 9_000_000, [10] * 16, (10, 5), ["k_bytes_count", "k_tier_emit"]),
    (60_000, 9_000_000, [200] * 16, (25, 10), ["k_bytes_emit_small"]), (24_577, 9_000_000, [1536] * 16, (25, 10), ["k_bytes_emit_small"]),
    (4_194_304, 90_000_000, [100], (10, 5), ["k_bytes_count", "k_tier_emit_small"]), (4_194_305, 90_000_000, [100], (10, 5), ["k_tier_count", "k_tier_emit"]),
    (2_000_000, 90_000_000, [114] * 8, (25, 10), ["k_tier_count", "k_tier_emit"]), (2_000_000, 90_000_000, [115] * 8, (25, 10), ["k_slice_mark", "k_slice_count", "k_slice_emit"]),
    (1_000_000, 90_000_000, [3600], (10, 100), ["k_slice_mark", "k_slice_count<192, 1>", "k_slice_emit_small<false>"]),
    (1_900_000, 90_000_000, [10_000], (20, 9), ["k_bytes_count", "k_tier_emit_small"]),
    (1_900_000, 90_000_000, [10_100], (20, 9), ["k_slice_mark", "k_slice_count<192, 1>", "k_slice_emit_small<false>"]),
    (2_000_000, 90_000_000, [2618], (20, 9), ["k_bytes_count", "k_tier_emit_small"]),
    (2_000_000, 90_000_000, [2640], (20, 9), ["k_slice_mark", "k_slice_count<192, 1>", "k_slice_emit_small<false>"])])
def test_tiers_from_bytes(n, edges, seeds, fanouts, tier):
    host_calls.run(f"""
c = context()
assert sample(c, {n}, {edges}, {seeds}, {fanouts}) == OK, lib.rg_last_error(c)
names = list(dict.fromkeys(k.split("<")[0] for k in kernels() if "tier" in k or "bytes" in k or "slice" in k))
assert names == {[t.split("<")[0] for t in tier]}, names
""")


# One launch for batches of up to 20,480 edges, but for 10,500 (a thousand more per hop) where lists don't fit LDS on graphs of 70 neighbours per node.
@pytest.mark.parametrize("n,edges,seeds,fanouts,small", [
    (100_000, 7_000_000, [161], (10, 5), True), (100_000, 7_000_000, [162], (10, 5), False), (100_000, 6_999_999, [162], (10, 5), True),
    (100_000, 7_000_000, [15], (10, 5, 10), True), (100_000, 7_000_000, [16], (10, 5, 10), False), (50_000, 7_000_000, [162], (10, 5), True),
    (64_000, 7_000_000, [36], (25, 10), True), (64_000, 7_000_000, [40], (25, 10), False)])
def test_batches_of_dense_graphs_that_one_launch_takes(n, edges, seeds, fanouts, small):
    host_calls.run(f"""
c = context()
assert sample(c, {n}, {edges}, {seeds}, {fanouts}) == OK, lib.rg_last_error(c)
assert (len(kernels()) == 1) == {small}
""")


def test_no_gather_allocates_after_reserve():
    """Neither the calls of rg_gather_features_static nor any gather behind rg_reserve: more of them on two streams than there are signals,
    with writes that land at once and with none that does; nor while another stream of the thread records a graph."""
    host_calls.run("""
c = context()
assert lib.rg_reserve(c, i64(1000), i64(1000), i64(60_000), i32(1)) == OK
held = rt.memory_held()
log()
for landing in (1, 0):
    rt.land_values(landing)
    for k in range(200):
        for rows, dim, static in ((1500, 64, True), (60_000, 256, True), (1500, 64, False), (60_000, 256, False)):
            assert gather(c, rows, dim, hit=0x51, miss=0x52, static=static) == OK, lib.rg_last_error(c)
    lines = log()
    assert not [x for x in lines if x.startswith(("malloc", "free", "no memory"))], lines[:20]
rt.land_values(1)
d = context()
log()
rt.begin_capture(0x77)
for k in range(70):
    assert gather(d, 1500, 64, hit=0x51, miss=0x52, static=True) == OK
rt.end_capture()
lines = log()
assert not [x for x in lines if "malloc" in x] and [x for x in lines if x.startswith("write")], lines[:20]
lib.rg_destroy(c), lib.rg_destroy(d)
assert rt.memory_held() == 0
rt.begin_capture(0x77)                                    # a context made while a graph is recorded on another stream
e = context()
assert not [x for x in log() if x == "malloc in a graph"]
rt.end_capture()
lib.rg_destroy(e)
""")


# One launch up to 14 MB by values, above by events; three launches (from 32 MiB or 98,305 rows on) up to 64 MB by values, above by events.
@pytest.mark.parametrize("rows,dim,launches,by_value", [
    (1500, 64, 1, True), (14_336, 256, 1, True), (14_337, 256, 1, False), (30_000, 256, 1, False), (32_768, 256, 1, False), (32_769, 256, 3, True),
    (98_305, 16, 3, True), (65_536, 256, 3, True), (65_537, 256, 3, False)])
def test_streams_are_ordered_by_values_or_by_events(rows, dim, launches, by_value):
    """Each order is a write on the earlier stream and behind it a wait of the later one for the same value, or a record and a wait."""
    host_calls.run(f"""
c = context()
log()
for static in (False, True):
    assert gather(c, {rows}, {dim}, hit=0x51, miss=0x52, static=static) == OK, lib.rg_last_error(c)
    lines = log()
    assert sum(x.startswith("launch") for x in lines) == {launches}, lines
    orders = [x.split() for x in lines if x.split()[0] in ("write", "await", "record", "wait")]
    assert [x[0] for x in orders] == (["write", "await"] if {by_value} else ["record", "wait"]) * 2, orders
    for first, then in (orders[:2], orders[2:]):
        if {by_value}:                                        # stream, address, value
            assert first[2:] == then[2:] and {{first[1], then[1]}} == {{"0x51", "0x52"}}, orders
        else:                                                 # event, stream; stream, event
            assert first[1] == then[2] and {{first[2], then[1]}} == {{"0x51", "0x52"}}, orders
    # one launch runs on the hit stream: behind the miss stream, and in front of it; three begin and end there
    streams = [orders[0][1 if {by_value} else 2], orders[2][1 if {by_value} else 2]]
    assert streams == (["0x52", "0x51"] if {launches} == 1 else ["0x51", "0x52"]), orders
""")


def test_streams_are_ordered_by_events_where_values_cannot():
    """A signal whose last write has not landed is left alone; a device, an allocation, a write or a wait that is refused; recorded streams."""
    host_calls.run("""
def orders(c, n=1):
    log()
    for _ in range(n):
        assert gather(c, 1500, 64, hit=0x51, miss=0x52) == OK, lib.rg_last_error(c)
    return [x.split()[0] for x in log() if x.split()[0] in ("write", "await", "record", "wait")]
VALUES, EVENTS = ["write", "await"], ["record", "wait"]
c = context()
assert orders(c, 3) == VALUES * 6
rt.land_values(0)
got = orders(c, 100)
n = got.count("write")
assert 32 <= n < 200 and got == VALUES * n + EVENTS * (200 - n)
rt.land_values(1)
assert orders(c, 100) == VALUES * 200
for kinds in (1, 2):
    rt.refuse_values(kinds)
    d = context()
    assert orders(d, 2) == EVENTS * 4 and "malloc signal" not in log()
    lib.rg_destroy(d)
rt.refuse_values(4)
d = context()
assert orders(d, 2) == ["write"] + EVENTS * 4             # one try
rt.refuse_values(8)
e = context()
assert orders(e, 2) == ["write", "await"] + EVENTS * 4
rt.refuse_values(0)
for recorded in (0x51, 0x52):
    rt.begin_capture(recorded)
    gather(c, 1500, 64, hit=0x51, miss=0x52)
    rt.end_capture()
    assert not [x for x in log() if x.startswith(("write", "await"))]
""")


@pytest.mark.parametrize("n", [1, 3072, 3073, 4096])
def test_schedule_of_up_to_4096_ids_needs_no_scratch(n):
    """One launch, also as a context's first call while a graph is recorded, and without memory."""
    host_calls.run(f"""
def schedule(c, n, stream=0):
    return lib.rg_epoch_schedule(c, p(address()), i64(n), u64(7), u32(1), p(address()), p(stream))
c = context()
log()
rt.begin_capture(0x51)
assert schedule(c, {n}, 0x51) == OK, lib.rg_last_error(c)
rt.end_capture()
rt.limit_memory(rt.memory_held())
assert schedule(c, {n}) == OK, lib.rg_last_error(c)
lines = log()
assert [x.split("<")[0] for x in lines if x.startswith("launch")] == ["launch k_sched_sort"] * 2 and not [x for x in lines if "malloc" in x], lines
assert schedule(c, 4097) == OOM
""")


@pytest.mark.parametrize("n,scatter,sort", [
    (3072, None, "3072,true,1024,3072"), (4096, None, "4096,true,1024,4096"), (4097, "true,1", "2560,false,512,1024"),
    (262_144, "true,1", "2560,false,512,1024"), (262_145, "true,4", "2560,false,512,1024"), (400_000, "true,4", "2560,false,512,1024"),
    (400_001, "true,4", "2560,false,512,2560"), (8 << 20, "true,4", "2560,false,512,2560"), ((8 << 20) + 1, "false,4", "2560,false,512,2560")])
def test_schedule_kernels(n, scatter, sort):
    """Buckets of either size have room for 2560 ids."""
    host_calls.run(f"""
c = context()
log()
assert lib.rg_epoch_schedule(c, p(address()), i64({n}), u64(7), u32(1), p(address()), None) == OK
got = [x[len("launch "):x.index(">") + 1] for x in log("launch k_sched_s") if "<" in x]
assert got == ["k_sched_scatter<{scatter}>"] * {int(scatter is not None)} + ["k_sched_sort<{sort}>"], got
""")


# Beside the bounds from 256 seeds on, 1024 to a workgroup of few batches, 64 workgroups to a batch at most, 1024 in all.
@pytest.mark.parametrize("n,batches,seeds,stride,beside", [
    (1_000_000, 8, 255, 150_000, False), (1_000_000, 8, 256, 150_000, True), (1_000_000, 8, 16_384, 150_000, True), (10_000_000, 8, 65_536, 600_000, True), (10_000_000, 8, 8192, 74_000, True),
    (100_000, 64, 200_000, 600_000, True), (2_449_029, 192, 1024, 600_000, True), (2_449_029, 192, 20_000, 600_000, True), (300_000, 2000, 80_000, 30_000, True)])
def test_seeds_beside_the_bounds(n, batches, seeds, stride, beside):
    host_calls.run(f"""
c = context()
log()
assert histogram(c, {n}, {batches}, 2, seeds={seeds}, stride={stride}) == OK
lines = [x.split()[1:4] for x in log("launch")]
own = [x for x in lines if x[0] == "k_histogram_seeds"]
(_, gx, gy), = [x for x in lines if x[0] == "k_hist_bounds"]
gx, rows = int(gx), int(gy) - {batches} * 2
assert len(own) == {int(not beside)} and (rows > 0) == {beside}, lines
if {beside}:
    blocks = min(-(-{seeds} // 1024), 64, -(-1024 // {batches}))                 # whole rows of them
    assert rows == {batches} * max(1, (blocks + gx // 2) // gx), lines
""")
