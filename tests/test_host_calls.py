"""What the library's host code asks of the HIP runtime, call by call, without a GPU: order of streams, scratch, choice of kernels."""
import pytest

import host_calls


# One launch up to 32 MiB of rows, more above.
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
assert [k.split("<")[0] for k in kernels()] == ["k_classify", "k_gather_hbm", "k_gather_miss"]
assert (len(eager) == 1) == ({rows} <= 16384), eager
rt.begin_capture(0x51)
assert gather(c, {rows}, 512, hit=0x51, static={static}) == OK
assert rt.end_capture() == 0 and len(kernels()) == len(eager)
""")
