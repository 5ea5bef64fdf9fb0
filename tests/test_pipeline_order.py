"""The order in which EpochPipeline queues a batch's work on its streams, with streams and events that only keep account."""
import types

import pytest

from paper_2505_10806_amd import binding as B
from paper_2505_10806_amd import pipeline as P


class Stream:
    def __init__(self, name):
        self.name, self.done = name, set()              # what the stream's next operation runs behind

    def run(self, what):
        self.done = self.done | {what}

    def wait_event(self, e):
        self.done = self.done | e.done


class Event:
    def __init__(self):
        self.done = set()

    def record(self, stream):
        self.done = set(stream.done)


@pytest.mark.parametrize("names", ["AAAAAA", "ABABAB", "AABBAA", "ABBAAB", "BAAABA"])
def test_miss_rows_wait_for_everything_that_uses_their_buffer(monkeypatch, names):
    """Six batches through two output buffers, each gathered and read on the stream that its letter names; the streams are not
    ordered with each other.  Before a batch's miss rows go into its buffer, the buffer's last batch has been copied and read."""
    main, side, began = {n: Stream(n) for n in "AB"}, Stream("side"), {}

    def run_part(ticket, part, *args, stream):
        began[ticket, part] = set(stream.done)
        stream.run((ticket, part))
    pipe = types.SimpleNamespace(
        state=types.SimpleNamespace(sizes=[10] * 6, cache=None), queue_depth=2, decoupled=True, consumer=None, side=side, _gathered=0,
        _gather_stream=None, out_ring=["one", "two"], _tickets={}, _fork_due={}, _rows_due=[False] * 2, prep_done=[Event(), Event()],
        ctx=types.SimpleNamespace(gather_run_part=run_part), cfg=types.SimpleNamespace(feat_dim=4),
        wl=types.SimpleNamespace(local_store=None, remote_store=None), _prepare=lambda st, batches: None,
        **{k: [Event(), Event()] for k in ("slot_free", "rows_done", "miss_done", "consumed")})
    for b, name in enumerate(names):
        monkeypatch.setattr(P.torch.cuda, "current_stream", lambda n=name: main[n])
        P.EpochPipeline.gather(pipe, b)
        assert (b, B.RG_GATHER_PART_MISS) in main[name].done and (b, B.RG_GATHER_PART_HBM) in main[name].done
        main[name].run(("read", b))
        if b >= 2:
            before = began[b, B.RG_GATHER_PART_MISS]
            assert (b - 2, B.RG_GATHER_PART_HBM) in before, b
            assert ("read", b - 2) in before, b
