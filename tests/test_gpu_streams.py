"""A call on another stream than the last waits for that call, and for nothing
else: the caller's stream may hold later work, be captured or be gone by then."""
import ctypes
import re

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


class _Two:
    """Two compressions whose streams are known, and what they need."""

    def __init__(self, orc):
        from paper_2511_04140_amd import codec as C
        rng = np.random.default_rng(11)
        self.c = C.Codec(0, blocking=False)
        x = [np.rint(rng.uniform(-90, 90, 1025 * 1500 - k) * 100) / 100 for k in (0, 7)]
        self.want = [np.frombuffer(orc.compress(v), np.uint8) for v in x]
        self.x = [torch.from_numpy(v).cuda() for v in x]
        self.buf = [torch.zeros(C.compress_bound(v.size, torch.float64), dtype=torch.uint8, device="cuda") for v in x]
        torch.cuda.synchronize()
        self.call(0, torch.cuda.Stream())  # grows the context's scratch
        self.check(0)

    def call(self, k, stream):
        self.len = self.c.compress_async(self.x[k], self.buf[k], stream=stream)

    def check(self, *ks):
        self.c.sync()
        torch.cuda.synchronize()
        for k in ks:
            assert np.array_equal(self.buf[k][: self.want[k].size].cpu().numpy(), self.want[k])
            self.buf[k].zero_()
        torch.cuda.synchronize()


def _cycles(ms):
    """Arguments of torch.cuda._sleep for a time."""
    a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    n = 10_000_000
    torch.cuda._sleep(1000)
    torch.cuda.synchronize()
    a.record()
    torch.cuda._sleep(n)
    b.record()
    b.synchronize()
    return int(n * ms / a.elapsed_time(b))


def _apart(t, long):
    """A stream that another one and the context's own overlap (streams can
    share a hardware queue), and that other one."""
    for _ in range(12):
        s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
        e1, e2 = torch.cuda.Event(), torch.cuda.Event()
        with torch.cuda.stream(s1):
            torch.cuda._sleep(long // 10)
            e1.record()
        with torch.cuda.stream(s2):
            torch.cuda._sleep(1000)
            e2.record()
        e2.synchronize()
        t.call(0, None)
        t.c.sync()
        apart = not e1.query()
        t.check(0)
        if apart:
            return s1, s2
    pytest.skip("every stream shares a hardware queue with another")


@pytest.mark.parametrize("what", ["call", "times"])
def test_later_work_on_the_last_stream(orc, what):
    t = _Two(orc)
    long = _cycles(600)
    s1, s2 = _apart(t, long)
    e1, e2 = torch.cuda.Event(), torch.cuda.Event()
    t.call(0, s1)
    with torch.cuda.stream(s1):
        torch.cuda._sleep(long)
        e1.record()
    if what == "call":
        t.call(1, s2)
        e2.record(s2)
        e2.synchronize()
    else:
        assert sum(t.c.call_stage_ms(0)) > 0
    assert not e1.query()  # the program's own work is still running
    torch.cuda.synchronize()
    t.check(*((0, 1) if what == "call" else (0,)))
    t.c.close()


def test_the_last_stream_is_captured(orc):
    """The runtime takes no wait for a stream that is being captured: the call
    is refused, not recorded into the program's graph, which is whole; after
    the capture the context works as before."""
    from paper_2511_04140_amd import codec as C
    t = _Two(orc)
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    own = torch.zeros(100, device="cuda")
    t.call(0, s1)
    g = torch.cuda.CUDAGraph()
    status = 0
    with torch.cuda.graph(g, stream=s1, capture_error_mode="thread_local"):
        own += 1
        try:
            t.call(1, s2)
        except C.FalconError as e:
            status = e.status
    assert status == 4  # FALCON_ERR_DEVICE
    t.check(0)
    for rep in range(1, 4):
        g.replay()
        torch.cuda.synchronize()
        assert (own == rep).all() and not t.buf[1].any()
        t.call(1, s2 if rep % 2 else s1)
        t.check(1)
    t.c.close()


def test_a_recorded_call_then_one_on_another_stream(orc):
    t = _Two(orc)
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    t.c.sync()
    with torch.cuda.graph(g, stream=s1, capture_error_mode="thread_local"):
        t.call(0, s1)
    t.call(1, s2)
    t.check(1)
    for rep in range(3):
        g.replay()
        torch.cuda.synchronize()
        t.call(1, s2 if rep % 2 else None)
        t.check(0, 1)
    t.c.close()


def test_the_last_stream_is_destroyed(orc):
    path = {m.group(0) for m in re.finditer(r"/\S*libamdhip64\S*", open("/proc/self/maps").read())}
    assert len(path) == 1
    hip = ctypes.CDLL(path.pop())
    t = _Two(orc)
    s2 = torch.cuda.Stream()
    for rep in range(4):
        raw = ctypes.c_void_p()
        assert hip.hipStreamCreateWithFlags(ctypes.byref(raw), 1) == 0
        s1 = torch.cuda.ExternalStream(raw.value)
        t.call(0, s1)
        assert hip.hipStreamDestroy(raw) == 0
        t.call(1, s2 if rep % 2 else None)
        t.check(0, 1)
    t.c.close()
