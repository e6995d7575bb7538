"""Calls recorded into a graph after eager calls of the same size: the scratch
is grown by then, and a decompression finds its own grown by the compression
that made its stream."""
import ctypes
import re

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _values(n, k, dt):
    return ((torch.arange(n, device="cuda") * 7919 + k) % 100003).to(dt) / 4


@pytest.mark.parametrize("dt", [torch.float64, torch.float32])
@pytest.mark.parametrize("chunks", [20, 4096, 4097, 17000])
@pytest.mark.parametrize("variant", [None, "dense"])
def test_decompression_recorded_after_a_compression(variant, chunks, dt):
    from paper_2511_04140_amd import codec as C
    n = 1025 * chunks - 9
    c = C.Codec(0, blocking=False)
    s = torch.cuda.Stream()
    x = _values(n, 0, dt)
    buf = torch.empty(C.compress_bound(n, dt), dtype=torch.uint8, device="cuda")
    y = torch.empty_like(x)
    torch.cuda.synchronize()

    def compress():
        if variant:
            c.compress_variant(x, variant, out=buf)
        else:
            c.compress_async(x, buf, stream=s)
            c.sync()
    compress()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        c.decompress_n_async(buf, n, dt, y, stream=s)
    for rep in range(3):
        x.copy_(_values(n, rep, dt))
        torch.cuda.synchronize()
        compress()
        y.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, x), rep
    c.close()


@pytest.mark.parametrize("warm,chunks", [(17000, 32768), (600, 1024), (2049, 4096)])
def test_calls_up_to_the_next_power_of_two(warm, chunks):
    """Scratch grows to powers of two: what fits is recorded without an eager
    call of its own size."""
    from paper_2511_04140_amd import codec as C
    n = 1025 * chunks
    c = C.Codec(0, blocking=False, device_lengths=True)
    s = torch.cuda.Stream()
    x = _values(n, 0, torch.float32)
    buf = torch.empty(C.compress_bound(n, x.dtype), dtype=torch.uint8, device="cuda")
    y = torch.empty_like(x)
    ln = torch.zeros(1, dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    c.compress_async(x[: 1025 * warm], buf, out_len=ln, stream=s)
    c.sync()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        c.compress_async(x, buf, out_len=ln, stream=s)
        c.decompress_n_async(buf, n, x.dtype, y, stream=s)
    for rep in range(3):
        x.copy_(_values(n, rep, x.dtype))
        y.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, x), rep
    c.close()


@pytest.mark.parametrize("chunks", [20, 5000])
@pytest.mark.parametrize("first", ["replay", "eager"])
def test_the_first_call_is_recorded(first, chunks):
    """Where the capture lets memory be allocated, a context's first call can
    be recorded.  The graph holds what a later capture of the call holds:
    nothing that clears words which eager calls use as well."""
    from paper_2511_04140_amd import codec as C
    n = 1025 * chunks
    c = C.Codec(0, blocking=False, device_lengths=True)
    s = torch.cuda.Stream()
    x = _values(n, 0, torch.float64)
    buf = torch.empty(C.compress_bound(n, x.dtype), dtype=torch.uint8, device="cuda")
    y = torch.empty_like(x)
    ln = torch.zeros(1, dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    hip = ctypes.CDLL(re.search(r"/\S*libamdhip64\S*", open("/proc/self/maps").read()).group(0))

    def call():
        c.compress_async(x, buf, out_len=ln, stream=s)
        c.decompress_n_async(buf, n, x.dtype, y, stream=s)

    def record():
        g = torch.cuda.CUDAGraph(keep_graph=True)
        with torch.cuda.graph(g, stream=s, capture_error_mode="relaxed"):
            call()
        nodes = ctypes.c_size_t()
        assert hip.hipGraphGetNodes(ctypes.c_void_p(g.raw_cuda_graph()), None, ctypes.byref(nodes)) == 0
        g.instantiate()
        return g, nodes.value
    g, nodes = record()
    for rep, how in enumerate((first, "replay", "eager", "replay")):
        x.copy_(_values(n, rep, x.dtype))
        y.zero_()
        torch.cuda.synchronize()
        if how == "replay":
            g.replay()
        else:
            call()
            c.sync()
        torch.cuda.synchronize()
        assert torch.equal(y, x), rep
    assert record()[1] == nodes
    c.close()
