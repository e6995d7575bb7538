"""One-launch compression at the sizes where its parts meet: one chunk and the
last partial chunk, the switch from 4- to 8-wave workgroups (1,024 chunks), the
scanning workgroup's rounds (1,024 and 2,048 sizes), payloads of every length
modulo 16 and the largest ones, many short series in one scan, several launches
in flight, and replays of a captured launch (the queue's words are left clear
for the next).  Every stream equals the oracle's byte for byte."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _data(n, dt, seed):
    """Chunks of all kinds in turn: decimals, random bits (every row dense: the
    largest payload), constants and zeros (the smallest)."""
    rng = np.random.default_rng(seed)
    u, f = (np.uint64, np.float64) if dt == "f64" else (np.uint32, np.float32)
    x = (np.rint(rng.uniform(-50, 50, n) * 100) / 100).astype(f)
    kind = rng.integers(0, 8, (n + 1024) // 1025)
    for c in np.nonzero(kind < 3)[0]:
        lo, hi = 1025 * c, min(n, 1025 * (c + 1))
        if kind[c] == 0:
            x[lo:hi] = rng.integers(0, np.iinfo(u).max, hi - lo, dtype=u).view(f)
        else:
            x[lo:hi] = 7.25 * (kind[c] - 1)
    return x


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("chunks", [1, 2, 5, 64, 1023, 1024, 1025, 2047, 2048, 2049, 4200])
def test_edges(orc, dt, chunks):
    from paper_2511_04140_amd import codec as C
    c = C.Codec(0)
    for k, n in enumerate((1025 * chunks, 1025 * chunks - 1024, 1025 * chunks - 3)):
        x = _data(n, dt, 100 * chunks + k)
        xd = torch.from_numpy(x).cuda()
        s = c.compress(xd)
        assert s.cpu().numpy().tobytes() == orc.compress(x), n
        y = c.decompress(s)
        assert torch.equal(y.view(torch.uint8), xd.view(torch.uint8)), n
    c.close()


@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_outputs_at_every_alignment(orc, dt):
    """Payload stores take any byte address; nothing outside the stream is
    written."""
    from paper_2511_04140_amd import codec as C
    c = C.Codec(0)
    x = _data(1025 * 40 - 5, dt, 9)
    xd = torch.from_numpy(x).cuda()
    want = orc.compress(x)
    cap = C.compress_bound(x.size, xd.dtype)
    for off in range(0, 128, 4):
        room = torch.full((cap + 256,), 0xA5, dtype=torch.uint8, device="cuda")
        n = c.compress(xd, out=room[off:off + cap]).numel()
        got = room.cpu().numpy()
        assert got[off:off + n].tobytes() == want
        assert (got[:off] == 0xA5).all() and (got[off + n:] == 0xA5).all()
    c.close()


def test_many_short_series(orc):
    """Series of 0 to 6 chunks: several first chunks in every block of the
    scan, split and mixed launches."""
    from paper_2511_04140_amd import codec as C
    rng = np.random.default_rng(5)
    xs = [_data(int(rng.integers(0, 6 * 1025)), "f64" if rng.random() < 0.6 else "f32", 1000 + i) for i in range(700)]
    xd = [torch.from_numpy(x).cuda() for x in xs]
    want = [orc.compress(x) for x in xs]
    c = C.Codec(0)
    for rep in range(2):
        for s, w in zip(c.compress_batch(xd), want):
            assert s.cpu().numpy().tobytes() == w
    plan = c.plan_compress(xd)
    for s, w in zip(plan.run(), want):
        assert s.cpu().numpy().tobytes() == w
    plan.close()
    c.close()


def test_launches_in_flight_together(orc):
    """Two contexts whose launches overlap on two streams, each filling the
    chip: neither waits for the other's workgroups."""
    from paper_2511_04140_amd import codec as C
    xs = [_data(1025 * 9000 + 17, "f64", 3), _data(1025 * 12000 + 5, "f32", 4)]
    xd = [torch.from_numpy(x).cuda() for x in xs]
    want = [orc.compress(x) for x in xs]
    cs = [C.Codec(0, blocking=False) for _ in xs]
    st = [torch.cuda.Stream() for _ in xs]
    bufs = [torch.zeros(C.compress_bound(x.size, d.dtype), dtype=torch.uint8, device="cuda") for x, d in zip(xs, xd)]
    torch.cuda.synchronize()
    for rep in range(5):
        lens = [c.compress_async(d, b, stream=s) for c, d, b, s in zip(cs, xd, bufs, st)]
        for c in cs:
            c.sync()
        for ln, b, w in zip(lens, bufs, want):
            assert b[:ln.value].cpu().numpy().tobytes() == w, rep
    for c in cs:
        c.close()


def test_replays_of_a_captured_launch(orc):
    from paper_2511_04140_amd import codec as C
    c = C.Codec(0, blocking=False, device_lengths=True)
    s = torch.cuda.Stream()
    xs = [_data(1025 * 3000 + 7, "f64", 20 + k) for k in range(3)]
    xd = torch.from_numpy(xs[0]).cuda()
    buf = torch.zeros(C.compress_bound(xd.numel(), xd.dtype), dtype=torch.uint8, device="cuda")
    ln = torch.zeros(1, dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    c.compress_async(xd, buf, out_len=ln, stream=s)  # grows the context's scratch
    c.sync()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        c.compress_async(xd, buf, out_len=ln, stream=s)
    for rep in range(4):
        x = xs[rep % 3]
        xd.copy_(torch.from_numpy(x))
        torch.cuda.synchronize()
        if rep == 2:  # an eager call between replays
            c.compress_async(xd, buf, out_len=ln, stream=s)
            c.sync()
        buf.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert buf[:int(ln.item())].cpu().numpy().tobytes() == orc.compress(x), rep
    c.close()


def test_streams_in_turn(orc):
    """Calls of one context on alternating streams, each reading what the one
    before it wrote: a call on another stream than the last waits for it, and
    stream lengths and errors arrive with the sync that follows."""
    from paper_2511_04140_amd import codec as C
    c = C.Codec(0, blocking=False)
    st = [torch.cuda.Stream(), torch.cuda.Stream()]
    x = torch.from_numpy(_data(1025 * 700 + 3, "f64", 9)).cuda()
    want = np.frombuffer(orc.compress(x.cpu().numpy()), np.uint8)
    torch.cuda.synchronize()
    for _ in range(3):
        src, lens, bufs, keep = x, [], [], []
        for k in range(6):
            buf = torch.empty(C.compress_bound(x.numel(), x.dtype), dtype=torch.uint8, device="cuda")
            y = torch.empty_like(x)
            lens.append(c.compress_async(src, buf, stream=st[k % 2]))
            c.decompress_n_async(buf, x.numel(), x.dtype, y, stream=st[(k + 1) % 2])
            src = y
            bufs.append(buf)
            keep.append(y)
        c.sync()
        assert torch.equal(src.view(torch.int64), x.view(torch.int64))
        for ln, buf in zip(lens, bufs):
            assert np.array_equal(buf[: ln.value].cpu().numpy(), want)
        torch.cuda.synchronize()
    c.close()


@pytest.mark.parametrize("chunks", [4607, 4608, 4609, 9217])
def test_scan_rounds_of_float32(orc, chunks):
    """float32 launches past 1,024 chunks run in workgroups of 12 waves, whose
    scanning one takes 4,608 sizes a round."""
    from paper_2511_04140_amd import codec as C
    c = C.Codec(0)
    x = _data(1025 * chunks - 9, "f32", chunks)
    xd = torch.from_numpy(x).cuda()
    want = np.frombuffer(orc.compress(x), np.uint8)
    torch.cuda.synchronize()
    for _ in range(2):
        assert np.array_equal(c.compress(xd).cpu().numpy(), want)
    c.close()


@pytest.mark.parametrize("dt,chunks", [("f64", 4087), ("f64", 4088), ("f64", 4089), ("f32", 6131), ("f32", 6132),
                                       ("f32", 6133)])
def test_a_wave_per_chunk(orc, dt, chunks):
    """Launches whose chunks all have a wave of their own (511 workgroups of 8
    waves in float64, of 12 in float32, beside the scanning one) draw nothing;
    one chunk more and they do.  In turn, on the same words."""
    from paper_2511_04140_amd import codec as C
    c = C.Codec(0)
    x = _data(1025 * chunks - 1000, dt, chunks)
    xd = torch.from_numpy(x).cuda()
    small = xd[: 1025 * 30 + 1].clone()
    want, want_small = (np.frombuffer(orc.compress(v.cpu().numpy()), np.uint8) for v in (xd, small))
    torch.cuda.synchronize()
    for _ in range(2):
        assert np.array_equal(c.compress(xd).cpu().numpy(), want)
        assert np.array_equal(c.compress(small).cpu().numpy(), want_small)
    c.close()


@pytest.mark.parametrize("tail", [0, 1, 64])
def test_series_of_a_batch_by_index(orc, tail):
    """Batches whose series begin and end around every 64th launch chunk, empty
    ones between them, at the front and at the end."""
    from paper_2511_04140_amd import codec as C
    c = C.Codec(0)
    chunks = [0, 1, 64, 0, 62, 1, 0, 128, 1, 0, 0, 63, 5, 64] * 4 + [1] * 130 + [tail]
    xs = [_data(max(0, 1025 * k - (i % 3)) if k else 0, "f64" if i % 2 else "f32", i) for i, k in enumerate(chunks)]
    xd = [torch.from_numpy(x).cuda() for x in xs]
    torch.cuda.synchronize()
    got = c.compress_batch(xd)
    for x, s in zip(xs, got):
        assert s.cpu().numpy().tobytes() == orc.compress(x)
    ys = c.decompress_batch(got, [x.size for x in xs], [x.dtype for x in xd])
    for x, y in zip(xs, ys):
        assert y.cpu().numpy().tobytes() == x.tobytes()
    c.close()
