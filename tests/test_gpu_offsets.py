"""Payload offsets of decompression where the way they are found changes: up
to 4,096 chunks the decoder's waves add the sizes up themselves, beyond that a
scan runs before it, and beyond 64 tiles of 4,096 chunks a second one.  Values
come back bit for bit, damaged sizes and headers are reported either way."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _values(n, dt, seed):
    rng = np.random.default_rng(seed)
    x = np.rint(rng.uniform(-9, 9, n) * 10.0 ** rng.integers(0, 4)) / 100
    return x.astype(np.float64 if dt == "f64" else np.float32)


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("chunks", [1, 63, 64, 65, 257, 4095, 4096, 4097, 8193])
def test_one_series(orc, dt, chunks):
    from paper_2511_04140_amd import codec as C
    c = C.Codec(0)
    x = _values(1025 * chunks - 7, dt, chunks)
    s = orc.compress(x)
    dev = lambda b: torch.from_numpy(np.frombuffer(bytes(b), np.uint8).copy()).cuda()
    good = dev(s)
    for y in (c.decompress(good), c.decompress_n(good, x.size, torch.from_numpy(x).dtype)):
        assert np.array_equal(y.cpu().numpy().view(np.uint8), x.view(np.uint8))
    # one byte of a size: too large, too small, and a sum that no longer fits
    for at, val in ((chunks // 2, 0xFFFFFFFF), (0, 1), (chunks - 1, None)):
        bad = bytearray(s)
        p = 32 + 4 * at
        v = int.from_bytes(bad[p:p + 4], "little") - 1 if val is None else val
        bad[p:p + 4] = v.to_bytes(4, "little")
        with pytest.raises(C.FalconError) as ei:
            c.decompress(dev(bad))
        assert ei.value.status == C.ERR_CORRUPT_STREAM
    c.close()


def test_more_than_64_tiles():
    from paper_2511_04140_amd import codec as C
    c = C.Codec(0)
    n = 1025 * (64 * 4096 + 300) + 11
    x = torch.zeros(n, dtype=torch.float32, device="cuda")
    x[::1300] = torch.randint(-5000, 5000, (x[::1300].numel(),), device="cuda").float()
    y = c.decompress(c.compress(x))
    assert torch.equal(x.view(torch.int32), y.view(torch.int32))
    c.close()


@pytest.mark.parametrize("long_chunks", [40, 4097])
def test_batches(orc, long_chunks):
    """Series of both dtypes, empty ones among them; a series past 4,096 chunks
    sends the whole batch through the scan."""
    from paper_2511_04140_amd import codec as C
    rng = np.random.default_rng(long_chunks)
    ns = [int(v) for v in rng.integers(0, 9 * 1025, 60)] + [0, 1, 1025, 1026, 1025 * long_chunks - 3]
    xs = [_values(n, "f64" if i % 3 else "f32", i) for i, n in enumerate(ns)]
    streams = [torch.from_numpy(np.frombuffer(orc.compress(x), np.uint8).copy()).cuda() for x in xs]
    c = C.Codec(0)
    args = (streams, [x.size for x in xs], [torch.from_numpy(x).dtype for x in xs])
    plan = c.plan_decompress(*args)
    for ys in (c.decompress_batch(*args), plan.run(), plan.run()):
        for x, y in zip(xs, ys):
            assert np.array_equal(y.cpu().numpy().view(np.uint8), x.view(np.uint8))
    # damage: the header of an empty series, of a full one, and a size
    for i, at in ((ns.index(0), 24), (len(ns) - 1, 16), (len(ns) - 1, 32 + 4 * (long_chunks - 2))):
        keep = streams[i].clone()
        streams[i][at] ^= 1
        torch.cuda.synchronize()  # the plan runs on a stream of its own
        for call in (lambda: c.decompress_batch(*args), plan.run):
            with pytest.raises(C.FalconError) as ei:
                call()
            assert ei.value.status == C.ERR_CORRUPT_STREAM
        streams[i].copy_(keep)
        torch.cuda.synchronize()
    for x, y in zip(xs, plan.run()):
        assert np.array_equal(y.cpu().numpy().view(np.uint8), x.view(np.uint8))
    plan.close()
    c.close()


@pytest.mark.parametrize("dt,chunks", [("f64", 16384), ("f64", 16385), ("f64", 16449), ("f32", 24576), ("f32", 24577),
                                       ("f32", 30000)])
def test_drawn_chunks(dt, chunks):
    """Up to four chunks a wave (4,096 waves in float64, 6,144 in float32) the
    chunks are dealt out, beyond that they are drawn from counters that each
    launch leaves clear: every chunk comes back, three times in a row, and on
    two contexts at once."""
    from paper_2511_04140_amd import codec as C
    cs = [C.Codec(0, blocking=False) for _ in range(2)]
    dtype = torch.float64 if dt == "f64" else torch.float32
    n = 1025 * chunks - 3
    x = (torch.arange(n, device="cuda") * 7919 % 100003).to(dtype)
    torch.cuda.synchronize()  # the codec has a stream of its own
    s = cs[0].compress(x)
    ys = [torch.empty_like(x) for _ in cs]
    st = [torch.cuda.Stream() for _ in cs]
    for _ in range(3):
        for y in ys:
            y.zero_()
        torch.cuda.synchronize()
        for c, y, q in zip(cs, ys, st):
            c.decompress_n_async(s, n, dtype, y, stream=q)
        for c in cs:
            c.sync()
        for y in ys:
            assert torch.equal(y, x)
    for c in cs:
        c.close()


def test_drawn_chunks_of_a_plan():
    """Replays of a decompression plan whose launches draw their chunks."""
    from paper_2511_04140_amd import codec as C
    c = C.Codec(0)
    xs = [(torch.arange(1025 * 60 + 11 * i, device="cuda") % 977).to(torch.float64 if i % 2 else torch.float32)
          for i in range(700)]
    torch.cuda.synchronize()
    streams = c.compress_batch(xs)
    outs = [torch.empty_like(x) for x in xs]
    torch.cuda.synchronize()
    plan = c.plan_decompress(streams, [x.numel() for x in xs], [x.dtype for x in xs], outs)
    for _ in range(3):
        for y in outs:
            y.zero_()
        torch.cuda.synchronize()
        plan.run()
        assert all(torch.equal(y, x) for x, y in zip(xs, outs))
    plan.close()
    c.close()
