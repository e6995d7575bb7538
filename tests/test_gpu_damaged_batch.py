"""Batches that hold damaged streams beside whole ones, with a series past
4,096 chunks so that the offsets come from the scan.  Size words just below
2^32 once gave the chunk after them an offset before its payload.  Every
stream lies in the middle of a larger allocation; the call reports the damage,
and the whole series come back bit for bit beside it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("first", [2**32 - 100, 2**32 - 6000, 2**32 - 8000, 2**31, 8212])
@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_large_sizes_in_a_short_series(orc, dt, first):
    from paper_2511_04140_amd import codec as C
    rng = np.random.default_rng(first % 997)
    f = np.float64 if dt == "f64" else np.float32
    xs = [(np.rint(rng.uniform(-90, 90, n) * 10) / 10).astype(f)
          for n in (1025 * 9 + 1, 1025 * 3, 1025 * 4 - 5, 1025 * 4100 - 3)]
    room = []
    for i, x in enumerate(xs):
        s = bytearray(orc.compress(x))
        if i == 1:
            s[32:36] = first.to_bytes(4, "little")
        buf = torch.zeros(len(s) + 65536, dtype=torch.uint8, device="cuda")
        buf[32768:32768 + len(s)] = torch.from_numpy(np.frombuffer(bytes(s), np.uint8).copy()).cuda()
        room.append(buf[32768:32768 + len(s)])
    outs = [torch.full((x.size,), -1.0, dtype=torch.from_numpy(x).dtype, device="cuda") for x in xs]
    args = (room, [x.size for x in xs], [o.dtype for o in outs], outs)
    c = C.Codec(0)
    torch.cuda.synchronize()
    plan = c.plan_decompress(*args, tune=False)
    for call in (lambda: c.decompress_batch(*args), plan.run):
        for o in outs:
            o.fill_(-1.0)
        torch.cuda.synchronize()
        with pytest.raises(C.FalconError) as ei:
            call()
        assert ei.value.status == C.ERR_CORRUPT_STREAM
        for i in (0, 2, 3):
            assert np.array_equal(outs[i].cpu().numpy().view(np.uint8), xs[i].view(np.uint8)), i
    plan.close()
    c.close()
