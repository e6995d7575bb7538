"""A run reports its own errors and no earlier run's: decompression plans made
(and tuned) over buffers that do not hold their streams yet, filled afterwards;
and good runs after failing ones, through plans and batch calls."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _case(orc, chunks):
    rng = np.random.default_rng(chunks)
    xs = [(np.rint(rng.uniform(-90, 90, 1025 * k - 7) * 10) / 10).astype(np.float64 if i % 2 else np.float32)
          for i, k in enumerate((1, 3, chunks, 2))]
    dev = [torch.from_numpy(np.frombuffer(orc.compress(x), np.uint8).copy()).cuda() for x in xs]
    return xs, dev, [x.size for x in xs], [torch.from_numpy(x).dtype for x in xs]


def _same(ys, xs):
    for y, x in zip(ys, xs):
        assert np.array_equal(y.cpu().numpy().view(np.uint8), x.view(np.uint8))


@pytest.mark.parametrize("chunks", [40, 4100])
@pytest.mark.parametrize("graph", [True, False])
@pytest.mark.parametrize("tune", [True, False])
def test_a_plan_made_before_its_streams(orc, tune, graph, chunks):
    from paper_2511_04140_amd import codec as C
    xs, dev, counts, dtypes = _case(orc, chunks)
    c = C.Codec(0)
    bufs = [torch.zeros_like(d) for d in dev]
    torch.cuda.synchronize()
    plan = c.plan_decompress(bufs, counts, dtypes, tune=tune, graph=graph)
    for rep in range(2):
        for b, d in zip(bufs, dev):
            b.copy_(d)
        torch.cuda.synchronize()
        _same(plan.run(), xs)
        for b in bufs:
            b.zero_()
        torch.cuda.synchronize()
        with pytest.raises(C.FalconError) as ei:
            plan.run()
        assert ei.value.status == C.ERR_CORRUPT_STREAM
    plan.close()
    c.close()


def test_a_batch_call_after_a_failed_one(orc):
    from paper_2511_04140_amd import codec as C
    xs, dev, counts, dtypes = _case(orc, 20)
    c = C.Codec(0)
    bad = [torch.zeros_like(d) for d in dev]
    torch.cuda.synchronize()
    for rep in range(2):
        with pytest.raises(C.FalconError):
            c.decompress_batch(bad, counts, dtypes)
        _same(c.decompress_batch(dev, counts, dtypes), xs)
        for s, d in zip(c.compress_batch([torch.from_numpy(x).cuda() for x in xs]), dev):
            assert torch.equal(s, d)
    c.close()
