"""The tuner times the geometry that an untuned plan runs (default_ms): it is
one of the candidates, also where its launches of the two dtypes take
workgroups of different sizes."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("chunks64,chunks32,candidates", [(1500, 0, 4), (0, 90, 4), (1500, 1200, 8), (200, 90, 8),
                                                          (1500, 90, 9), (90, 1500, 9)])
def test_the_default_is_a_candidate(chunks64, chunks32, candidates):
    from paper_2511_04140_amd import codec as C
    c = C.Codec(0)
    xs = [torch.arange(1025 * k, device="cuda").to(dt) / 4
          for k, dt in ((chunks64, torch.float64), (chunks32, torch.float32)) if k]
    torch.cuda.synchronize()
    want = [s.clone() for s in c.compress_batch(xs)]
    plan = c.plan_compress(xs)
    info = plan.info()
    assert info["candidates"] == candidates and 0 < info["best_ms"] <= info["default_ms"]
    for s, w in zip(plan.run(), want):
        assert torch.equal(s, w)
    plan.close()
    c.close()
