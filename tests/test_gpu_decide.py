"""The case decision where its range test and its hint change course: values
at both ends of the range, NaN (quiet and signalling), infinities, zeros of
either sign and subnormals, alone, among decimals and among zeros; and runs of
chunks whose decimal places rise, fall and repeat.  Streams are the oracle's
byte for byte."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _specials(dt):
    f, u = (np.float64, np.uint64) if dt == "f64" else (np.float32, np.uint32)
    mant, amax, bmax = (52, 22, 15) if dt == "f64" else (23, 10, 6)
    top = 0x7FF << 52 if dt == "f64" else 0xFF << 23
    sign = 1 << (63 if dt == "f64" else 31)
    bits = [0, sign, 1, sign | 1, top, sign | top, top | 1, top | (1 << (mant - 1)), sign | top | 5]
    vals = list(np.array(bits, u).view(f))
    lo, hi = f(float(f"1e-{amax}")), f(float(f"1e{bmax}"))
    for v in (lo, hi):
        vals += [v, -v, np.nextafter(v, f(0)), np.nextafter(v, f(np.inf))]
    return vals, f


@pytest.mark.parametrize("fill", ["decimals", "zeros", "itself"])
@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_special_values(orc, dt, fill):
    from paper_2511_04140_amd import codec as C
    c = C.Codec(0)
    vals, f = _specials(dt)
    rng = np.random.default_rng(3)
    chunks = []
    for v in vals:
        for at in (0, 1, 63, 64, 700, 1024):
            x = {"decimals": np.rint(rng.uniform(-900, 900, 1025)) / 10, "zeros": np.zeros(1025),
                 "itself": np.zeros(1025)}[fill].astype(f)
            if fill == "itself":
                x[:] = v
            x[at] = v
            chunks.append(x)
    x = np.concatenate(chunks)
    for part in (x, x[: 1025 * 4], x[1025 * 6 * 6: 1025 * 6 * 6 + 1000]):
        xd = torch.from_numpy(part.copy()).cuda()
        torch.cuda.synchronize()
        s = c.compress(xd)
        assert s.cpu().numpy().tobytes() == orc.compress(part)
        assert torch.equal(c.decompress(s).view(torch.uint8), xd.view(torch.uint8))
    c.close()


@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_places_that_change(orc, dt):
    from paper_2511_04140_amd import codec as C
    c = C.Codec(0)
    f = np.float64 if dt == "f64" else np.float32
    rng = np.random.default_rng(4)
    out = []
    for i in range(9000):  # more chunks than waves, so a wave meets several
        p = [0, 0, 1, 3, 2, 2, 1, 4][(i // 700) % 8]
        m = np.rint(rng.uniform(-40, 40, 1025) * 10.0 ** p) / 10.0 ** p
        if i % 11 == 0:
            m[::17] = np.rint(m[::17])   # first values with fewer places
        if i % 13 == 0:
            m[900] = np.pi
        out.append(m.astype(f))
    x = np.concatenate(out)
    xd = torch.from_numpy(x).cuda()
    torch.cuda.synchronize()
    assert c.compress(xd).cpu().numpy().tobytes() == orc.compress(x)
    c.close()
