"""Operand planes of very small FP32 values.  A waveform or gradient times a power of two gives the
same projections and gradients times it, bit for bit, down to the rounding of results that are
subnormal: every value is the exact sum of its planes, and the accumulators hold them with room to
spare."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


@pytest.fixture(scope="module")
def melt():
    import paper_2606_01009_amd as m
    m.load_library()
    return m


def _normal(shape, seed):
    """Values in +-[0.5, 1) with all 24 significand bits."""
    r = np.random.default_rng(seed)
    return (r.choice([-1.0, 1.0], shape) * (0.5 + 0.5 * r.random(shape) * (1 - 2.0 ** -24))).astype(np.float32)


def _scaled(x, k):
    y = (x.astype(np.float64) * 2.0 ** -k).astype(np.float32)
    assert np.array_equal(y.astype(np.float64) * 2.0 ** k, x)
    return y


@pytest.mark.parametrize("k", [60, 100, 112, 118, 124])
@pytest.mark.parametrize("geom", [(400, 160, 80), (480, 161, 24), (1024, 256, 40)])
def test_projections(torch, melt, geom, k):
    N, H, M = geom
    plan = melt.MeltPlan(sample_rate=16000, n_fft=N, hop=H, n_mels=M)
    assert "split-planes" in melt.melt_variant_name(plan.handle, 0)
    x = _normal(70 * H + N + 3, 1)
    off = torch.tensor([0, x.size], device="cuda")
    T = melt.total_frames(off.cpu(), N, H)
    proj = [torch.empty((T, 2 * M), device="cuda") for _ in range(2)]
    plan.forward(torch.from_numpy(x).cuda(), off, T, proj=proj[0])
    plan.forward(torch.from_numpy(_scaled(x, k)).cuda(), off, T, proj=proj[1])
    want, got = (p.cpu().numpy().astype(np.float64) for p in proj)
    assert np.all(np.abs(got - want * 2.0 ** -k) <= 2.0 ** -149)


def test_projections_of_subnormal_samples(torch, melt):
    """Multiples of 2^-149 against the same whole numbers."""
    N, H, M = 400, 160, 40
    plan = melt.MeltPlan(sample_rate=16000, n_fft=N, hop=H, n_mels=M)
    n = np.random.default_rng(2).integers(-(1 << 22), 1 << 22, 40 * H + N)
    off = torch.tensor([0, n.size], device="cuda")
    T = melt.total_frames(off.cpu(), N, H)
    proj = [torch.empty((T, 2 * M), device="cuda") for _ in range(2)]
    plan.forward(torch.from_numpy(n.astype(np.float32)).cuda(), off, T, proj=proj[0])
    plan.forward(torch.from_numpy((n * 2.0 ** -149).astype(np.float32)).cuda(), off, T, proj=proj[1])
    want, got = (p.cpu().numpy().astype(np.float64) for p in proj)
    assert np.all(np.abs(got - want * 2.0 ** -149) <= 2.0 ** -149)


@pytest.mark.parametrize("what", ["upstream", "wave"])
@pytest.mark.parametrize("k", [60, 100, 112, 118, 124])
@pytest.mark.parametrize("geom", [(400, 160, 40), (300, 33, 17)])
def test_gradients(torch, melt, geom, k, what):
    """G = 2 R g of a power output with R, g in +-[0.5, 1); d/dbasis passes through one subnormal
    rounding for each of at most 64 partial sums."""
    N, H, M = geom
    plan = melt.MeltPlan(sample_rate=16000, n_fft=N, hop=H, n_mels=M, output=melt.MELT_OUT_POWER)
    x = _normal(90 * H + N, 3)
    off = torch.tensor([0, x.size], device="cuda")
    T = melt.total_frames(off.cpu(), N, H)
    g, proj = _normal((T, M), 4), torch.from_numpy(_normal((T, 2 * M), 5)).cuda()
    dev = lambda a: torch.from_numpy(a).cuda()
    gw0, gb0 = plan.backward(dev(x), off, T, dev(g), proj=proj)
    gw1, gb1 = plan.backward(dev(_scaled(x, k) if what == "wave" else x), off, T,
                             dev(_scaled(g, k) if what == "upstream" else g), proj=proj)
    f64 = lambda t: t.cpu().numpy().astype(np.float64)
    if what == "upstream":
        assert np.all(np.abs(f64(gw1) - f64(gw0) * 2.0 ** -k) <= 2.0 ** -149)
    assert np.all(np.abs(f64(gb1) - f64(gb0) * 2.0 ** -k) <= 64 * 2.0 ** -149)
