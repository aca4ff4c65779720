"""The split-plane kernel (FP32 on three bfloat16 planes per operand, BF16X3 / FP16X3 on two)
at the sizes where its tiles, item shapes and staging change, against the FP64 oracle with the
per-bin bounds of the other MelT tests (tests/parity.py), and its treatment of samples that the
planes cannot hold."""
import numpy as np
import pytest

import workloads
from tests.test_gpu_melt import _check, _gpu_forward

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


def _plan(melt, geom, prec, **kw):
    sr, N, H, M = geom
    plan = melt.MeltPlan(sample_rate=sr, n_fft=N, hop=H, n_mels=M, precision=prec, **kw)
    assert "split-planes" in melt.melt_variant_name(plan.handle, 0)
    return plan


@pytest.mark.parametrize("M", [1, 7, 8, 9, 13, 24, 40, 72, 100, 129, 200, 512])
def test_mel_counts(torch, melt, orc, M):
    """Row tiles of 8 bins: a partial one, an odd count, one more than a wave pair holds, several
    row parts, and widths that take no 16-byte stores."""
    plan = _plan(melt, (16000, 400, 160, M), "fp32")
    wave, off = workloads.random_clips([399, 400, 15 * 160 + 400, 16 * 160 + 400, 130 * 160 + 401], seed=M)
    L, _ = _gpu_forward(torch, melt, plan, wave, off)
    _check(orc, melt, plan, L, wave, off, "fp32", label=f"M={M}")


@pytest.mark.parametrize("frames", [1, 15, 33, 65, 129, 700, 5000])
@pytest.mark.parametrize("geom", [(16000, 400, 160, 80), (22050, 1024, 256, 128), (16000, 480, 161, 64),
                                  (16000, 400, 50, 40)])
def test_item_shapes(torch, melt, orc, geom, frames):
    """From one frame to several chunks per compute unit: 32-, 64- and 128-frame items with one
    or more row parts; whole and padded hop rows; a second clip that ends inside a 4-sample
    vector."""
    sr, N, H, M = geom
    plan = _plan(melt, geom, "fp32")
    wave, off = workloads.random_clips([(frames - 1) * H + N, 3 * H + N + 1], seed=frames)
    L, _ = _gpu_forward(torch, melt, plan, wave, off)
    _check(orc, melt, plan, L, wave, off, "fp32", label=f"{geom} {frames} frames")


@pytest.mark.parametrize("geom", [(16000, 400, 160, 80), (16000, 480, 161, 64), (22050, 1024, 256, 128)])
def test_rows_do_not_depend_on_the_item_shape(torch, melt, geom):
    """A clip alone (small items) and inside a batch (128-frame items) gives the same bits."""
    sr, N, H, M = geom
    plan = _plan(melt, geom, "fp32")
    wave, off = workloads.random_clips([100 * H + N + 2] + [300 * H + N] * 200, seed=5)
    many, _ = _gpu_forward(torch, melt, plan, wave, off)
    alone, _ = _gpu_forward(torch, melt, plan, wave[:off[1]].copy(), off[:2])
    assert np.array_equal(many[:101], alone)


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan, np.finfo(np.float32).max])
def test_samples_the_planes_cannot_hold(torch, melt, bad):
    """An infinity, a NaN, or a sample that rounds to infinity in bfloat16: the frames that hold
    it come out as plain FP32 arithmetic gives them, all others bit for bit as without it."""
    N, H, M = 480, 161, 40
    kw = dict(output=melt.MELT_OUT_MAGNITUDE)
    plan = _plan(melt, (16000, N, H, M), "fp32", **kw)
    wave, off = workloads.random_clips([60 * H + N, 5 * H + N], seed=3)
    wave[20 * H + 100] = 0.0
    clean, _ = _gpu_forward(torch, melt, plan, wave, off)
    wave[20 * H + 100] = bad
    got, _ = _gpu_forward(torch, melt, plan, wave, off)
    hit = np.zeros(clean.shape[0], bool)
    hit[[t for t in range(61) if t * H <= 20 * H + 100 < t * H + N]] = True
    assert hit.sum() == 3 and np.array_equal(got[~hit], clean[~hit])
    W = plan.basis()
    for t in np.flatnonzero(hit):
        x = torch.from_numpy(wave[t * H:t * H + N])
        y = (torch.from_numpy(W) * x).sum(1).numpy()        # FP32
        with np.errstate(over="ignore", invalid="ignore"):
            want = np.sqrt(y[:M] * y[:M] + y[M:] * y[M:])
        assert np.array_equal(np.isnan(got[t]), np.isnan(want))
        assert np.array_equal(np.isinf(got[t]), np.isinf(want))


def test_overflow_after_a_frame_stays_outside(torch, melt):
    """FP16X3, N 1200 at hop 160 (the last segment of 80 samples ends half-way through a k-group of
    32): a sample beyond binary16's range in the 16 samples after a frame does not reach it."""
    N, H = 1200, 160
    plan = _plan(melt, (16000, N, H, 128), "fp16x3")
    wave, off = workloads.random_clips([30 * H + N], seed=4)
    clean, _ = _gpu_forward(torch, melt, plan, wave, off)
    at = 10 * H + N + 5
    wave[at] = 1000.0
    got, _ = _gpu_forward(torch, melt, plan, wave, off)
    for t in range(31):
        if t * H <= at < t * H + N:
            assert not np.isfinite(got[t]).all()
        else:
            assert np.array_equal(got[t], clean[t])


@pytest.mark.parametrize("geom", [(16000, 480, 161, 64), (16000, 400, 160, 9), (8000, 256, 80, 24), (16000, 320, 160, 65),
                                  (16000, 300, 33, 17), (22050, 1024, 256, 128), (16000, 400, 160, 3)])
def test_backward_shapes(torch, melt, orc, geom):
    """d/dwave and d/dbasis on operand planes: hops and Mel counts that fill no tile, blocks of
    128 x 256 basis elements with remainders, frame ranges that end inside a step of 32, clips
    shorter than a chunk of hop rows, and (3 Mel bins) the FP32-MFMA d/dwave kernel beside the
    plane d/dbasis."""
    from tests.test_gpu_backward import _case
    sr, N, H, M = geom
    wave, off = workloads.random_clips([N - 1, N, 70 * H + N + 3, 5 * H + N + 1, 131 * H + N], seed=N + M)
    _case(torch, melt, orc, wave, off, float(sr), N, H, M, label=f"backward {geom}")


@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_upstream_gradients_the_planes_cannot_hold(torch, melt, bad):
    """One infinite or NaN upstream gradient: the samples and basis rows it reaches are non-finite
    in the way FP32 arithmetic makes them, everything else is bit for bit as without it.  The
    samples that only share the frame's last hop-block row meet it with zero weights, so they are
    recomputed in plain FP32: finite, and within both sums' rounding of the clean ones."""
    N, H, M = 400, 160, 40
    plan = melt.MeltPlan(sample_rate=16000, n_fft=N, hop=H, n_mels=M, output=melt.MELT_OUT_POWER)
    wave, off = workloads.random_clips([200 * H + N, 40 * H + N], seed=6)
    T = melt.total_frames(off, N, H)
    d_wave, d_off = torch.from_numpy(wave).cuda(), torch.from_numpy(off).cuda()
    proj = torch.empty((T, 2 * M), device="cuda")
    plan.forward(d_wave, d_off, T, proj=proj)
    g = torch.randn((T, M), generator=torch.Generator().manual_seed(1))
    g[50, 7] = 0.0
    gw0, gb0 = (x.cpu().numpy() for x in plan.backward(d_wave, d_off, T, g.cuda(), proj=proj))
    g[50, 7] = bad
    gw, gb = (x.cpu().numpy() for x in plan.backward(d_wave, d_off, T, g.cuda(), proj=proj))
    hit = np.zeros(wave.size, bool)
    hit[50 * H:50 * H + N] = True
    last = np.zeros(wave.size, bool)
    last[50 * H + N:53 * H] = True
    assert np.array_equal(gw[~hit & ~last], gw0[~hit & ~last])
    W, P = plan.basis(), proj.cpu().numpy()
    G = 2 * P.astype(np.float64) * np.repeat(g.double().numpy(), 2, axis=1)
    G[50, 14:16] = 0.0
    Wq = np.abs(W.reshape(2, M, N).transpose(1, 0, 2).reshape(2 * M, N).astype(np.float64))      # interleaved rows
    mass = np.array([sum(np.abs(G[t]) @ Wq[:, s - t * H] for t in range(50, 53) if t * H <= s < t * H + N)
                     for s in np.flatnonzero(last)])
    terms = 2 * M * 3 + 3
    assert np.all(np.abs(gw[last].astype(np.float64) - gw0[last]) <= 2 * terms * 2.0 ** -24 * (1 + 1e-3) * mass)
    rows = np.zeros(2 * M, bool)
    rows[[7, M + 7]] = True
    assert np.array_equal(gb[~rows], gb0[~rows])
    # G of the bin is inf (sign of R, I) or NaN; a product with it is inf, or NaN where the weight is 0
    with np.errstate(invalid="ignore"):
        gr, gi = np.float32(2) * P[50, 14] * np.float32(bad), np.float32(2) * P[50, 15] * np.float32(bad)
        want_w = gr * W[7] + gi * W[M + 7]
        want_b = np.stack([gr * wave[50 * H:50 * H + N], gi * wave[50 * H:50 * H + N]])
    for got, want in ((gw[hit], want_w), (gb[rows], want_b)):
        assert np.array_equal(np.isnan(got), np.isnan(want))
        inf = np.isinf(want)
        assert np.array_equal(np.isinf(got), inf) and np.array_equal(got[inf], want[inf])
