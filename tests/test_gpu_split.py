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
