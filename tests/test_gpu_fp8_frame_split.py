"""The frame-split FP8 kernel against the row-split one, bit for bit: the two quantise the same
frames with the same scales and add the same products in the same order."""
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


@pytest.mark.parametrize("M", [1, 16, 17, 40, 64, 80, 96, 100, 128])
@pytest.mark.parametrize("N,H", [(400, 160), (512, 128), (256, 128), (250, 32), (500, 96), (448, 160)])
def test_equals_the_row_split_kernel(torch, melt, orc, N, H, M):
    """One to eight row tiles (basis in LDS and streamed), 4, 7 and 8 k-groups, frames that end
    inside a block of 32 and inside a vector of 4; clips that end chunks of 128 frames exactly,
    one past and mid-way, and more chunks than compute units."""
    plan = melt.MeltPlan(sample_rate=16000, n_fft=N, hop=H, n_mels=M, precision="fp8")
    names = [melt.melt_variant_name(plan.handle, v) for v in range(melt.melt_variant_count(plan.handle))]
    assert names[0].startswith("f8-frame-split")
    other = next(v for v, n in enumerate(names) if n.startswith("f8-row-split"))
    lengths = [N - 1, N, N + 3, 127 * H + N, 128 * H + N + 1, 33 * H + N, 300 * 128 * H + N]
    wave, off = workloads.random_clips(lengths, seed=M + N)
    wave[: N - 1 + N] = 0.0                    # a silent frame
    melt.melt_set_variant(plan.handle, 0, 0)
    got, _ = _gpu_forward(torch, melt, plan, wave, off)
    melt.melt_set_variant(plan.handle, other, 0)
    want, _ = _gpu_forward(torch, melt, plan, wave, off)
    assert np.array_equal(got, want)


def test_not_pinned_small_and_large_calls_agree(torch, melt, orc):
    """The plan's own choice (row-split for a small call, frame-split for a large one)."""
    plan = melt.MeltPlan(sample_rate=16000, n_fft=400, hop=160, n_mels=80, precision="fp8")
    wave, off = workloads.random_clips([400 + 160 * 200] * 100, seed=2)
    many, _ = _gpu_forward(torch, melt, plan, wave, off)
    one, _ = _gpu_forward(torch, melt, plan, wave[:off[1]].copy(), off[:2])
    assert np.array_equal(many[:201], one)
    _check(orc, melt, plan, one, wave[:off[1]], off[:2], "fp8", label="small call")
