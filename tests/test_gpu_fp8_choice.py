"""Which FP8 kernel a call, a prepared batch, a push or the noalloc forward takes: the row-split one where
calls are small or their clips short, the frame-split one otherwise, with the same bits."""
import numpy as np
import pytest

from tests.hip_graph import kernels_of

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


def _plan(melt, M):
    plan = melt.MeltPlan(sample_rate=16000, n_fft=400, hop=160, n_mels=M, precision="fp8")
    assert melt.melt_variant_name(plan.handle, 0).startswith("f8-frame-split")
    return plan


def _batch(torch, clips, frames):
    off = np.arange(clips + 1, dtype=np.int64) * ((frames - 1) * 160 + 400)
    wave = torch.randn(int(off[-1]), generator=torch.Generator(device="cuda").manual_seed(clips), device="cuda")
    return wave, torch.from_numpy(off).cuda(), clips * frames


def _fp8(names):
    return [n for n in names if "k_melt_f8" in n][0]


# (Mel bins, clips, frames each) -> frame-split
CHOICES = [(80, 1, 98, False), (80, 16, 398, False), (80, 64, 2998, True), (80, 65, 98, False), (80, 512, 28, False),
           (80, 256, 98, False), (80, 512, 98, True), (80, 256, 398, True), (128, 512, 28, False), (128, 256, 98, False), (128, 100, 298, True), (128, 600, 256, True),
           (128, 64, 1000, True), (40, 1, 98, True), (40, 256, 28, False), (40, 256, 98, True), (16, 512, 8, False),
           (16, 512, 28, True), (16, 1, 98, True)]


@pytest.mark.parametrize("M,clips,frames,split", CHOICES)
def test_calls_and_prepared_batches(torch, melt, M, clips, frames, split):
    plan = _plan(melt, M)
    wave, off, T = _batch(torch, clips, frames)
    out, prep, noalloc, pinned = (torch.full((T, M), float("nan"), device="cuda") for _ in range(4))
    name = "k_melt_f8_fs" if split else "k_melt_f8_as"
    assert name in _fp8(kernels_of(torch, melt, lambda: plan.forward(wave, off, T, out=out)))
    plan.forward(wave, off, T, out=out)
    melt.melt_batch_prepare(plan.handle, off, T)
    assert name in _fp8(kernels_of(torch, melt, lambda: melt.melt_forward_prepared(plan.handle, wave, prep)))
    melt.melt_forward_prepared(plan.handle, wave, prep)
    assert name in _fp8(kernels_of(torch, melt, lambda: melt.melt_forward_noalloc(plan.handle, wave, off, T, noalloc)))
    melt.melt_forward_noalloc(plan.handle, wave, off, T, noalloc)
    melt.melt_set_variant(plan.handle, 0, 0)
    assert "k_melt_f8_fs" in _fp8(kernels_of(torch, melt, lambda: plan.forward(wave, off, T, out=pinned)))
    plan.forward(wave, off, T, out=pinned)
    assert torch.equal(out, pinned) and torch.equal(prep, pinned) and torch.equal(noalloc, pinned)


@pytest.mark.parametrize("M,streams,chunk,split", [(80, 1, 160, False), (80, 16, 1600, False), (80, 2048, 1600, True),
                                                   (40, 1, 160, False), (40, 16, 1600, True)])
def test_pushes(torch, melt, M, streams, chunk, split):
    plan = _plan(melt, M)
    st = melt.MeltStream(plan, streams, chunk)
    x = torch.randn(streams, chunk, device="cuda")
    names = kernels_of(torch, melt, lambda: melt.melt_stream_push(st.handle, x, st.out, st.count))
    assert ("k_melt_f8_fs" if split else "k_melt_f8_as") in _fp8(names)


def test_a_failed_autotune_pins_nothing(torch, melt):
    """A batch that no GPU holds: the run is refused, the plan chooses by call as before, and the next
    launch does not report the failed allocation."""
    plan = _plan(melt, 80)
    wave, off, T = _batch(torch, 1, 98)
    out = torch.empty((T, 80), device="cuda")
    with pytest.raises(melt.MeltError) as e:
        melt.melt_autotune(plan.handle, 4 * 10 ** 9)
    assert e.value.status == melt.MELT_E_NO_MEMORY
    assert "k_melt_f8_as" in _fp8(kernels_of(torch, melt, lambda: plan.forward(wave, off, T, out=out)))
    plan.forward(wave, off, T, out=out)
    torch.cuda.synchronize()
