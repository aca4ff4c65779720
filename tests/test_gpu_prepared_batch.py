"""Which batch is the plan's prepared one after a call: the last forward's or backward's, whether its
kernel read a chunk table or found its own chunks; and the noalloc forward leaves it alone."""
import numpy as np
import pytest

import workloads
from tests.hip_graph import kernels_of

pytestmark = pytest.mark.gpu

SPEECH, SYSTEMS, LONG, CEPSTRAL = (16000, 400, 160, 80), (16000, 512, 128, 128), (22050, 1024, 256, 128), (16000, 1200, 160, 128)


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


class _Batch:
    def __init__(self, torch, melt, plan, lengths, seed):
        wave, off = workloads.random_clips(lengths, seed=seed)
        self.T = melt.total_frames(off, plan.n_fft, plan.hop)
        self.wave, self.off = torch.from_numpy(wave).cuda(), torch.from_numpy(off).cuda()

    def out(self, torch, plan):
        return torch.full((self.T, plan.n_mels), float("nan"), device="cuda")


def _two(torch, melt, plan, clips):
    """Two batches of the same clip count and frame count, laid out differently."""
    N, H = plan.n_fft, plan.hop
    r = np.random.default_rng(clips)
    frames = r.integers(1, 300, clips)
    a = frames * H + N - H
    b = a[::-1].copy()
    b[0] += 3
    return _Batch(torch, melt, plan, a, 1), _Batch(torch, melt, plan, b, 2)


CASES = [("fp32", SPEECH, None), ("bf16", SPEECH, None), ("bf16", SYSTEMS, None), ("bf16", LONG, None), ("bf16", CEPSTRAL, None),
         ("bf16x3", SPEECH, None), ("bf16x3", SPEECH, "h16-row-split-lds-dma-bf96"), ("fp16x3", LONG, None), ("fp8", SPEECH, None),
         ("fp8", SPEECH, "f8-frame-split"), ("fp8b", SPEECH, None), ("stft", SPEECH, None), ("stft", LONG, None)]


@pytest.mark.parametrize("clips", [1, 7, 64, 65])
@pytest.mark.parametrize("prec,geom,variant", CASES)
def test_the_last_forward_is_prepared(torch, melt, prec, geom, variant, clips):
    sr, N, H, M = geom
    plan = melt.MeltPlan(sample_rate=sr, n_fft=N, hop=H, n_mels=M, precision="fp32" if prec == "stft" else prec)
    if variant:
        names = [melt.melt_variant_name(plan.handle, v) for v in range(melt.melt_variant_count(plan.handle))]
        melt.melt_set_variant(plan.handle, next(v for v, n in enumerate(names) if n.startswith(variant)), 0)
    forward = plan.stft_mel if prec == "stft" else plan.forward
    prepared = melt.stft_mel_forward_prepared if prec == "stft" else melt.melt_forward_prepared
    a, b = _two(torch, melt, plan, clips)

    def again(batch):
        out = batch.out(torch, plan)
        prepared(plan.handle, batch.wave, out)
        return out

    # on a plan that has prepared nothing
    want_a = forward(a.wave, a.off, a.T, out=a.out(torch, plan))
    assert torch.equal(again(a), want_a)
    # over an earlier prepared batch of the same size
    melt.melt_batch_prepare(plan.handle, a.off, a.T)
    want_b = forward(b.wave, b.off, b.T, out=b.out(torch, plan))
    got_b = again(b)
    assert not torch.isnan(want_b).any() and torch.equal(got_b, want_b)
    # the chunk table that the forward left is the one that a prepare makes
    melt.melt_batch_prepare(plan.handle, b.off, b.T)
    assert torch.equal(again(b), want_b)


@pytest.mark.parametrize("clips", [3, 65])
def test_after_a_backward(torch, melt, clips):
    plan = melt.MeltPlan(sample_rate=16000, n_fft=400, hop=160, n_mels=80)
    a, b = _two(torch, melt, plan, clips)
    proj = torch.empty((b.T, 160), device="cuda")
    want = plan.forward(b.wave, b.off, b.T, proj=proj)
    melt.melt_batch_prepare(plan.handle, a.off, a.T)
    plan.backward(b.wave, b.off, b.T, torch.ones_like(want), proj=proj)
    got = b.out(torch, plan)
    melt.melt_forward_prepared(plan.handle, b.wave, got)
    assert torch.equal(got, want)


def test_the_noalloc_forward_leaves_it(torch, melt):
    plan = melt.MeltPlan(sample_rate=16000, n_fft=400, hop=160, n_mels=80)
    a, b = _two(torch, melt, plan, 5)
    want = plan.forward(a.wave, a.off, a.T)
    melt.melt_forward_noalloc(plan.handle, b.wave, b.off, b.T, b.out(torch, plan))
    got = a.out(torch, plan)
    melt.melt_forward_prepared(plan.handle, a.wave, got)
    assert torch.equal(got, want)


def test_a_capture_that_cannot_grow_the_table(torch, melt):
    """A large call that finds its own chunks, captured before the plan's table is large enough to
    take them: it is still one kernel, and no batch is prepared."""
    plan = melt.MeltPlan(sample_rate=16000, n_fft=400, hop=160, n_mels=8)
    T = 62 * 256 * 128
    d_off = torch.tensor([0, (T - 1) * 160 + 400], dtype=torch.int64, device="cuda")
    x = torch.empty(1, device="cuda")                   # captured, never run
    names = kernels_of(torch, melt, lambda: melt.melt_forward(plan.handle, x, d_off, T, x))
    assert len(names) == 1 and "k_melt_split" in names[0]
    with pytest.raises(melt.MeltError):
        melt.melt_forward_prepared(plan.handle, x, x)
