"""Kernels that find their own chunks (calls of at most 64 clips) against the same kernels over a
prepared chunk table: bit for bit, over clip counts, empty and short clips, and batches at and
beyond the size where a workgroup's chunk list is full."""
import numpy as np
import pytest

import workloads

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


def _both(torch, melt, plan, wave, off, stft):
    T = melt.total_frames(off, plan.n_fft, plan.hop)
    d_wave = torch.from_numpy(wave).cuda() if isinstance(wave, np.ndarray) else wave
    d_off = torch.from_numpy(np.asarray(off, np.int64)).cuda()
    a, b = (torch.full((T, plan.n_mels), float("nan"), device="cuda") for _ in range(2))
    melt.melt_batch_prepare(plan.handle, d_off, T)
    (plan.stft_mel if stft else plan.forward)(d_wave, d_off, T, out=a)
    # the batch prepared before the self-scheduled call is still the plan's
    (melt.stft_mel_forward_prepared if stft else melt.melt_forward_prepared)(plan.handle, d_wave, b)
    torch.cuda.synchronize()
    assert not torch.isnan(a).any()
    assert torch.equal(a, b)


@pytest.mark.parametrize("n_clips", [1, 2, 63, 64])
@pytest.mark.parametrize("prec,geom", [("fp32", SPEECH), ("bf16", SPEECH), ("bf16", SYSTEMS), ("bf16", LONG), ("bf16", CEPSTRAL),
                                       ("fp16", SYSTEMS), ("bf16x3", SPEECH), ("fp16x3", LONG), ("fp8", SPEECH),
                                       ("fp8b", SPEECH), ("stft", SPEECH), ("stft", LONG)])
def test_equals_the_prepared_batch(torch, melt, prec, geom, n_clips):
    sr, N, H, M = geom
    plan = melt.MeltPlan(sample_rate=sr, n_fft=N, hop=H, n_mels=M, precision="fp32" if prec == "stft" else prec)
    r = np.random.default_rng(n_clips)
    lengths = r.integers(0, 4 * N + 140 * H, n_clips)
    lengths[::5] = np.minimum(lengths[::5], N - 1)          # clips without a frame
    lengths[-1] = 260 * H + N + 1
    wave, off = workloads.random_clips(lengths, seed=n_clips)
    _both(torch, melt, plan, wave, off, prec == "stft")


@pytest.mark.parametrize("prec", ["fp32", "bf16", "fp8", "fp8b", "stft"])
@pytest.mark.parametrize("chunks", [64 * 256 - 4, 64 * 256 + 4])
def test_full_chunk_lists(torch, melt, prec, chunks):
    """Chunks (of the kernel's own size) for 64 per workgroup of 256 and a few more or less."""
    sr, N, H, M = 16000, 400, 160, 16
    plan = melt.MeltPlan(sample_rate=sr, n_fft=N, hop=H, n_mels=M, precision="fp32" if prec == "stft" else prec)
    bf = 6 if prec == "stft" else int(melt.melt_variant_name(plan.handle, 0).rsplit("bf", 1)[1])
    L = (chunks // 3 * bf - 1) * H + N
    gen = torch.Generator(device="cuda").manual_seed(3)
    wave = torch.randn(3 * L, generator=gen, device="cuda")
    _both(torch, melt, plan, wave, np.arange(4) * L, prec == "stft")
