"""The largest call whose kernel finds its own chunks, for every kernel that does: its lists and rings are
full, to the last entry, and its rows are bit for bit those over a chunk table; one frame more is a
table's.  Which of the two a call takes is read from its launches."""
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


# precision, geometry, variant (None: the plan's), entries a workgroup can hold, workgroups that share a chunk
CASES = [("fp32", (16000, 400, 160, 16), None, 63, 1), ("fp32", (16000, 400, 160, 136), None, 63, 2),
         ("fp16x3", (16000, 512, 128, 16), None, 63, 1),
         ("bf16", (16000, 400, 160, 16), None, 64, 1), ("bf16x3", (16000, 400, 160, 16), None, 64, 1),
         ("fp8b", (16000, 400, 160, 16), None, 64, 1), ("fp8", (16000, 400, 160, 16), "f8-frame-split", 64, 1),
         ("fp8", (16000, 400, 160, 16), "f8-row-split-lds-dma-bf128", 32, 1), ("bf16", (16000, 512, 128, 16), None, 32, 1),
         ("bf16", (16000, 400, 160, 16), "h16-row-split-lds-dma-bf64", 32, 1),
         ("bf16", (22050, 1024, 256, 16), None, 32, 1), ("bf16", (16000, 1200, 160, 72), None, 32, 2),
         ("stft", (16000, 400, 160, 16), None, 8, 1), ("stft", (16000, 512, 128, 16), None, 8, 1)]


@pytest.mark.parametrize("prec,geom,variant,entries,share", CASES)
def test_full(torch, melt, prec, geom, variant, entries, share):
    sr, N, H, M = geom
    plan = melt.MeltPlan(sample_rate=sr, n_fft=N, hop=H, n_mels=M, precision="fp32" if prec == "stft" else prec)
    names = [melt.melt_variant_name(plan.handle, v) for v in range(melt.melt_variant_count(plan.handle))]
    v = 0 if variant is None else next(i for i, n in enumerate(names) if n.startswith(variant))
    if variant:
        melt.melt_set_variant(plan.handle, v, 0)
    call = plan.stft_mel if prec == "stft" else plan.forward
    prepared = melt.stft_mel_forward_prepared if prec == "stft" else melt.melt_forward_prepared
    bf = None if prec == "stft" else int(names[v].rsplit("bf", 1)[1])
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    x, clips = torch.empty(1, device="cuda"), 3
    most = 16 << 20
    zeros = torch.zeros(clips + 1, dtype=torch.int64, device="cuda")
    melt.melt_batch_prepare(plan.handle, zeros, most)                   # tables that no capture has to grow

    def finds(T):
        return not any("k_schedule" in n for n in kernels_of(torch, melt, lambda: call(x, zeros, T, out=x)))

    lo, hi = 1, most
    assert finds(lo) and not finds(hi)
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (mid, hi) if finds(mid) else (lo, mid)
    # lo: the most frames of three clips.  Clips of whole chunks, so that the chunks are nearly as many as
    # the rule allows for: beyond the last but one entry of a workgroup's list
    step = bf or 2 * {400: 3, 512: 4}[N] * 8
    each = lo // clips // step * step
    T = clips * each
    if bf:
        assert T // bf > (entries - 1) * cus // share
    else:
        assert T >= (entries - 1) * 4 * cus
    assert finds(T)
    off = np.arange(clips + 1, dtype=np.int64) * ((each - 1) * H + N)
    d_off = torch.from_numpy(off).cuda()
    wave = torch.randn(int(off[-1]), generator=torch.Generator(device="cuda").manual_seed(3), device="cuda")
    own, table = (torch.full((T, M), float("nan"), device="cuda") for _ in range(2))
    call(wave, d_off, T, out=own)
    melt.melt_batch_prepare(plan.handle, d_off, T)
    prepared(plan.handle, wave, table)
    assert not torch.isnan(own).any() and torch.equal(own, table)
