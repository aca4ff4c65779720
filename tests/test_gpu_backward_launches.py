"""The launches of a backward that recomputes its projections."""
import numpy as np
import pytest

import workloads
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


@pytest.mark.parametrize("clips,tables", [(64, 0), (65, 1)])
@pytest.mark.parametrize("prec", ["fp32", "bf16", "fp8"])
def test_one_chunk_table(torch, melt, prec, clips, tables):
    """More than 64 clips: the forward's chunk table also serves the frame starts; the gradients are
    those with the projections passed in."""
    plan = melt.MeltPlan(sample_rate=16000, n_fft=400, hop=160, n_mels=40, precision=prec)
    lengths = np.random.default_rng(clips).integers(0, 40 * 160 + 400, clips)
    wave, off = workloads.random_clips(lengths, seed=1)
    T = melt.total_frames(off, 400, 160)
    wave, off = torch.from_numpy(wave).cuda(), torch.from_numpy(off).cuda()
    g = torch.randn((T, 40), generator=torch.Generator().manual_seed(2)).cuda()
    gw, gb, proj = torch.empty_like(wave), torch.empty((80, 400), device="cuda"), torch.empty((T, 80), device="cuda")
    run = lambda: melt.melt_backward(plan.handle, wave, off, T, g, None, gw, gb)
    run()
    names = kernels_of(torch, melt, run)
    assert sum("k_schedule" in n and "rows" not in n for n in names) == tables
    plan.forward(wave, off, T, proj=proj)
    want = plan.backward(wave, off, T, g, proj=proj)
    assert torch.equal(gw, want[0]) and torch.equal(gb, want[1])
