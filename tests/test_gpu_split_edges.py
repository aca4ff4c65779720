"""Where the split-plane forward stops being a plan's default: frames of few samples with few Mel bins.
Both sides of each edge, against the oracle."""
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


@pytest.mark.parametrize("prec,N,H,M,planes", [
    ("fp32", 127, 64, 16, False), ("fp32", 128, 64, 16, True), ("fp32", 127, 64, 17, True), ("fp32", 40, 20, 8, False),
    ("bf16x3", 127, 64, 16, False), ("bf16x3", 128, 64, 16, True), ("bf16x3", 64, 64, 16, True), ("bf16x3", 63, 63, 40, False),
    ("bf16x3", 63, 63, 41, True), ("fp16x3", 40, 20, 16, False), ("fp16x3", 48, 48, 16, True), ("fp16x3", 40, 20, 17, True)])
def test_default(torch, melt, orc, prec, N, H, M, planes):
    plan = melt.MeltPlan(sample_rate=16000, n_fft=N, hop=H, n_mels=M, precision=prec)
    names = [melt.melt_variant_name(plan.handle, v) for v in range(melt.melt_variant_count(plan.handle))]
    assert ("split-planes" in names[0]) == planes
    at = next(v for v, n in enumerate(names) if "split-planes" in n)        # it can still be chosen
    wave, off = workloads.random_clips([300 * H + N, N - 1, N, 5 * H + N + 1], seed=M)
    for v in {0, at}:
        melt.melt_set_variant(plan.handle, v, 0)
        L, _ = _gpu_forward(torch, melt, plan, wave, off)
        _check(orc, melt, plan, L, wave, off, prec, label=f"{prec} {N} {H} {M} {names[v]}")


# front end, clips, frames each -> (frame tiles, row tiles, frame groups) of a multiply wave, as every shape timed
SHAPES = [((400, 160, 80), 32, 998, (4, 5, 2)), ((400, 160, 80), 16, 998, (4, 3, 1)), ((400, 160, 80), 64, 2998, (4, 5, 2)),
          ((400, 160, 80), 1, 98, (1, 2, 2)), ((120, 40, 24), 16, 3998, (4, 2, 2)), ((1024, 256, 128), 16, 122, (1, 2, 2)),
          ((480, 161, 64), 16, 196, (1, 2, 2)), ((400, 160, 40), 16, 198, (1, 2, 2))]


@pytest.mark.parametrize("geom,clips,frames,shape", SHAPES)
def test_shape(torch, melt, geom, clips, frames, shape):
    from tests.hip_graph import kernels_of
    N, H, M = geom
    plan = melt.MeltPlan(sample_rate=16000, n_fft=N, hop=H, n_mels=M)
    off = torch.zeros(clips + 1, dtype=torch.int64, device="cuda")      # captured, never run
    x = torch.empty(1, device="cuda")
    names = kernels_of(torch, melt, lambda: melt.melt_forward(plan.handle, x, off, clips * frames, x))
    want = "Li%dELi%dELi%dE" % shape
    assert any("k_melt_split" in n and want in n for n in names), names


@pytest.mark.parametrize("geom,frames", [((480, 161, 64), 41154), ((480, 160, 64), 41403)])
def test_shape_of_mixed_lengths(torch, melt, geom, frames):
    """61 clips of 0.5 to 12 s: 64-frame items of all rows are 14 % faster than 128-frame ones."""
    from tests.hip_graph import kernels_of
    N, H, M = geom
    plan = melt.MeltPlan(sample_rate=16000, n_fft=N, hop=H, n_mels=M)
    off = torch.zeros(62, dtype=torch.int64, device="cuda")             # captured, never run
    x = torch.empty(1, device="cuda")
    names = kernels_of(torch, melt, lambda: melt.melt_forward(plan.handle, x, off, frames, x))
    assert any("k_melt_split" in n and "Li4ELi2ELi1E" in n for n in names), names
