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
