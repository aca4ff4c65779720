"""A plan packs its basis only into layouts that one of its kernels reads."""
import pytest

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


@pytest.mark.parametrize("prec", ["fp32", "bf16x3"])
def test_no_planes_without_their_kernel(torch, melt, prec):
    """N 1024 at hop 1 and 512 Mel bins: the split-plane forward would pad every hop of one sample to 32
    and is not among the variants; its planes alone would be 64 tiles x 1024 groups x P KB."""
    melt.MeltPlan(sample_rate=16000, n_fft=400, hop=160, n_mels=8, precision=prec).close()      # what the first plan holds
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    plan = melt.MeltPlan(sample_rate=16000, n_fft=1024, hop=1, n_mels=512, precision=prec)
    used = before - torch.cuda.mem_get_info()[0]
    assert not any("split-planes" in melt.melt_variant_name(plan.handle, v) for v in range(melt.melt_variant_count(plan.handle)))
    planes = 64 * 1024 * (3 if prec == "fp32" else 2) << 10
    # row tiles of 32: FP32 and two 16-bit layouts of k-groups of 8 and 16 samples (one a hop), E4M3, and
    # the backward's fragments of one column tile; a few MB of tables
    layouts = (32 * 1024 + 2 * 32 * 1024 + 32 * 16 * 2 + 1024 * 128) << 10
    plan.close()
    assert used < layouts + planes // 4
