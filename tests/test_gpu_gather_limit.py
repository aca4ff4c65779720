"""Pushes on both sides of the stream count where one launch gathers and two do."""
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


@pytest.mark.parametrize("n_streams,kernels", [(1536, ["k_stream_gather"]), (1537, ["k_stream_pack", "k_stream_copy"])])
def test_gather(torch, melt, n_streams, kernels):
    plan = melt.MeltPlan(sample_rate=16000, n_fft=256, hop=128, n_mels=16)
    X = torch.randn(n_streams, 6 * 150, generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    off = torch.arange(n_streams + 1, dtype=torch.int64, device="cuda") * X.shape[1]
    T = melt.total_frames(np.arange(n_streams + 1) * X.shape[1], 256, 128)
    ref = plan.forward(X.reshape(-1), off, T).view(n_streams, -1, 16)
    st = melt.MeltStream(plan, n_streams, 150)
    names = kernels_of(torch, melt, lambda: melt.melt_stream_push(st.handle, X[:, :150].contiguous(), st.out, st.count))
    assert [k for k in ("k_stream_gather", "k_stream_pack", "k_stream_copy") if any(k in n for n in names)] == kernels
    at = 0
    for k in range(6):
        out, cnt = st.push(X[:, 150 * k:150 * (k + 1)].contiguous())
        n = int(cnt[0])
        assert bool((cnt == n).all()) and torch.equal(out[:, :n], ref[:, at:at + n])
        at += n
    assert at == ref.shape[1]
