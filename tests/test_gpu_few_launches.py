"""The single-launch forms of the backward's tables and of a push's gathering, against the forms
they replace, which larger calls still take: more than 64 clips, more than 2048 streams."""
import numpy as np
import pytest

import workloads

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


@pytest.mark.parametrize("clips", [1, 5, 64])
@pytest.mark.parametrize("N,H,M", [(400, 160, 80), (512, 128, 24), (300, 33, 17)])
def test_backward_of_few_clips_equals_that_of_many(torch, melt, clips, N, H, M):
    """The same clips followed by empty ones up to 65: d/dwave and d/dbasis bit for bit (empty
    clips, clips without a frame, clips of several row chunks)."""
    plan = melt.MeltPlan(sample_rate=16000, n_fft=N, hop=H, n_mels=M)
    r = np.random.default_rng(clips + N)
    lengths = r.integers(0, 140 * H + 2 * N, clips)
    lengths[::7] = np.minimum(lengths[::7], N - 1)
    lengths[-1] = 300 * H + N + 5
    wave, off = workloads.random_clips(lengths, seed=clips)
    T = melt.total_frames(off, N, H)
    d_wave = torch.from_numpy(wave).cuda()
    g = torch.randn((T, M), generator=torch.Generator().manual_seed(2)).cuda()
    proj = torch.empty((T, 2 * M), device="cuda")
    few = torch.from_numpy(off).cuda()
    many = torch.from_numpy(np.concatenate([off, np.full(65 - clips, off[-1])])).cuda()
    plan.forward(d_wave, few, T, proj=proj)
    a = plan.backward(d_wave, few, T, g, proj=proj)
    b = plan.backward(d_wave, many, T, g, proj=proj)
    c = plan.backward(d_wave, few, T, g, proj=None)
    for x, y, z in zip(a, b, c):
        assert torch.equal(x, y) and torch.equal(x, z)


@pytest.mark.parametrize("n_streams", [1, 255, 257, 2048, 2049])
def test_pushes_equal_the_batch(torch, melt, n_streams):
    plan = melt.MeltPlan(sample_rate=16000, n_fft=256, hop=128, n_mels=16)
    r = np.random.default_rng(n_streams)
    X = (0.3 * r.standard_normal((n_streams, 6 * 150))).astype(np.float32)
    off = np.arange(n_streams + 1, dtype=np.int64) * X.shape[1]
    T = melt.total_frames(off, 256, 128)
    ref = plan.forward(torch.from_numpy(X.reshape(-1)).cuda(), torch.from_numpy(off).cuda(), T).view(n_streams, -1, 16)
    st = melt.MeltStream(plan, n_streams, 150)
    at = 0
    for k in range(6):
        out, cnt = st.push(torch.from_numpy(np.ascontiguousarray(X[:, 150 * k:150 * (k + 1)])).cuda())
        n = int(cnt[0])
        assert bool((cnt == n).all())
        assert torch.equal(out[:, :n], ref[:, at:at + n])
        at += n
    assert at == ref.shape[1]
