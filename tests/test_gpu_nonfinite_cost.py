"""Non-finite samples and gradients: what comes of them, and that the plain FP32 arithmetic which they
are recomputed with takes a bounded multiple of a call without them."""
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


def _ms(torch, call):
    """The shortest of three calls after a first one, in ms."""
    call()
    times = []
    for _ in range(3):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        call()
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b))
    return min(times)


def _setup(torch, melt, geom, clips, seconds, **kw):
    sr, N, H, M = geom
    plan = melt.MeltPlan(sample_rate=sr, n_fft=N, hop=H, n_mels=M, **kw)
    L = int(seconds * sr)
    off = np.arange(clips + 1, dtype=np.int64) * L
    gen = torch.Generator(device="cuda").manual_seed(1)
    wave = torch.randn(clips * L, generator=gen, device="cuda")
    return plan, wave, torch.from_numpy(off).cuda(), melt.total_frames(off, N, H), gen


# FP32 matrix cores take 2.7 times as long as the six plane products, which are taken first
COST = 8.0


@pytest.mark.parametrize("bad", ["one", "all"])
@pytest.mark.parametrize("geom,clips,seconds", [((16000, 400, 160, 80), 16, 10.0), ((22050, 1024, 256, 128), 32, 10.0)])
def test_cost_of_d_dbasis(torch, melt, geom, clips, seconds, bad):
    plan, wave, off, T, gen = _setup(torch, melt, geom, clips, seconds)
    proj = torch.empty((T, 2 * plan.n_mels), device="cuda")
    plan.forward(wave, off, T, proj=proj)
    g = torch.randn((T, plan.n_mels), generator=gen, device="cuda")
    gb = torch.empty((2 * plan.n_mels, plan.n_fft), device="cuda")
    run = lambda: melt.melt_backward(plan.handle, wave, off, T, g, proj, None, gb)
    clean = _ms(torch, run)
    g[7 if bad == "one" else slice(None), 3 if bad == "one" else slice(None)] = float("nan")
    dirty = _ms(torch, run)
    print(f"\nd/dbasis {geom} {bad}: {clean:.3f} -> {dirty:.3f} ms")
    assert torch.isnan(gb).any() and dirty < COST * clean


@pytest.mark.parametrize("bad", ["one", "all"])
@pytest.mark.parametrize("geom,clips,seconds", [((16000, 400, 160, 80), 64, 30.0), ((22050, 1024, 256, 128), 32, 10.0),
                                                ((16000, 400, 160, 16), 1, 1.0)])
def test_cost_of_a_forward(torch, melt, geom, clips, seconds, bad):
    plan, wave, off, T, _ = _setup(torch, melt, geom, clips, seconds)
    out = torch.empty((T, plan.n_mels), device="cuda")
    run = lambda: plan.forward(wave, off, T, out=out)
    clean = _ms(torch, run)
    wave[12345 if bad == "one" else slice(None)] = float("nan")
    dirty = _ms(torch, run)
    print(f"\nforward {geom} {bad}: {clean:.3f} -> {dirty:.3f} ms")
    assert torch.isnan(out).any() and dirty < COST * clean


@pytest.mark.parametrize("bad", ["one", "all"])
@pytest.mark.parametrize("geom,clips,seconds", [((16000, 400, 160, 80), 16, 10.0), ((22050, 1024, 256, 128), 32, 10.0)])
def test_cost_of_d_dwave(torch, melt, geom, clips, seconds, bad):
    plan, wave, off, T, gen = _setup(torch, melt, geom, clips, seconds)
    proj = torch.empty((T, 2 * plan.n_mels), device="cuda")
    plan.forward(wave, off, T, proj=proj)
    g = torch.randn((T, plan.n_mels), generator=gen, device="cuda")
    gw = torch.empty_like(wave)
    run = lambda: melt.melt_backward(plan.handle, wave, off, T, g, proj, gw, None)
    clean = _ms(torch, run)
    g[7 if bad == "one" else slice(None), 3 if bad == "one" else slice(None)] = float("nan")
    dirty = _ms(torch, run)
    print(f"\nd/dwave {geom} {bad}: {clean:.3f} -> {dirty:.3f} ms")
    assert torch.isnan(gw).any() and dirty < COST * clean


@pytest.mark.parametrize("frames", [20, 3000])
@pytest.mark.parametrize("N,H,M", [(400, 160, 1), (400, 160, 8), (400, 160, 13), (400, 160, 24), (400, 160, 80), (480, 161, 40),
                                   (400, 50, 64), (1024, 256, 128), (401, 160, 100), (512, 128, 200), (400, 160, 512)])
def test_values_of_a_forward(torch, melt, N, H, M, frames):
    """Samples of 2^110, beyond what the planes hold, in some frames, at every count of row tiles a
    wave: their projections are within FP32's rounding of the 64-bit ones (2 N steps of 2^-24 of the
    terms' sum: products and sums), all others' are bit for bit as without them."""
    plan = melt.MeltPlan(sample_rate=16000, n_fft=N, hop=H, n_mels=M, output=melt.MELT_OUT_LOG_MAGNITUDE)
    assert "split-planes" in melt.melt_variant_name(plan.handle, 0)
    wave, off = workloads.random_clips([frames * H + N, 2 * H + N + 1], seed=M)
    T = melt.total_frames(off, N, H)
    d_off = torch.from_numpy(off).cuda()

    def run():
        proj, out = torch.empty((T, 2 * M), device="cuda"), torch.empty((T, M), device="cuda")
        plan.forward(torch.from_numpy(wave).cuda(), d_off, T, out=out, proj=proj)
        return out.cpu().numpy(), proj.cpu().numpy()

    clean_out, clean = run()
    at = [5, 3 * H + 7, (frames // 2) * H + N - 1, off[-1] - 1]
    wave[at] = 2.0 ** 110
    out, got = run()
    starts = np.concatenate([np.arange(a, b - N + 1, H) for a, b in zip(off[:-1], off[1:])])
    hit = np.zeros(T, bool)
    for p in at:
        hit |= (starts <= p) & (p < starts + N)
    # (frames that meet such a sample with zero weights alone are recomputed too)
    near = np.zeros(T, bool)
    for p in at:
        near |= (starts <= p) & (p < starts + -(-N // H) * H + 32)
    assert np.array_equal(got[~near], clean[~near]) and np.array_equal(out[~near], clean_out[~near])
    W = plan.basis().astype(np.float64).reshape(2, M, N).transpose(1, 0, 2).reshape(2 * M, N)
    X = wave[starts[near][:, None] + np.arange(N)].astype(np.float64)
    want, mass = X @ W.T, np.abs(X) @ np.abs(W).T
    assert np.all(np.abs(got[near] - want) <= 2 * N * 2.0 ** -24 * mass)
    assert np.all(np.isfinite(out[near & ~hit]))


@pytest.mark.parametrize("frames", [20, 3000])
@pytest.mark.parametrize("N,H,M", [(400, 160, 40), (401, 16, 17), (300, 33, 9), (512, 128, 100), (250, 250, 24), (400, 160, 5)])
def test_values_of_d_dwave(torch, melt, N, H, M, frames):
    """Upstream gradients that make G 2^110, beyond what the planes hold, in some frames: the samples of
    those frames are within FP32's rounding of the 64-bit gradients, all others bit for bit as without
    them but for the samples that only share such a frame's last hop (recomputed too)."""
    plan = melt.MeltPlan(sample_rate=16000, n_fft=N, hop=H, n_mels=M, output=melt.MELT_OUT_POWER)
    wave, off = workloads.random_clips([frames * H + N, N - 1, 2 * H + N + 1], seed=M)
    T = melt.total_frames(off, N, H)
    g = np.random.default_rng(1).standard_normal((T, M)).astype(np.float32)
    proj = np.random.default_rng(2).uniform(0.5, 1, (T, 2 * M)).astype(np.float32)
    dev = lambda a: torch.from_numpy(a).cuda()

    def grad():
        return plan.backward(dev(wave), dev(off), T, dev(g), proj=dev(proj), want_basis=False)[0].cpu().numpy()

    clean = grad()
    at = [0, 3, frames // 2, T - 1]
    g[at, [0, M - 1, M // 2, 1]] = 2.0 ** 110
    got = grad()
    starts = np.concatenate([np.arange(a, b - N + 1, H) for a, b in zip(off[:-1], off[1:])])
    W = plan.basis().astype(np.float64).reshape(2, M, N).transpose(1, 0, 2).reshape(2 * M, N)
    G = (2 * proj * np.repeat(g, 2, axis=1)).astype(np.float64)
    near, want, mass = np.zeros(wave.size, bool), np.zeros(wave.size), np.zeros(wave.size)
    for t in at:
        near[starts[t]:min(starts[t] + -(-N // H) * H, off[np.searchsorted(off, starts[t], "right")])] = True
    reach = np.flatnonzero([near[s:s + N].any() for s in starts])
    for t in reach:
        want[starts[t]:starts[t] + N] += G[t] @ W
        mass[starts[t]:starts[t] + N] += np.abs(G[t]) @ np.abs(W)
    assert np.array_equal(got[~near], clean[~near])
    terms = 2 * M * -(-N // H)
    assert np.all(np.abs(got[near] - want[near]) <= 2 * terms * 2.0 ** -24 * mass[near])


@pytest.mark.parametrize("geom", [(16000, 400, 160, 40), (16000, 301, 33, 17), (16000, 512, 128, 100)])
def test_values_of_d_dbasis(torch, melt, geom):
    """NaN and both infinities in samples and upstream gradients, over several frame ranges: d/dbasis is
    NaN and infinite where 64-bit arithmetic makes it so, and as without them where none meets it."""
    sr, N, H, M = geom
    plan = melt.MeltPlan(sample_rate=sr, n_fft=N, hop=H, n_mels=M, output=melt.MELT_OUT_POWER)
    wave, off = workloads.random_clips([500 * H + N, N - 1, 90 * H + N + 2], seed=N)
    T = melt.total_frames(off, N, H)
    g = np.random.default_rng(1).standard_normal((T, M)).astype(np.float32)
    proj = np.random.default_rng(2).uniform(0.5, 1, (T, 2 * M)).astype(np.float32)
    dev = lambda a: torch.from_numpy(a).cuda()

    def grad():
        return plan.backward(dev(wave), dev(off), T, dev(g), proj=dev(proj), want_wave=False)[1].cpu().numpy()

    clean = grad()
    g[[3, 300, T - 2], [0, 5, M - 1]] = [np.inf, -np.inf, np.nan]
    g[444, 5] = np.inf
    wave[200 * H + 17] = np.inf
    got = grad()
    starts = np.concatenate([np.arange(a, b - N + 1, H) for a, b in zip(off[:-1], off[1:])])
    X = wave[starts[:, None] + np.arange(N)].astype(np.float64)
    G = (2 * proj.astype(np.float64) * np.repeat(g, 2, axis=1)).reshape(T, M, 2).transpose(0, 2, 1).reshape(T, 2 * M)
    with np.errstate(invalid="ignore"):
        want = G.T @ X
    assert np.array_equal(np.isnan(got), np.isnan(want))
    assert np.array_equal(np.isposinf(got), np.isposinf(want)) and np.array_equal(np.isneginf(got), np.isneginf(want))
    finite = np.isfinite(want)
    assert finite.any() and np.array_equal(got[finite], clean[finite])
