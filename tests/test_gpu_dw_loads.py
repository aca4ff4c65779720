"""d/dbasis where its loads and steps change: frame lengths of every remainder of 4 (four columns
a lane, with and without a lane that has fewer), frames of fewer than four samples, and frame
counts around a step of 32 and a pair of steps, against the FP64 chain rule with the bounds of
the other backward tests."""
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


@pytest.mark.parametrize("frames", [1, 32, 33, 65, 97, 300])
@pytest.mark.parametrize("geom", [(16000, 400, 160, 80), (16000, 401, 160, 20), (16000, 258, 100, 65), (16000, 403, 160, 9),
                                  (16000, 7, 3, 5), (16000, 3, 2, 5)])
def test_frame_lengths_and_steps(torch, melt, orc, geom, frames):
    from tests.test_gpu_backward import _case
    sr, N, H, M = geom
    # the last clip ends with its last frame: nothing may be read behind it
    wave, off = workloads.random_clips([N - 1, N + (frames - 1) * H], seed=N + frames)
    _case(torch, melt, orc, wave, off, float(sr), N, H, M, label=f"d/dbasis {geom} {frames}")
