"""The deposit and the kick keep to their LDS window wherever the particles and
the box allow it: on boxes narrower than the window, whose cells it holds more
than once, and with masses too far apart for fixed point.  What leaves it still gives the right sums (the other tests), but
takes eight adds to memory a particle instead of one a cell and chunk, ten times
the time and more; the bounds of 4 lie between."""
import numpy as np
import pytest

from mhd_inputs import problems as P
from tests.gpu_util import needs_gpu
from tests.test_gpu_nbody import TOL, _pair, _particle_errors, _run_both

pytestmark = [pytest.mark.gpu, needs_gpu]

N = 1 << 18


def _ms(shape, x, m):
    """Milliseconds of the gravity and particle kernels of a step, FP32."""
    import torch
    from paper_1502_02935_amd import Sim, config_from_problem
    pb = P.gravity_box(shape, d=tuple(1.0 / k for k in shape)).astype("float32")
    s = Sim(config_from_problem(pb, precision=1, npart=N), pb.cell5, pb.bx, pb.by, pb.bz)
    s.set_particles(x, np.zeros((3, N)), m)
    s.step(3, dt=1e-6)
    best = np.inf
    for _ in range(3):
        s.profile(True)
        s.step(4, dt=1e-6)
        torch.cuda.synchronize()
        p = s.profile_get()
        best = min(best, p["gravity"][0] + p["nbody"][0])
    s.close()
    return best


@pytest.mark.parametrize("shape,wide", [((8, 8, 8), (16, 16, 16)), ((64, 64, 8), (64, 32, 16)),
                                        ((4, 64, 64), (16, 32, 32)), ((64, 2, 64), (32, 16, 16))])
def test_narrow_boxes_keep_to_the_window(shape, wide):
    x = np.random.default_rng(71).uniform(0.0, 1.0, (3, N))
    m = np.full(N, 1.0 / N)
    assert _ms(shape, x, m) <= 4.0 * _ms(wide, x, m)


@pytest.mark.parametrize("width", [1.0, 0.02])
def test_masses_far_apart_keep_to_the_window(width):
    rng = np.random.default_rng(73)
    x = 0.5 + width * rng.uniform(-0.5, 0.5, (3, N))
    m = np.full(N, 1.0 / N)
    apart = m * 10.0 ** rng.uniform(-9.0, 0.0, N)
    assert _ms((32, 32, 32), x, apart) <= 4.0 * _ms((32, 32, 32), x, m)


@pytest.mark.parametrize("shape", [(8, 8, 8), (4, 16, 8), (1, 2, 16), (32, 8, 2), (16, 1, 4)])
def test_narrow_boxes_match_the_oracle(shape):
    """Tiles of more than 256 particles, so the kick reads the window too."""
    rng = np.random.default_rng(72)
    pb = P.gravity_box(shape, d=tuple(1.0 / k for k in shape))
    x = rng.uniform(0.0, 1.0, (3, 5000))
    o, s = _pair(pb, x, 0.2 * rng.standard_normal((3, 5000)), rng.uniform(0.5, 1.5, 5000) / 5000)
    _run_both(o, s, 3)
    ex, ev = _particle_errors(s, o, pb)
    assert ex <= TOL and ev <= TOL, (ex, ev)
