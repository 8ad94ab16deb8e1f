"""The Poisson solve at line lengths of every axis where the kernels' split of a
line over threads differs and no other test reaches: z of 16, 32, 64, 128, 512 and
1024 points (one or two turns of the solve's loop, the largest registers and LDS),
y of 2, 16, 32, 128, 256 and 1024, x of 1, 8, 32, 256 and 512; FP64 against the
oracle's potential, gradient and state (1e-11), FP32 against its potential."""
import numpy as np
import pytest

from tests import test_gpu_gravity as G
from tests.gpu_util import gpu_sim, needs_gpu
from tests.helpers import oracle_of

pytestmark = [pytest.mark.gpu, needs_gpu]

SHAPES = [(2, 2, 128), (2, 2, 512), (2, 1, 1024), (1, 4, 16), (2, 8, 32), (8, 2, 64), (2, 16, 2),
          (32, 32, 1), (2, 128, 4), (2, 256, 2), (2, 1024, 2), (256, 2, 2), (512, 2, 4)]


@pytest.mark.parametrize("shape", SHAPES)
def test_fp64_lengths(shape):
    G.test_potential_and_state_match_oracle(shape)


@pytest.mark.parametrize("shape", SHAPES)
def test_fp32_lengths(shape):
    """A value is rounded some 5 times a pass, 5 passes, each 6e-8 of the largest:
    2e-6 of the largest potential with the errors all of one sign."""
    pb = G._gravity_box(shape, seed=43).astype("float32")
    o, s = oracle_of(pb), gpu_sim(pb, precision=1)
    dt = 0.1 * o.dt()
    o.step(dt)
    s.step(1, dt=dt)
    sl = (slice(2, 2 + pb.nz), slice(2, 2 + pb.ny), slice(2, 2 + pb.nx))
    g, r = s.debug_array(35).double().cpu().numpy()[sl], o.debug_array(41)[sl]
    assert np.abs(g - r).max() <= 2e-6 * np.abs(r).max()
