"""mhd_get_particles on both sides of its choice between placing each value and
going through records: particles in the caller's order, value for value, with
either output left out."""
import ctypes as C

import pytest

from mhd_inputs import problems as P
from tests.gpu_util import needs_gpu

pytestmark = [pytest.mark.gpu, needs_gpu]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("shape,n", [((32, 32, 32), 1), ((32, 32, 32), 1 << 17),
                                     ((32, 32, 32), (1 << 17) + 1), ((8, 16, 8), 200001),
                                     ((32, 16, 8), 200001)])
def test_order_and_values(shape, n, precision):
    import torch
    from paper_1502_02935_amd import Sim, config_from_problem
    pb = P.gravity_box(shape, d=tuple(1.0 / k for k in shape), G=0.0)
    s = Sim(config_from_problem(pb, precision=precision, npart=n), pb.cell5, pb.bx, pb.by, pb.bz)
    dt = s.cfg.work_dtype
    g = torch.Generator(device="cuda").manual_seed(74)
    x = torch.rand((3, n), generator=g, device="cuda", dtype=dt).clamp(0.0, 0.99)
    v = torch.arange(3 * n, device="cuda", dtype=dt).view(3, n) * 2.0 ** -30  # each value its own
    s.set_particles(x, v, torch.full((n,), 1.0 / n, device="cuda", dtype=dt))
    s.step(3, dt=2.0 ** -40)  # sorts; without gravity velocities stay
    xo, vo = s.get_particles()
    assert torch.equal(vo, v)
    assert float((xo - x).abs().max()) <= 1e-6
    only = torch.empty_like(x)
    assert s.L.mhd_get_particles(s.ctx, C.c_void_p(only.data_ptr()), None) == 0
    assert torch.equal(only, xo)
    assert s.L.mhd_get_particles(s.ctx, None, C.c_void_p(only.data_ptr())) == 0
    assert torch.equal(only, v)
    s.step(1, dt=2.0 ** -40)
    assert torch.equal(s.get_particles()[1], v)
