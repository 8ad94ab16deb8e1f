"""FP64 reciprocals and roots of the kernels are the correctly rounded ones, for
every argument: a uniform state at rest without a field has dt = cfl / (c / dx)
with c^2 = (2 a^2)/2 through two roots, so mhd_dt shows both.  Arguments where a
form short of that falls off: mantissas next to a power of two, results that are
denormal, roots of arguments whose residual underflows.  Expected: the same
expression in NumPy's IEEE arithmetic, bit for bit."""
import numpy as np
import pytest

from tests.gpu_util import needs_gpu

pytestmark = [pytest.mark.gpu, needs_gpu]

GAMMA = 2.0


def _gpu_dt(rho, p, dx):
    from paper_1502_02935_amd import Sim
    from paper_1502_02935_amd.sim import MHDConfig
    cfg = MHDConfig(nx=2, ny=1, nz=1, dx=dx, dy=dx, dz=dx, gamma=GAMMA, cfl=1.0)
    c5 = np.zeros((5, 1, 1, 2))
    c5[0], c5[4] = rho, p / (GAMMA - 1.0)
    z = np.zeros((1, 1, 2))
    s = Sim(cfg, c5, z, z, z)
    dt = s.dt()
    s.close()
    return dt


def _dt(rho, p, dx):
    with np.errstate(all="ignore"):
        rho, p, dx, one = (np.float64(v) for v in (rho, p, dx, 1.0))
        a2 = np.float64(GAMMA) * p * (one / rho)
        c = np.sqrt(np.float64(0.5) * (a2 + np.sqrt(a2 * a2)))
        return one / (c * (one / dx))


def _square(s):
    """p of sound speed s: gamma p / rho = s^2 at rho = 1."""
    return float(np.float64(s) * np.float64(s) / GAMMA)


ULP = 2.0 ** -52
CASES = (
    # 1/s and 1/rho just above a power of two's reciprocal
    [(1.0, _square(2.0 - k * ULP), 1.0) for k in range(1, 13)]
    + [(1.0, _square(1.0 + k * ULP), 1.0) for k in range(1, 5)]
    + [((2.0 - k * ULP) * 2.0 ** e, 2.0 ** e, 1.0) for k in (1, 3, 6) for e in (-40, 0, 900)]
    # 1/s denormal, s denormal
    + [(1.0, _square(2.0 - k * ULP), 2.0 ** -1022) for k in (1, 2, 3, 5)]
    + [(1.0, _square(1.0 + k * ULP), 2.0 ** -1022) for k in (1, 2, 3)]
    + [(1.0, _square(c), 2.0 ** 1021) for c in (0.3, 0.26, 0.7)]
    # roots of arguments near the smallest
    + [(1.0, m * 2.0 ** -e, 1.0) for m in (1.0, 1.1, 1.3, 1.7) for e in (940, 964, 980, 1000)])


@pytest.mark.parametrize("rho,p,dx", CASES)
def test_time_step_is_correctly_rounded(rho, p, dx):
    assert _gpu_dt(rho, p, dx) == _dt(rho, p, dx)


@pytest.mark.parametrize("lo", [0, 1 << 10, 1 << 30])
def test_time_step_of_random_states(lo):
    rng = np.random.default_rng(7 + lo)
    for _ in range(100):
        s = 2.0 - (lo + int(rng.integers(0, 2 * lo + 64))) * ULP
        rho = float(2.0 ** rng.uniform(-300, 300))
        p = _square(s) * rho
        assert _gpu_dt(rho, p, 1.0) == _dt(rho, p, 1.0), (rho, p)
