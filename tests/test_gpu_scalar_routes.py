"""Passive scalars on both sides of the choice between walking tiles and one
cell a thread: against the oracle on boxes that fill the tiles and on boxes that
leave them nearly empty, in FP64 (1e-11) and FP32 (some 20 roundings a stage, 6
stages: 1e-5), and the time of a box one cell wide."""
import numpy as np
import pytest

from mhd_inputs import problems as P
from tests.gpu_util import needs_gpu
from tests.test_gpu_scalars import TOL, _pair, _run_both, _scalar_errors

pytestmark = [pytest.mark.gpu, needs_gpu]

PER, OUT = (P.PERIODIC,) * 6, (P.OUTFLOW,) * 6
MIXED = (P.OUTFLOW, P.OUTFLOW, P.PERIODIC, P.PERIODIC, P.OUTFLOW, P.OUTFLOW)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n,ns,bc", [
    ((64, 8, 17), 2, PER), ((120, 15, 19), 8, MIXED), ((128, 16, 5), 3, OUT), ((190, 8, 2), 1, PER),
    ((1, 9, 7), 4, PER), ((2, 3, 40), 8, PER), ((5, 17, 4), 3, MIXED), ((16, 40, 3), 1, OUT),
    ((66, 9, 6), 2, PER)])
def test_both_kernels_match_the_oracle(n, ns, bc, precision):
    pb = P.random_smooth(n, seed=57, bc=bc)
    if precision:
        pb = pb.astype("float32")
    rx = P.mass_fractions(pb, ns, "random", seed=58).astype(np.float32).astype(np.float64)
    o, s = _pair(pb, rx, precision=precision)
    _run_both(o, s, 3)
    assert max(_scalar_errors(s, o)) <= (1e-5 if precision else TOL)


def test_narrow_box_does_not_fill_tiles():
    """A row of one cell is 24 bytes in memory of which 4 are read, so up to six
    times a full row's traffic a cell; a tile's wave holds 64 columns of which one
    is in the box.  The bound of 9 times a wide box's time lies between."""
    import torch

    def ms(n):
        pb = P.random_smooth(n, seed=59).astype("float32")
        _, s = _pair(pb, P.mass_fractions(pb, 4, "random", seed=60), precision=1)
        s.step(3, dt=1e-6)
        best = np.inf
        for _ in range(3):
            s.profile(True)
            s.step(5, dt=1e-6)
            torch.cuda.synchronize()
            best = min(best, s.profile_get()["scalars"][0])
        return best

    assert ms((1, 512, 512)) <= 9.0 * ms((64, 64, 64))
