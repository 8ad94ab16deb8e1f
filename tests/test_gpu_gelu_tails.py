"""The in-step network's GELU far outside its table: hidden units whose
arguments are huge (a cold, strongly magnetised state scales its features by
1/c).  GELU is 0 there on the negative side and the argument itself on the
positive one, in a step against the FP64 oracle.

The first layer ignores the inputs (zero weights), so every face has the same
hidden values: 0 or 2^e (exact in bfloat16), and the second layer's arguments are
+-64 x 2^e 2^-e + b2, exact but for b2's rounding.  The correction is of order
1e-2 of the flux scale and moves a field by 1e-3 in 3 steps; a hidden value of the
second layer (below 1) may round to the neighbouring bfloat16 (2^-9) on the
table's error: 2^-9 x 0.002 x dt/dx < 1 x 3 steps, 2e-5 for a few of them."""
import numpy as np
import pytest

from mhd_inputs import problems as P
from oracle import pyorc as O
from tests.gpu_util import field_errors, gpu_sim, host_state, needs_gpu
from tests.helpers import oracle_of

pytestmark = [pytest.mark.gpu, needs_gpu]

B1, W2, B2, W3, B3 = 64 * 32, 64 * 32 + 64, 64 * 32 + 64 + 4096, 6272, 6784


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("sign,e", [(-1, 8), (-1, 40), (-1, 67), (-1, 100), (-1, 120), (1, 8),
                                    (1, 40), (1, 100), (1, 119), (1, 122)])
def test_step_with_huge_hidden_arguments(sign, e, precision):
    import torch
    rng = np.random.default_rng(11)
    p = np.zeros(O.MLP_NPARAM)
    p[B1:W2] = sign * 2.0 ** e
    p[W2:B2] = 2.0 ** -e if sign > 0 else 2.0 ** -6
    p[B2:W3] = rng.uniform(-1.0, 1.0, 64) - (64.0 if sign > 0 else 0.0)
    p[W3:B3] = rng.normal(0, 0.002, 512)
    p = p.astype(np.float32).astype(np.float64)
    pb = P.random_smooth((21, 9, 6), seed=5)
    if precision:
        pb = pb.astype("float32")
    o = oracle_of(pb)
    o.set_mlp(p, tau=0.5, jump=0.5, tau_flux=0.1)
    s = gpu_sim(pb, precision=precision)
    t = torch.as_tensor(p, dtype=torch.float32, device="cuda")
    s.set_mlp(t, tau=0.5, jump=0.5, tau_flux=0.1)
    dts = []
    for _ in range(3):
        dts.append(o.dt())
        o.step(dts[-1])
    s.step(3, dt=dts)
    err = field_errors(host_state(s), o.get_state())
    assert max(err.values()) <= (2e-5 if precision == 0 else 1e-4), err
    assert s.diag()["n_mlp_faces"] > 0
