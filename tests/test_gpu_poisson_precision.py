"""The FP32 Poisson solve is no less accurate than the plain way: full complex
transforms in single precision, radix-2 stage by stage along x, y and z, division
by the Laplacian's eigenvalues, the same back -- each against the solve in 64
bits of the very density the step used, by the error of the potential and of its
central gradient (which shows the short waves).  The plain way is the bound
itself; the kernels' half spectra and paired rows must not fall behind it."""
import numpy as np
import pytest

from mhd_inputs import problems as P
from tests.gpu_util import needs_gpu

pytestmark = [pytest.mark.gpu, needs_gpu]

C64 = np.complex64


def _fft(a, axis, sign):
    """Radix-2 transform along an axis in complex64."""
    a = np.ascontiguousarray(np.moveaxis(a, axis, -1)).astype(C64)
    n = a.shape[-1]
    bits = n.bit_length() - 1
    order = [int(format(i, "0%db" % bits)[::-1], 2) for i in range(n)] if bits else [0]
    a = a[..., order]
    m = 1
    while m < n:
        w = np.exp(sign * 1j * np.pi * np.arange(m) / m).astype(C64)
        b = a.reshape(a.shape[:-1] + (n // (2 * m), 2, m))
        u, v = b[..., 0, :], (b[..., 1, :] * w).astype(C64)
        a = np.stack([u + v, u - v], axis=-2).reshape(a.shape)
        m *= 2
    return np.moveaxis(a, -1, axis)


def _eigenvalues(shape, d):
    lam = 0.0
    for axis, (n, h) in enumerate(zip(shape, d)):
        e = (2.0 * np.cos(2.0 * np.pi * np.arange(n) / n) - 2.0) / h ** 2
        lam = lam + e.reshape([n if a == axis else 1 for a in range(3)])
    return lam


def _solve(rho, lam, G, forward, back):
    f = forward(rho)
    s = np.zeros_like(lam)
    s[lam != 0] = 4.0 * np.pi * G / lam[lam != 0] / rho.size
    return back((f * s.astype(np.float32 if f.dtype == C64 else np.float64)))


def _plain(rho, lam, G):
    def along(sign):
        def f(a):
            for axis in (2, 1, 0):
                a = _fft(a, axis, sign)
            return a
        return f
    return _solve(rho.astype(np.float32), lam, G, along(-1), along(+1)).real


def _errors(psi, grad, ref, d):
    g = [(np.roll(ref, -1, a) - np.roll(ref, 1, a)) / (2.0 * d[a]) for a in range(3)]
    e = sum(float(((grad[a] - g[a]) ** 2).sum()) for a in range(3))
    return (np.sqrt(float(((psi - ref) ** 2).sum()) / float((ref ** 2).sum())),
            np.sqrt(e / sum(float((q ** 2).sum()) for q in g)))


@pytest.mark.parametrize("n", [(64, 32, 32), (32, 32, 32), (32, 32, 128), (256, 32, 16)])
def test_no_less_accurate_than_full_transforms(n):
    from paper_1502_02935_amd import Sim, config_from_problem
    G, h = 1.0, 1.0 / 64
    shape, d = n[::-1], (h, h, h)
    lam = _eigenvalues(shape, d)
    mine, plain = [], []
    for seed in (81, 82, 83):
        rng = np.random.default_rng(seed)
        k2 = -lam * h ** 2
        k2[0, 0, 0] = 1.0
        g = np.fft.ifftn(np.fft.fftn(rng.standard_normal(shape)) / k2).real
        pb = P.gravity_box(n, G=G, couple_gas=True, rho=1.0, p=1.0, d=d)
        pb.cell5[0] = np.exp((g - g.mean()) / g.std())
        pb = pb.astype("float32")
        s = Sim(config_from_problem(pb, precision=1), pb.cell5, pb.bx, pb.by, pb.bz)
        s.step(1, dt=1e-6)
        rho, psi, gx, gy, gz = (s.debug_array(w).double().cpu().numpy()[2:-3, 2:-3, 2:-3]
                                for w in (27, 35, 36, 37, 38))
        s.close()
        ref = _solve(rho, lam, G, np.fft.fftn, lambda a: np.fft.ifftn(a) * a.size).real
        mine.append(_errors(psi, (gz, gy, gx), ref, d))
        p = _plain(rho, lam, G)
        f32 = [((np.roll(p, -1, a) - np.roll(p, 1, a)) * np.float32(0.5 / d[a])).astype(np.float64)
               for a in range(3)]
        plain.append(_errors(p.astype(np.float64), f32, ref, d))
    mine, plain = np.mean(mine, axis=0), np.mean(plain, axis=0)
    assert (mine <= plain).all(), (mine, plain)
