"""The FP64 march's own quotients, square root and logarithm over the range of their arguments:
one-sided derivatives of rough data whose second derivatives run from 1e-6 (series only) past
the series' limit to 1e9 (antiderivative only), against the oracle.

Tolerance: a cell mean differs from the oracle's by at most 1.2e-14 relative (the
antiderivatives' rounding over the smallest wide gap), a weight by 4 such and the two squares'
2 ulp, so a derivative, a weighted mean of candidates of at most 11/6 + 7/6 + 1/3 times the
largest difference, by under 2 * 4 * 1.2e-14 * 10/3 = 3.3e-13 of it."""
import numpy as np
import pytest

import emulator as EM
import oracle as O

SCALES = [1e-6, 1e-2, 0.3, 1.0, 30.0, 1e4, 1e9]


def _case(scale):
    rng = np.random.default_rng(int(1e7 * scale) % 97)
    shape, h = (70, 150), (0.02, 0.03)
    # rough data whose second differences over h^2 are about `scale`
    phi = scale * h[0] ** 2 * rng.normal(size=shape) + 0.5 * np.arange(shape[1]) * h[0]
    return phi, h, O.derivatives(O.Problem(shape, h, O.H_LINEAR, (1.0, 0.0), 0), phi)


def _check(got, ref):
    for g, r in zip(got, ref):
        # the ramp's wrap makes steep jumps at the periodic edge; they count as data
        assert np.abs(g - r).max() <= 3.3e-13 * np.abs(r).max()


@pytest.mark.parametrize("scale", SCALES)
def test_emulated_march(scale):
    EM.set_tile(16, 8)
    phi, h, ref = _case(scale)
    _check(EM.derivatives(phi, h, 0, 0), ref)


@pytest.mark.gpu
@pytest.mark.parametrize("scale", SCALES)
def test_gpu_march(scale):
    from paper_1909_13263_amd import hjw
    phi, h, ref = _case(scale)
    ny, nx = phi.shape
    g = hjw.Grid(phi.shape, (0.0, 0.0), (nx * h[0], ny * h[1]), prec=hjw.FP64)
    g.set_phi(phi)
    _check([d.cpu().numpy() for d in g.derivatives()], ref)
    g.close()
