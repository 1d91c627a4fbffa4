"""The adjoint of a problem with its axes renamed cyclically is the renamed
adjoint, element by element.  The x axis has kernels of its own (rows), apart
from those of y and z (marches), so each form is held against the other on
grids of several blocks, ragged rows and segments, and rows shorter than the
stencil.

Bound: the two sides evaluate the same derivative at half-step states that
differ by the order of their flux differences, a few 1e-16; the derivative
varies with the state by at most about 1e3 of its scale (the eigenvectors turn
over B_perp, 1e-3 or more here), so 1e-10 of each field's largest element is two
orders above rounding, while one missing or doubled term is of order one."""
import numpy as np
import pytest

from oracle import ref
from paper_2402_05240_amd import inputs as I
from parity_util import FIELDS
from test_gpu_adjoint import _gpu_vjp, _need_gpu, _random_cotangent
from test_gpu_parity import _shaped_state

pytestmark = pytest.mark.gpu

# the field of the renamed problem (x', y', z') = (y, z, x) and where it comes from
TURN = {"rho": "rho", "E": "E", "mx": "my", "my": "mz", "mz": "mx", "bx": "by", "by": "bz",
        "bz": "bx"}


def _turned(g, s):
    t = I.Grid(g.ny, g.nz, g.nx, g.dy, g.dz, g.dx, g.gamma, g.cfl, g.recon, g.bc)
    return t, {f: np.ascontiguousarray(s[TURN[f]].transpose(2, 0, 1)) for f in FIELDS}


@pytest.mark.parametrize("shape", [(70, 9, 6), (33, 17, 9), (64, 66, 4), (2, 130, 3), (3, 1, 67)])
@pytest.mark.parametrize("recon", [1, 2, 3, 4, 5])
def test_adjoint_of_renamed_axes(recon, shape):
    _need_gpu()
    g, s = _shaped_state(shape, recon, (0, 0, 0), 51)
    dt = ref.cfl_dt(g, s)
    lam = _random_cotangent(g, 52)
    want = _gpu_vjp(g, s, lam, dt)
    for turn in range(2):
        _, want = _turned(g, want)
        _, lam = _turned(g, lam)
        g, s = _turned(g, s)
        got = _gpu_vjp(g, s, lam, dt)
        for f in FIELDS:
            err = np.abs(got[f] - want[f]).max() / np.abs(want[f]).max()
            assert err <= 1e-10, (turn, f, err)
