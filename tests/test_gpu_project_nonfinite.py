"""The projection beside infinite and NaN velocities: they reach what links
carry them to, and nothing else; what no link carries comes out at rest."""
import numpy as np
import pytest

from oracle import invariants
from paper_1703_08015_amd import lbm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("iterations", [1, 2, 3])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("shape,q", [((10, 9, 20), 19), ((1, 18, 40), 9)])
def test_nonfinite_velocities(iterations, bad, shape, q):
    """A component that no link carries adds nothing anywhere, so the result is
    that of a 0 in its place, to the bars of the projection tests (rho to
    1e-13, u to 1e-14 of its largest value), and 0 itself."""
    import torch
    assert torch.cuda.is_available()
    rng = np.random.default_rng(iterations)
    mask = rng.random(shape) < 0.5
    z, y = shape[0] // 2, 8
    mask[max(z - 2, 0):z + 3, y - 3:y + 4, 2:18] = True
    mask[z, y, 6] = False            # a node without links
    mask[z, y, 10:13] = False        # a row: no link carries y or z
    rho = np.where(mask, 1.0, 1.0 + 0.01 * rng.normal(size=shape))
    u = np.where(mask[None], 0.0, 0.01 * rng.normal(size=(3,) + shape))
    if q == 9:
        u[2] = 0.0
    u[:, z, y, 6] = u[1, z, y, 11] = 0.0
    ref_r, ref_u = invariants.project(mask, rho, u, q, iterations=iterations, periodic=0)
    u[:2, z, y, 6] = u[1, z, y, 11] = bad
    inv = lbm.Invariants(mask, q, periodic=0)
    r, v = torch.from_numpy(rho.copy()).cuda(), torch.from_numpy(u.copy()).cuda()
    inv.project(r, v, iterations=iterations)
    r, v, fl = r.cpu().numpy(), v.cpu().numpy(), ~mask
    assert np.abs(r[fl] - ref_r[fl]).max() <= 1e-13
    assert np.abs(v[:, fl] - ref_u[:, fl]).max() <= 1e-14 * max(np.abs(ref_u[:, fl]).max(), 1e-3)
    assert np.all(v[:2, z, y, 6] == 0) and v[1, z, y, 11] == 0
