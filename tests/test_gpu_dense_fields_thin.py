"""Dense fields and checkpoints where every group of four tiles holds one tile:
lattices of at most four nodes in x, few and many, and a sparse mesh."""
import numpy as np
import pytest

from paper_1703_08015_amd import lbm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,tile", [((16, 24, 4), (4, 4, 4)), ((9, 13, 3), (4, 4, 8)), ((170, 200, 4), (4, 4, 4)),
                                        ((201, 190, 2), (4, 4, 4)), ((344, 203, 4), (4, 4, 8)), ((24, 24, 64), (4, 4, 4))])
@pytest.mark.parametrize("storage", ["f64", "f16"])
@pytest.mark.parametrize("pattern,steps", [("two-copy", 2), ("single-copy", 3)])
def test_single_tiles(shape, tile, storage, pattern, steps):
    """export is 0 on solid nodes and, put back with import, exports the same
    bits; rho is the sum of the export (FP64 sums of 19 values of order 1)."""
    import torch
    assert torch.cuda.is_available()
    rng = np.random.default_rng(sum(shape))
    m = rng.random(shape) < 0.3
    if shape[2] > 4:  # one tile in every group of four, not always the first
        keep = np.zeros(shape, bool)
        for k, (z, y) in enumerate(np.ndindex(shape[0] // 4, shape[1] // 4)):
            for g in range(shape[2] // 16):
                x = 16 * g + 4 * ((k + g) % 4)
                keep[4 * z:4 * z + 4, 4 * y:4 * y + 4, x:x + 4] = True
        m |= ~keep
    t = lbm.Tiles(m, tile, 0)
    s = lbm.Solver(t, lattice=19, storage=storage, tau=0.8, g=(1e-4, 2e-4, 0.0), pattern=pattern)
    s.init(torch.from_numpy(np.where(m, 0.0, rng.uniform(0.99, 1.01, shape))))
    s.step(steps)
    f = s.pdfs_export()
    rho, _ = s.moments()
    fl = torch.from_numpy(~m).cuda()
    assert not bool(f[:, ~fl].any()) and not bool(rho[~fl].any())
    assert float((rho - f.sum(0))[fl].abs().max()) <= 2e-14
    s.pdfs_import(f)
    assert torch.equal(s.pdfs_export(), f)
    two = lbm.Solver(t, lattice=19, storage=storage, tau=0.8, g=(1e-4, 2e-4, 0.0), pattern=pattern)
    two.pdfs_import(f)
    two.step(3)
    s.step(3)
    assert torch.equal(two.pdfs_export(), s.pdfs_export())
