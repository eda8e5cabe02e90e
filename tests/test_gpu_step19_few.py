"""The D3Q19 step of few tiles stores directly, that of more through LDS: the
same bits on both sides of the line, and as the persistent step, which always
goes through LDS."""
import numpy as np
import pytest

from paper_1703_08015_amd import lbm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage,nz", [("f64", 8), ("f32", 16)])
@pytest.mark.parametrize("nx", [5, 256, 257])  # the last two: the line exactly, and 32 or 64 tiles more
@pytest.mark.parametrize("pattern", ["two-copy", "single-copy"])
def test_few_and_many_tiles(storage, nz, nx, pattern):
    import torch
    assert torch.cuda.is_available()
    shape = (nz, 64, nx)
    rng = np.random.default_rng(nx)
    m = rng.random(shape) < 0.2
    t = lbm.Tiles(m, (4, 4, 4), 0)
    rho = torch.from_numpy(np.where(m, 0.0, rng.uniform(0.99, 1.01, shape)))
    out = []
    for persistent in (False, True):
        s = lbm.Solver(t, lattice=19, storage=storage, tau=0.8, g=(1e-4, 2e-4, 0.0), pattern=pattern,
                       persistent=persistent)
        s.init(rho)
        s.step(5)
        out.append(s.pdfs_export())
    assert bool((out[0] == out[1]).all())
