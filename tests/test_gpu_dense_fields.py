"""Dense fields and checkpoints written over the tile mesh: whole rows for groups
of four tiles, or a fill and the tiles alone where most groups are empty, at
ragged edges, for both tile shapes, 2D, batches and both layouts of the
single copy."""
import numpy as np
import pytest

from paper_1703_08015_amd import lbm

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available()
    return t


def _mask(shape, empty, seed):
    """Random solids; with `empty`, one corner holds the only fluid nodes (most groups of tiles are empty)."""
    m = np.random.default_rng(seed).random(shape) < 0.3
    if empty:
        m[:, :, shape[2] // 5 + 1:] = True
        m[:, shape[1] // 5 + 1:] = True
    m.flat[0] = False
    return m


CASES = [((5, 6, 7), (4, 4, 4)), ((12, 20, 36), (4, 4, 4)), ((9, 13, 30), (4, 4, 8)), ((16, 8, 64), (4, 4, 8)),
         ((1, 40, 48), (16, 16, 1)), ((1, 17, 33), (16, 16, 1))]


@pytest.mark.parametrize("shape,tile", CASES)
@pytest.mark.parametrize("empty", [False, True])
@pytest.mark.parametrize("storage", ["f64", "f16"])
@pytest.mark.parametrize("pattern,steps", [("two-copy", 2), ("single-copy", 2), ("single-copy", 3)])
def test_fields_of_the_stored_state(torch, shape, tile, empty, storage, pattern, steps):
    """export is 0 on solid nodes and, put back with import, exports the same
    bits; rho and u are the sums of the export (the FP64 sums of at most 19
    values of order 1: 19 x 2^-53 each, a few times that after the division
    by rho)."""
    q = 9 if tile[2] == 1 else 19
    m = _mask(shape, empty, 7)
    rng = np.random.default_rng(3)
    t = lbm.Tiles(m, tile, (0, 0, 0))
    s = lbm.Solver(t, lattice=q, storage=storage, tau=0.8, g=(1e-4, 2e-4, 0.0), pattern=pattern)
    u = torch.from_numpy(np.where(m, 0.0, rng.uniform(-0.02, 0.02, (3,) + shape)))
    s.init(torch.from_numpy(np.where(m, 0.0, rng.uniform(0.99, 1.01, shape))), u)
    s.step(steps)
    junk = torch.full((64, 1024, 32), float("nan"), dtype=torch.float64, device="cuda")  # what torch hands out next
    del junk
    f = s.pdfs_export()
    rho, v = s.moments()
    fl = torch.from_numpy(~m).cuda()
    assert not bool(f[:, ~fl].any()) and not bool(rho[~fl].any()) and not bool(v[:, ~fl].any())
    c, _, _ = lbm.lattice(q)
    total = f.sum(0)
    j = torch.tensordot(torch.from_numpy(c.T.astype(np.float64)).cuda(), f, 1)
    assert float((rho - total)[fl].abs().max()) <= 2e-14
    g = torch.tensor([1e-4, 2e-4, 0.0], dtype=torch.float64, device="cuda")[:, None]
    assert float((v[:, fl] - (j[:, fl] / total[fl] - 0.5 * g)).abs().max()) <= 4e-14
    s.pdfs_import(f)
    assert torch.equal(s.pdfs_export(), f)


@pytest.mark.parametrize("empty", [False, True])
def test_batch_fields_equal_single_runs(torch, empty):
    masks = [_mask(sh, empty, k) for k, sh in enumerate([(8, 8, 8), (12, 16, 20), (4, 4, 36), (20, 8, 12)])]
    tiles = [lbm.Tiles(m, (4, 4, 4), (1, 1, 1)) for m in masks]
    b = lbm.Solver(lbm.Tiles.concat(tiles), storage="f32", tau=0.8, g=(1e-5, 0.0, 0.0), persistent=1)
    b.init()
    b.step(5)
    rho, u, f = b.moments() + (b.pdfs_export(),)
    at = 0
    for m, t in zip(masks, tiles):
        s = lbm.Solver(t, storage="f32", tau=0.8, g=(1e-5, 0.0, 0.0))
        s.init()
        s.step(5)
        r, v = s.moments()
        n = m.size
        assert torch.equal(rho[at:at + n].view(m.shape), r)
        assert torch.equal(u[3 * at:3 * (at + n)].view((3,) + m.shape), v)
        assert torch.equal(f[19 * at:19 * (at + n)].view((19,) + m.shape), s.pdfs_export())
        at += n


def test_all_solid_fields_are_zero(torch):
    s = lbm.Solver(lbm.Tiles(np.ones((6, 5, 9), bool), (4, 4, 4), (0, 0, 0)))
    s.init()
    rho, u = s.moments()
    assert not bool(rho.any()) and not bool(u.any()) and not bool(s.pdfs_export().any())
