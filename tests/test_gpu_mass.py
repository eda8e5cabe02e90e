"""Mass over many steps: every step kernel, in both models, loses what the
weights lack, and no more."""
from fractions import Fraction

import numpy as np
import pytest

from paper_1703_08015_amd import lbm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q,shape,tile,kernel", [(9, (1, 64, 64), (16, 16, 1), "auto"),
                                                 (19, (16, 16, 16), (4, 4, 4), "generic"),
                                                 (19, (16, 16, 16), (4, 4, 4), "scalar")])
@pytest.mark.parametrize("model", ["quasi-compressible", "incompressible"])
@pytest.mark.parametrize("pattern", ["two-copy", "single-copy"])
@pytest.mark.parametrize("tau", [0.7, 1.0])
def test_mass_follows_the_weights(q, shape, tile, kernel, model, pattern, tau):
    """BGK takes omega sum_i w_i of the density in and omega of it out.  The
    weights as doubles do not sum to 1, so a step changes the mass by
    omega (sum w - 1) of it, -omega 2^-54 on both lattices; the roundings of
    single nodes have either sign and average out over some thousand nodes and
    20,000 steps, to within half of that."""
    import torch
    assert torch.cuda.is_available()
    steps = 20_000
    rng = np.random.default_rng(3)
    m = rng.random(shape) < 0.2
    rho = torch.from_numpy(np.where(m, 0.0, rng.uniform(0.99, 1.01, shape)))
    s = lbm.Solver(lbm.Tiles(m, tile, 7), lattice=q, tau=tau, g=(1e-6, 2e-6, 0.0), model=model, pattern=pattern,
                   step_kernel=kernel, graph_steps=100)
    s.init(rho)
    before = s.reduce()[0, 0]
    s.step(steps)
    drift = (s.reduce()[0, 0] - before) / before / steps
    want = float(sum(Fraction(float(w)) for w in lbm.lattice(q)[1]) - 1) / tau
    assert want < 0 and abs(drift - want) <= 0.5 * abs(want)
