"""efunc_fit_step_static at the largest J that its scratch array held before the
tile kernel cut tiles (64 MiB; wide lattices with few queries, where the array is
filled by the parameters): still accepted, and equal to the fit step of a context
up to the order of float additions."""
import numpy as np
import pytest
import torch

from oracle import variants as V
from tests import parity as PT
from tests.test_oracle_var_pins import random_theta

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,deg,grid,moved,learn,J", [(50, 2, 1, 1, 1, 238), (57, 2, 0, 1, 1, 1412),
                                                      (66, 0, 0, 1, 1, 1428), (76, 0, 1, 0, 0, 444)])
def test_scratch_holds_what_it_held(R, deg, grid, moved, learn, J):
    from paper_2505_21319_amd import efunc as E
    m = V.Model(R=R, degree=deg, grid_keys=grid, moved_keys=moved, learn_scale=learn, rho_fixed=7.0)
    th = PT.to_dev(random_theta(m, J, rho=(6.8, 7.2), offset=0.35))
    rng = np.random.default_rng(R)
    q, o = PT.to_dev(rng.uniform(-1, 1, (J, 3))), PT.to_dev(rng.uniform(-0.5, 0.5, J))
    adam = E.efunc_default_adam()
    adam.lr = 0.0
    cfg = dict(degree=deg, grid_keys=grid, offsets=moved, learn_scale=learn, rho_fixed=7.0)
    out = []
    with E.Engine(R, J, **cfg) as eng:
        for static in (True, False):
            mom, v = torch.zeros(th.numel(), device=PT.DEV), torch.zeros(th.numel(), device=PT.DEV)
            loss = torch.zeros(2, device=PT.DEV, dtype=torch.float64)
            if static:
                E.efunc_fit_step_static(eng.cfg, th, mom, v, 1, q, o, loss, adam)
            else:
                eng.fit_step(th, mom, v, 1, q, o, loss, adam)
            out.append((loss.cpu().numpy(), mom.cpu().numpy().reshape(-1, V.channels(m))))
    (ls, ms), (lc, mc) = out
    assert np.all(np.abs(ls - lc) <= 1e-5 * np.abs(lc)) and np.abs(mc).max() > 0
    assert np.all(np.abs(ms - mc) <= 1e-4 * np.abs(mc) + 1e-5 * np.abs(mc).max(axis=0))
