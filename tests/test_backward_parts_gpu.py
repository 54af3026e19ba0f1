"""The backward's parts: a batch of n kept keys is taken in parts of 256, 128, ...
keys with 1, 2, ... lanes each, by one rule for tiles of 64 queries and more (two
lanes for up to 192 keys left, four for up to 96, eight for 48, sixteen for 24) and
another for fewer (as many lanes as fit).  One tile whose every key near the lattice
is kept, the others moved far out, at counts on both sides of those lines and across
a whole batch; fit step and gradient against the FP64 variant oracle under the
global definition, with the tolerances of tests/parity.py."""
import numpy as np
import pytest
import torch

from oracle import variants as V
from tests import parity as PT
from tests.test_oracle_var_pins import random_theta

pytestmark = pytest.mark.gpu

# (kept keys, R, grid_keys): moved keys beyond the count lie far away
COUNTS = [(8, 2, 1), (16, 2, 1), (24, 3, 0), (25, 3, 0), (48, 3, 1), (49, 3, 1), (64, 4, 1), (65, 4, 1), (96, 4, 1),
          (97, 4, 1), (128, 4, 1), (129, 5, 1), (192, 5, 1), (193, 5, 1), (256, 6, 1), (257, 6, 1), (352, 6, 1),
          (432, 6, 1)]


@pytest.mark.parametrize("P", [1, 3, 63, 64, 65, 130])
@pytest.mark.parametrize("kept,R,grid", COUNTS, ids=[str(c[0]) for c in COUNTS])
def test_parts_of_a_batch(kept, R, grid, P):
    from paper_2505_21319_amd import efunc as E
    m = V.Model(R=R, grid_keys=grid)
    th = random_theta(m, kept, rho=(0.8, 1.2), offset=0.2)
    L = V.layout(m)
    rng = np.random.default_rng(kept + P)
    far = rng.permutation(m.I)[kept - grid * m.I:]
    th[far, L["moved_delta"]] = 100.0
    h = 2.0 / (R - 1)
    cell = (R - 1) // 2
    q = (-1.0 + h * (cell + rng.uniform(0.1, 0.9, (P, 3)))).astype(np.float32)
    o = (np.linalg.norm(q, axis=1) - 0.5).astype(np.float32)
    keys = V.build_keys(m, th)
    O, lse, _ = V.eval_global(keys, 1, q)
    dl = (2 * (O - o) / P).astype(np.float32)
    n, nch = th.size, V.channels(m)
    fr = V.fit_step(m, th, np.zeros(n), np.zeros(n), 1, q, o)
    gr, ar, br = (V.grad_theta(m, th, x) for x in V.grad_global(keys, 1, q, dl.astype(np.float64), T=PT.T_TAIL))
    with E.Engine(R, P, grid_keys=grid) as eng:
        t, tq, to = PT.to_dev(th), PT.to_dev(q), PT.to_dev(o)
        mom, v = torch.zeros(n, device=PT.DEV), torch.zeros(n, device=PT.DEV)
        loss = torch.zeros(2, device=PT.DEV, dtype=torch.float64)
        G = eng.grad(t, tq, PT.to_dev(O), PT.to_dev(lse), PT.to_dev(dl))
        eng.fit_step(t, mom, v, 1, tq, to, loss)
        st = eng.stats()
        # the premise (for a lone query at 3^3 keys of the far corner fall below e^-20)
        assert st["n_tiles"] == 1 and st["n_uncertified"] == 0, st
        assert kept * P - (2 if P == 1 and R == 3 else 0) <= st["bwd_pairs"] <= kept * P, st
        loss, G, g = loss.cpu().numpy(), G.cpu().numpy(), mom.cpu().numpy().astype(np.float64) / (1.0 - np.float32(0.9))
    assert abs(loss[0] - fr["loss"]) <= 1e-5 * fr["loss"] and abs(loss[1] - fr["l1"]) <= 1e-5 * fr["l1"]
    PT.check_grad(G, gr, ar, br, nch=nch)
    PT.check_grad(g, fr["grad"], ar, br, nch=nch)
