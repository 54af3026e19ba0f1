"""Heavy tiles cut into pieces: one lattice cell holds P queries and its window
every key of the lattice, so that the tile's estimated cost is far above both
limits of the cut; P runs over the edges of the cut (128 queries, 256, the
second round's 128, the tile cap).  Eval with normals, gradient, fit step
(plain, deterministic and batched) against the FP64 oracle under the global
definition, with the tolerances of tests/parity.py."""
import numpy as np
import pytest
import torch

import oracle as orc
import workloads as W
from tests import parity as PT

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def E():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2505_21319_amd import efunc
    efunc.lib()
    return efunc


@pytest.mark.parametrize("P", [33, 128, 129, 255, 257, 384, 385, 512, 700])
def test_pieces_of_one_crowded_cell(E, P):
    R, extra = 10, 11
    rng = np.random.default_rng(P)
    h = 2.0 / (R - 1)
    cell = -1.0 + 4 * h
    q = np.concatenate([cell + h * rng.uniform(0.05, 0.95, (P, 3)), rng.uniform(-1, 1, (extra, 3))]).astype(np.float32)
    J = len(q)
    o = (np.linalg.norm(q, axis=1) - 0.5).astype(np.float32)
    th = W.perturbed_theta(R, 7, rho0=2.0)
    n = th.size
    tq, to = PT.to_dev(q), PT.to_dev(o)
    ref = PT.reference(R, th, q)
    dl = (2 * (ref["O"] - o) / J).astype(np.float32)

    def fit(eng):
        t, m, v = PT.to_dev(th), torch.zeros(n, device=PT.DEV), torch.zeros(n, device=PT.DEV)
        loss = torch.zeros(2, device=PT.DEV, dtype=torch.float64)
        eng.fit_step(t, m, v, 1, tq, to, loss)
        torch.cuda.synchronize()
        return m.cpu().numpy(), loss.cpu().numpy()

    with E.Engine(R, J) as eng:
        O, lse, dq, nu = eng.eval(PT.to_dev(th), tq, with_qgrad=True)
        G = eng.grad(PT.to_dev(th), tq, PT.to_dev(ref["O"]), PT.to_dev(ref["lse"]), PT.to_dev(dl))
        torch.cuda.synchronize()
        # the premise: every query is certified by its window, 2 R^3 keys for the crowded cell
        assert int(nu.item()) == 0 and eng.stats()["W"] >= R - 5
        fits = [fit(eng)]
    with E.Engine(R, J, deterministic=1) as eng:
        fits += [fit(eng), fit(eng)]
    assert np.array_equal(fits[1][0], fits[2][0]) and np.array_equal(fits[1][1], fits[2][1])
    mb, vb = [torch.zeros(n, device=PT.DEV) for _ in range(2)], [torch.zeros(n, device=PT.DEV) for _ in range(2)]
    lb = torch.zeros(2, 2, device=PT.DEV, dtype=torch.float64)
    with E.BatchEngine([R, R], [J, J]) as b:
        b.bind([PT.to_dev(th).reshape(-1) for _ in range(2)], mb, vb, [tq, tq], [to, to], lb)
        b.fit(1, 1, use_graph=True)
        torch.cuda.synchronize()
    fits += [(mb[s].cpu().numpy(), lb[s].cpu().numpy()) for s in range(2)]

    PT.check_eval(O.cpu().numpy(), lse.cpu().numpy(), ref)
    PT.check_qgrad(dq.cpu().numpy(), PT.qgrad_reference(orc.build_keys(orc.Grid(R=R), th), q))
    gr, ar, br = PT.oracle_grad(R, th, q, dl)
    PT.check_grad(G.cpu().numpy(), gr, ar, br)
    fr = orc.fit_step(orc.Grid(R=R), th, np.zeros(n), np.zeros(n), 1, q, o)
    for m1, loss in fits:
        assert abs(loss[0] - fr["loss"]) <= 1e-5 * fr["loss"] and abs(loss[1] - fr["l1"]) <= 1e-5 * fr["l1"]
        PT.check_grad(m1.astype(np.float64) / (1.0 - np.float32(0.9)), fr["grad"], ar, br)
