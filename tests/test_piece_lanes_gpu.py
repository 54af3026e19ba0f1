"""Crowded tiles of few queries, where a cut fit tile's queries keep their
several lanes (256 / P each, four more per lane in a small piece) and a gradient's
pieces share the window's keys: P at the steps of the lanes (16 lanes, 15, 8, 4, 3,
2 and 1), of the pieces (16 queries each, 64 lanes) and of the second round, in a
window of every key of the lattice.  Against the FP64 oracle under the global
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


@pytest.mark.parametrize("P", [16, 17, 32, 64, 85, 127, 256, 272, 400])
def test_lanes_of_a_cut_tile(E, P):
    R = 18
    rng = np.random.default_rng(P)
    h = 2.0 / (R - 1)
    cell = -1.0 + 8 * h
    q = np.concatenate([cell + h * rng.uniform(0.05, 0.95, (P, 3)), rng.uniform(-1, 1, (7, 3))]).astype(np.float32)
    J = len(q)
    o = (np.linalg.norm(q, axis=1) - 0.5).astype(np.float32)
    th = W.perturbed_theta(R, 7, rho0=2.0)
    n = th.size
    tq, to = PT.to_dev(q), PT.to_dev(o)
    fr = orc.fit_step(orc.Grid(R=R), th, np.zeros(n), np.zeros(n), 1, q, o)
    ref = PT.reference(R, th, q)
    dl = (2 * (ref["O"] - o) / J).astype(np.float32)
    gr, ar, br = PT.oracle_grad(R, th, q, dl)
    fits = []
    for det in (0, 1, 1):
        with E.Engine(R, J, deterministic=det) as eng:
            t, m, v = PT.to_dev(th), torch.zeros(n, device=PT.DEV), torch.zeros(n, device=PT.DEV)
            loss = torch.zeros(2, device=PT.DEV, dtype=torch.float64)
            G = eng.grad(t, tq, PT.to_dev(ref["O"]), PT.to_dev(ref["lse"]), PT.to_dev(dl))
            torch.cuda.synchronize()
            assert eng.stats()["W"] >= R - 9  # the premise: every key in the crowded cell's window
            PT.check_grad(G.cpu().numpy(), gr, ar, br)
            eng.fit_step(t, m, v, 1, tq, to, loss)
            torch.cuda.synchronize()
            fits.append((m.cpu().numpy(), loss.cpu().numpy()))
    assert np.array_equal(fits[1][0], fits[2][0]) and np.array_equal(fits[1][1], fits[2][1])
    for m1, loss in fits:
        assert abs(loss[0] - fr["loss"]) <= 1e-5 * fr["loss"] and abs(loss[1] - fr["l1"]) <= 1e-5 * fr["l1"]
        PT.check_grad(m1.astype(np.float64) / (1.0 - np.float32(0.9)), fr["grad"], ar, br)
