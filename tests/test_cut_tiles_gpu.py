"""Cut tiles of every model: one lattice cell holds P queries and a window of
hundreds or thousands of keys, so that its tile is cut in every call (asserted
from the library's count of work items).  Degrees 0 and 2, grid keys alone,
moved keys alone (whose reference exponent is an exact maximum), a fixed scale,
and a forced window that certifies only part of the crowded cell's queries, so
that the others fall back to all keys while the tile's pieces run.  Values, lse,
query gradients, parameter gradients and a fit step, plain and deterministic,
against the FP64 variant oracle under the global definition, with the tolerances
of tests/parity.py."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import variants as V
from tests import parity as PT
from tests.test_oracle_var_pins import random_theta

# (name, degree, grid_keys, moved_keys, learn_scale, R, P, cell, rho, forced window)
CASES = [
    ("f0_both", 0, 1, 1, 1, 10, 400, 4, (1.5, 2.5), 0),
    ("f2_both", 2, 1, 1, 1, 10, 512, 4, (1.5, 2.5), 0),
    ("f2_both_few", 2, 1, 1, 1, 18, 33, 8, (1.5, 2.5), 0),
    ("f2_grid", 2, 1, 0, 1, 12, 300, 5, (1.5, 2.5), 0),
    ("f1_moved", 1, 0, 1, 1, 12, 512, 5, (1.5, 2.5), 0),
    ("f1_moved_few", 1, 0, 1, 1, 18, 60, 8, (1.5, 2.5), 0),
    ("f2_moved_fixed", 2, 0, 1, 0, 12, 512, 5, (2.0, 2.0), 0),
    ("f1_fallback", 1, 1, 1, 1, 14, 450, 6, (3.8, 4.0), 4),
    ("f2_fallback", 2, 1, 1, 1, 14, 450, 6, (3.8, 4.0), 4),
    ("f1_moved_fallback", 1, 0, 1, 1, 14, 450, 6, (3.8, 4.0), 4),
]


@pytest.fixture(scope="module")
def E():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2505_21319_amd import efunc
    efunc.lib()
    V.build_var_oracle(force=False)
    return efunc


def test_item_counts_reject_null():
    from paper_2505_21319_amd import efunc as B
    n = (ctypes.c_int64 * 2)()
    assert B.lib().efunc_get_items(None, n) == B.EFUNC_EINVAL


@pytest.mark.gpu
@pytest.mark.parametrize("det", [0, 1])
@pytest.mark.parametrize("c", CASES, ids=[c[0] for c in CASES])
def test_cut_tiles_of_every_model(E, c, det):
    name, deg, grid, moved, learn, R, P, cell, rho, window = c
    m = V.Model(R=R, degree=deg, grid_keys=grid, moved_keys=moved, learn_scale=learn, rho_fixed=rho[0])
    th = random_theta(m, 11 + R, rho=rho, offset=0.35)
    n, nch = th.size, V.channels(m)
    rng = np.random.default_rng(P + R)
    h = 2.0 / (R - 1)
    q = (-1.0 + cell * h + h * rng.uniform(0.02, 0.98, (P, 3))).astype(np.float32)
    o = (np.linalg.norm(q, axis=1) - 0.5).astype(np.float32)
    keys = V.build_keys(m, th)
    O, lse, sig = V.eval_global(keys, deg, q)
    kap, tail = V.eval_cond(keys, deg, q, PT.T_TAIL, with_tail=True)
    ref = dict(O=O, lse=lse, sigma=sig, kappa=kap, tail=tail)
    dl = (2 * (O - o) / P).astype(np.float32)
    fr = V.fit_step(m, th, np.zeros(n), np.zeros(n), 1, q, o)
    gk, ak, bk = V.grad_global(keys, deg, q, dl.astype(np.float64), T=PT.T_TAIL)
    gr, ar, br = (V.grad_theta(m, th, x) for x in (gk, ak, bk))

    cfg = dict(degree=deg, grid_keys=grid, offsets=moved, learn_scale=learn, rho_fixed=rho[0], window=window,
               deterministic=det)
    with E.Engine(R, P, **cfg) as eng:
        def cut(rest=False):
            st, items = eng.stats(), eng.items()
            assert items[0] > st["n_tiles"] and (items[1] > 1) == rest, (items, st)
            assert 0 < st["n_uncertified"] < P if window else st["n_uncertified"] == 0, st

        t, tq, to = PT.to_dev(th), PT.to_dev(q), PT.to_dev(o)
        for normals in (False, True):
            Og, lg, dq, _ = eng.eval(t, tq, with_qgrad=normals)
            cut()
            PT.check_eval(Og.cpu().numpy(), lg.cpu().numpy(), ref)
        PT.check_qgrad(dq.cpu().numpy(), PT.qgrad_reference(keys, q, degree=deg))
        G = eng.grad(t, tq, PT.to_dev(O), PT.to_dev(lse), PT.to_dev(dl))
        cut()
        PT.check_grad(G.cpu().numpy(), gr, ar, br, nch=nch)
        mom, v = torch.zeros(n, device=PT.DEV), torch.zeros(n, device=PT.DEV)
        loss = torch.zeros(2, device=PT.DEV, dtype=torch.float64)
        eng.fit_step(t, mom, v, 1, tq, to, loss)
        cut(rest=bool(det))
        loss = loss.cpu().numpy()
        assert abs(loss[0] - fr["loss"]) <= 1e-5 * fr["loss"] and abs(loss[1] - fr["l1"]) <= 1e-5 * fr["l1"]
        PT.check_grad(mom.cpu().numpy().astype(np.float64) / (1.0 - np.float32(0.9)), fr["grad"], ar, br, nch=nch)


@pytest.mark.gpu
@pytest.mark.parametrize("c", [c for c in CASES if not c[9]], ids=[c[0] for c in CASES if not c[9]])
def test_cut_tiles_of_every_model_in_a_batch(E, c):
    """The same crowded cells as shapes of a batch, whose tiles are cut by the
    same rule; direct launches and replays of the captured iteration."""
    name, deg, grid, moved, learn, R, P, cell, rho, _ = c
    m = V.Model(R=R, degree=deg, grid_keys=grid, moved_keys=moved, learn_scale=learn, rho_fixed=rho[0])
    th = random_theta(m, 11 + R, rho=rho, offset=0.35)
    n, nch = th.size, V.channels(m)
    rng = np.random.default_rng(P + R)
    h = 2.0 / (R - 1)
    q = (-1.0 + cell * h + h * rng.uniform(0.02, 0.98, (P, 3))).astype(np.float32)
    o = (np.linalg.norm(q, axis=1) - 0.5).astype(np.float32)
    keys = V.build_keys(m, th)
    fr = V.fit_step(m, th, np.zeros(n), np.zeros(n), 1, q, o)
    _, ak, bk = V.grad_global(keys, deg, q, 2 * (fr["O"] - o) / P, T=PT.T_TAIL)
    ar, br = V.grad_theta(m, th, ak), V.grad_theta(m, th, bk)
    tq, to = PT.to_dev(q), PT.to_dev(o)
    adam = E.efunc_default_adam()
    adam.lr = 0.0  # the second iteration meets the same parameters
    for use_graph in (False, True):
        mb, vb = ([torch.zeros(n, device=PT.DEV) for _ in range(2)] for _ in range(2))
        lb = torch.zeros(2, 2, device=PT.DEV, dtype=torch.float64)
        with E.BatchEngine([R, R], [P, P], degree=deg, grid_keys=grid, offsets=moved, learn_scale=learn,
                           rho_fixed=rho[0]) as b:
            b.bind([PT.to_dev(th).reshape(-1) for _ in range(2)], mb, vb, [tq, tq], [to, to], lb)
            for _ in range(2):
                for x in mb:
                    x.zero_()
                b.fit(1, 1, use_graph=use_graph, adam=adam)
                torch.cuda.synchronize()
                for s in range(2):
                    loss = lb[s].cpu().numpy()
                    assert abs(loss[0] - fr["loss"]) <= 1e-5 * fr["loss"] and abs(loss[1] - fr["l1"]) <= 1e-5 * fr["l1"]
                    g = mb[s].cpu().numpy().astype(np.float64) / (1.0 - np.float32(0.9))
                    PT.check_grad(g, fr["grad"], ar, br, nch=nch)


@pytest.mark.gpu
@pytest.mark.parametrize("det", [0, 1])
def test_cut_shares_the_work_among_the_launched_workgroups(E, det):
    """Equal tiles, two or more per CU: with the default tuning each is above the
    share of one of four workgroups per CU, with one workgroup per CU all are
    below its share and stay whole.  The fits agree either way."""
    R, P, tiles = 18, 60, 600
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert 2 * cus <= tiles <= 3 * cus
    th = random_theta(V.Model(R=R), 3, rho=(1.5, 2.5), offset=0.35)
    rng = np.random.default_rng(det)
    h = 2.0 / (R - 1)
    cells = rng.permutation((R - 1) ** 3)[:tiles]
    corner = np.stack([cells // (R - 1) ** 2, cells // (R - 1) % (R - 1), cells % (R - 1)], 1)
    q = (-1.0 + h * (corner[:, None, :] + rng.uniform(0.05, 0.95, (tiles, P, 3)))).reshape(-1, 3).astype(np.float32)
    o = (np.linalg.norm(q, axis=1) - 0.5).astype(np.float32)
    t, tq, to = PT.to_dev(th), PT.to_dev(q), PT.to_dev(o)
    dl = PT.to_dev(rng.standard_normal(len(q)) / len(q))
    moms, values = [], []
    with E.Engine(R, len(q), deterministic=det) as eng:
        for bpc in (8, 1):
            eng.set_tuning(group_cells=0, blocks_per_cu=bpc)

            def check():
                items = eng.items()
                assert eng.stats()["n_tiles"] == tiles
                assert items[0] > tiles if bpc == 8 else items == (tiles, 0), (bpc, items)

            O, lse, _, _ = eng.eval(t, tq)
            check()
            eng.eval(t, tq, with_qgrad=True)
            check()
            eng.grad(t, tq, O, lse, dl)
            check()
            mom, v = torch.zeros(th.size, device=PT.DEV), torch.zeros(th.size, device=PT.DEV)
            adam = E.efunc_default_adam()
            adam.lr = 0.0
            eng.fit_step(t, mom, v, 1, tq, to, None, adam)
            check()
            moms.append(mom.cpu().numpy())
            values.append(O.cpu().numpy())
    scale = np.abs(moms[0].reshape(-1, 13)).max(axis=0)
    assert np.all(np.abs(moms[0] - moms[1]).reshape(-1, 13) <= 1e-4 * np.abs(moms[0]).reshape(-1, 13) + 1e-5 * scale)
    keys = V.build_keys(V.Model(R=R), th)
    s = slice(0, len(q), 97)
    O, _, sig = V.eval_global(keys, 1, q[s])
    kap, tail = V.eval_cond(keys, 1, q[s], PT.T_TAIL, with_tail=True)
    for x in values:
        PT.check_values(x[s], O, sig, kappa=kap, tail=tail)


@pytest.mark.gpu
def test_cut_of_a_fit_counts_the_gather_of_its_keys(E):
    """A lattice of tiles of one query, each with every key in its window, and one
    tile of 40: its pieces would gather the window's keys again for a share of the
    work that the small tiles' own gathers outweigh, so a fit leaves it whole."""
    R, P = 26, 40
    th = random_theta(V.Model(R=R), 4, rho=(1.5, 2.5), offset=0.35)
    rng = np.random.default_rng(1)
    h = 2.0 / (R - 1)
    c = np.stack(np.meshgrid(*[np.arange(R - 1)] * 3, indexing="ij"), -1).reshape(-1, 3)
    crowd = np.full((P, 3), 12)
    q = (-1.0 + h * (np.concatenate([c, crowd]) + rng.uniform(0.05, 0.95, (len(c) + P, 3)))).astype(np.float32)
    o = (np.linalg.norm(q, axis=1) - 0.5).astype(np.float32)
    t, tq, to = PT.to_dev(th), PT.to_dev(q), PT.to_dev(o)
    with E.Engine(R, len(q)) as eng:
        eng.set_tuning(group_cells=0)
        mom, v = torch.zeros(th.size, device=PT.DEV), torch.zeros(th.size, device=PT.DEV)
        loss = torch.zeros(2, device=PT.DEV, dtype=torch.float64)
        O, _, _, _ = eng.eval(t, tq)
        eng.fit_step(t, mom, v, 1, tq, to, loss)
        st = eng.stats()
        assert st["W"] >= R - 2 and st["n_tiles"] == len(c) and eng.items() == (len(c), 0), (st, eng.items())
        mse = float(((O - to).double() ** 2).mean())
        assert abs(float(loss[0]) - mse) <= 1e-5 * mse


@pytest.mark.gpu
@pytest.mark.parametrize("det", [0, 1])
def test_even_launches_keep_small_tiles_whole(E, det):
    """A dense lattice of about equal tiles, two to four per CU, each up to twice the
    floor of the cut: no tile outlasts the others, so the eval and the fit leave all
    of them whole."""
    R, P = 11, 250
    th = random_theta(V.Model(R=R), 5, rho=(4.6, 5.4), offset=0.3)
    rng = np.random.default_rng(2)
    h = 2.0 / (R - 1)
    c = np.stack(np.meshgrid(*[np.arange(R - 1)] * 3, indexing="ij"), -1).reshape(-1, 1, 3)
    q = (-1.0 + h * (c + rng.uniform(0.05, 0.95, (len(c), P, 3)))).reshape(-1, 3).astype(np.float32)
    o = (np.linalg.norm(q, axis=1) - 0.5).astype(np.float32)
    t, tq, to = PT.to_dev(th), PT.to_dev(q), PT.to_dev(o)
    with E.Engine(R, len(q), deterministic=det) as eng:
        eng.set_tuning(group_cells=0)
        mom, v = torch.zeros(th.size, device=PT.DEV), torch.zeros(th.size, device=PT.DEV)
        loss = torch.zeros(2, device=PT.DEV, dtype=torch.float64)
        O, _, _, _ = eng.eval(t, tq, with_qgrad=True)
        st = eng.stats()
        assert eng.items() == (len(c), 0), eng.items()
        # the premise: window keys times queries about the floor of an eval in the mean
        # (and up to 1.4 times that, away from the lattice's faces)
        assert st["n_tiles"] == len(c) and 0.9e5 < st["window_keys"] / len(c) * P < 1.1e5, st
        eng.fit_step(t, mom, v, 1, tq, to, loss)
        assert eng.items() == (len(c), 0), eng.items()
        mse = float(((O - to).double() ** 2).mean())
        assert abs(float(loss[0]) - mse) <= 1e-5 * mse
