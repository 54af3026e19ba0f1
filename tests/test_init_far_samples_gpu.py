"""efunc_init_params with a bandwidth so small, or a lattice so small, that
samples of weights that add up to e^-39 lie far enough away to move the weighted
mean: they must not be passed over.  Against the oracle's mean-shift step, to the rounding of the
float32 result (one ulp), as the sums are FP64 on both sides."""
import numpy as np
import pytest
import torch

import oracle as orc
from tests import parity as PT


def samples(bw, half, n):
    """n samples about the lattice, then n at a weight of e^-39.5 / 2 n (runs of as
    many as a workgroup's waves look at together)."""
    u = np.random.default_rng(n).standard_normal((n, 3))
    near = 0.6 * half * u / np.linalg.norm(u, axis=1, keepdims=True)
    far = np.tile([[np.sqrt((39.5 + np.log(2 * n)) / bw), 0.0, 0.0]], (n, 1))
    return np.concatenate([near, far]).astype(np.float32)


CASES = [(3, 1e-24, 1.0, 256), (9, 1e-20, 1.0, 256), (17, 1e-24, 1.0, 64), (33, 1e-20, 1.0, 2), (5, 1.0, 1e-10, 256)]


@pytest.mark.parametrize("R,bw,half,ns", CASES)
def test_the_far_samples_matter(R, bw, half, ns):
    """The premise of the cases: without the far samples some offsets are off by
    more than the tolerance below."""
    bw, half, s = float(np.float32(bw)), float(np.float32(half)), samples(bw, half, ns).astype(np.float64)
    g = orc.Grid(R=R, lo=-half, hi=half)
    D, D0 = orc.meanshift(g, s, bw), orc.meanshift(g, s[:ns], bw)
    assert np.any(np.abs(D - D0) > 4 * (PT.ulp32(D) + 1e-12 * half))


@pytest.mark.gpu
@pytest.mark.parametrize("R,bw,half,ns", CASES)
def test_far_samples_are_not_passed_over(R, bw, half, ns):
    from paper_2505_21319_amd import efunc as E
    bw, half, s = float(np.float32(bw)), float(np.float32(half)), samples(bw, half, ns)
    with E.Engine(R, 1, lo=-half, hi=half) as eng:
        th = torch.zeros(R ** 3, 13, device=PT.DEV)
        eng.init_params(th, PT.to_dev(s), bw, 7.0)
        torch.cuda.synchronize()
        got = th[:, 5:8].cpu().numpy()
    D = orc.meanshift(orc.Grid(R=R, lo=-half, hi=half), s.astype(np.float64), bw).reshape(-1, 3)
    assert np.all(np.abs(got - D) <= PT.ulp32(D) + 1e-12 * half)
