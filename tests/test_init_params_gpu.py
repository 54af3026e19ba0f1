"""efunc_init_params at the edges of its block sizes (4, 16 and 64 vertices per
workgroup; lattices that fill their last blocks and that do not), of its sample
chunks, and at a scale where the float32 distances cannot serve as reference,
against the oracle's mean-shift step.  The sums are FP64 on both sides, so the
offsets agree to the rounding of the float32 result (one ulp)."""
import numpy as np
import pytest
import torch

import oracle as orc
from tests import parity as PT

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,ns,scale", [(2, 1, 1.0), (5, 2049, 1.0), (16, 700, 1.0), (17, 2048, 1.0), (26, 300, 1.0),
                                        (32, 129, 1.0), (5, 3000, 1000.0)])
def test_init_params_blocks_match_oracle(R, ns, scale):
    from paper_2505_21319_amd import efunc as E
    rng = np.random.default_rng(R + ns)
    u = rng.standard_normal((ns, 3))
    surf = (scale * 0.6 * u / np.linalg.norm(u, axis=1, keepdims=True)).astype(np.float32)
    with E.Engine(R, 1, lo=-scale, hi=scale) as eng:
        th = torch.full((R, R, R, 13), 3.0, device=PT.DEV)
        eng.init_params(th, PT.to_dev(surf), 100.0, 7.0)
        torch.cuda.synchronize()
        th = th.cpu().numpy()
    D = orc.meanshift(orc.Grid(R=R, lo=-scale, hi=scale), surf.astype(np.float64), 100.0).reshape(R, R, R, 3)
    assert np.all(th[..., [0, 1, 2, 3, 8, 9, 10, 11]] == 0.0) and np.all(th[..., [4, 12]] == 7.0)
    assert np.all(np.abs(th[..., 5:8] - D) <= PT.ulp32(D) + 1e-12 * scale)
