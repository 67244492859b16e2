"""Long sums with few outputs, as single steps: no further from 64 bits than 256 / 2^(m bits) lanes with a run of the
sum each, added one by one (for the figure see test_gpu_fused_sums)."""

import numpy as np
import pytest

from gpu_util import rel_err, require_gpu, say
from test_gpu_contract import make_case, reference, run
from test_gpu_split_accuracy import ROUNDING
from test_gpu_step_kernels import plan_layout

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nm,nn,nk,batch", [(1, 0, 11, 223), (0, 0, 9, 500), (0, 0, 12, 300), (3, 3, 9, 100), (2, 1, 7, 511),
                                            (0, 0, 9, 1500), (3, 1, 5, 1024), (5, 2, 8, 64), (9, 4, 5, 3), (6, 0, 12, 40),
                                            (3, 3, 9, 1024), (3, 0, 11, 1100), (0, 0, 12, 1024), (2, 2, 8, 1030)])
def test_no_further_off_than_lane_sums_one_by_one(nm, nn, nk, batch):
    torch = require_gpu()
    rng = np.random.default_rng(100 * nk + nm)
    _, A, B = make_case(rng, nm, nn, nk, batch)
    pos = plan_layout(rng, nm, nn, nk)
    K = 1 << nk
    lanes = min(256 >> min(nm, 8), K)
    L = K // lanes
    E = lanes * (L * L + L / 2) + L * (lanes * (lanes + 1) / 2 - 1)
    e = rel_err(run(torch, pos, A, B, nm, nn, nk, 0), reference(pos, A, B, nm, nn, nk))
    # (a few hundred outputs: 8% of statistics)
    tol = 1.08 * ROUNDING * np.sqrt(E / K)
    say(f"long sums {nm}/{nn}/{nk} x {batch}: {e:.2e}, one by one {tol:.2e}")
    assert e < tol
