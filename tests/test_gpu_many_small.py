"""Small sums over more instances than there are blocks: a block takes several (the last turn a part of one)."""

import numpy as np
import pytest

from gpu_util import rel_err, require_gpu
from test_gpu_contract import make_case, reference, run
from test_gpu_step_kernels import plan_layout

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shuffled", [False, True])
@pytest.mark.parametrize("nm,nn,nk,batch", [(8, 0, 0, 5000), (8, 0, 1, 2049), (7, 1, 0, 4099), (3, 2, 1, 70001), (5, 0, 3, 20001),
                                            (8, 1, 1, 4097), (8, 2, 2, 2048), (10, 0, 0, 2051), (9, 1, 0, 4096), (9, 0, 1, 2047),
                                            (8, 0, 4, 2049)])
def test_every_instance_is_computed(nm, nn, nk, batch, shuffled):
    torch = require_gpu()
    rng = np.random.default_rng(100 * nk + nm)
    pos, A, B = make_case(rng, nm, nn, nk, batch)
    if not shuffled:
        pos = plan_layout(rng, nm, nn, nk)
    got, want = run(torch, pos, A, B, nm, nn, nk, 0), reference(pos, A, B, nm, nn, nk)
    # a component is 2 K rounded multiply-adds: off by 2 K 2^-24 of its terms' sum, which is at most
    # sqrt(2 K) times their rms, and so sqrt(2 K) times the result's
    assert rel_err(got, want) < (2 << nk) * 2.0**-24 * np.sqrt(2 << nk)
