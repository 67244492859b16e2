"""Plans whose budget leaves no room for split sums of a whole slice batch, or for many fused slices per launch: the
same amplitudes, bit for bit."""

import numpy as np
import pytest

from gpu_util import rel_err, require_gpu, say
from test_gpu_step_kernels import tolerance
from test_memory_budget import split_sum_network

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [1, 3, 8])
def test_split_sums_slice_by_slice(batch):
    require_gpu()
    from paper_2212_04749_amd import api
    net, pairs, s = split_sum_network(3)
    words = np.arange(16, dtype=np.uint64)
    A, B, D = net.tensors
    C = np.einsum("mks,qkns->qmn", A.reshape(64, 2048, 8), B.reshape(16, 2048, 4, 8))
    amps = np.einsum("qmn,mn->q", C, D.reshape(64, 4)).reshape(2, 2, 2, 2)
    ref = np.array([amps[w & 1, (w >> 1) & 1, (w >> 2) & 1, (w >> 3) & 1] for w in range(16)])
    full, need = None, 0
    for _ in range(4):
        run = api.Contraction(net, api.PlanSpec(pairs, s, (), 32), words, slice_batch=batch,
                              memory_budget=need - 1 if need else 0)
        need = int(run.info.workspace_bytes)
        say(f"split sums, batch {batch}: workspace {need}, {run.info.n_chunks} chunks")
        a = run.amplitudes()
        timed = run.new_amplitudes()
        run.execute_timed(timed, 0)
        timed = timed.cpu().numpy()
        run.close()
        if full is None:
            full = a
            assert rel_err(a, ref) < tolerance(11) + tolerance(8)
        assert np.array_equal(a, full)
        assert np.array_equal(timed[:, 0, 0] + 1j * timed[:, 0, 1], full)


def test_fused_slices_with_room_for_some():
    require_gpu()
    from paper_2212_04749_amd import api, planner
    from paper_2212_04749_amd.circuit_tn import build_network
    from workload import GridSpec, random_circuit, uniform_bitstrings
    net = build_network(random_circuit(GridSpec(3, 4), 8, 51))
    words = uniform_bitstrings(12, 37, 52)
    pl = planner.find_plan(net, words, (), 4, trials=4, refine_top=0)
    spec = api.PlanSpec(pl.pairs, pl.sliced, (), 4)
    full = None
    for less in (0, 1, 200 * 37 * 8, 1000 * 37 * 8):
        run = api.Contraction(net, spec, words, slice_batch=3, memory_budget=need - less if less else 0)
        if full is None:
            need, full = int(run.info.workspace_bytes), run.amplitudes()
        say(f"fused slices: workspace {run.info.workspace_bytes}")
        assert run.info.n_chunks == 1 and np.array_equal(run.amplitudes(), full)
        run.close()
