"""Workspace budgets (host code only): room that a plan can do without is given up before the keys are cut into
chunks, as it makes no difference to results while each further chunk repeats work."""

import numpy as np
import pytest

from paper_2212_04749_amd import api, binding as B, planner
from paper_2212_04749_amd.circuit_tn import TensorNetwork, build_network
from workload import GridSpec, random_circuit, uniform_bitstrings


def figures(net, pairs, sliced, words, batch, budget):
    ranks, ids, data = api.network_arrays(net)
    h = B.matnc_network_create(ranks, ids, data, net.n_qubits, net.output_index)
    try:
        p = B.matnc_plan_create_ex(h, pairs, sliced, [], words, B.MATNC_C64, 32, batch, budget, -1)
        info = B.matnc_plan_info(p)
        B.matnc_plan_destroy(p)
        return int(info.workspace_bytes), int(info.n_chunks)
    finally:
        B.matnc_network_destroy(h)


def test_fused_slices_give_up_slices_per_launch_first():
    net = build_network(random_circuit(GridSpec(3, 4), 8, 51))
    words = uniform_bitstrings(12, 37, 52)
    pl = planner.find_plan(net, words, (), 4, trials=4, refine_top=0)
    need, chunks = figures(net, pl.pairs, pl.sliced, words, 3, 0)
    assert chunks == 1
    root = len(words) * 8  # a slice's results
    for less in (1, root, 100 * root, 1000 * root):
        got, chunks = figures(net, pl.pairs, pl.sliced, words, 3, need - less)
        assert chunks == 1 and need - less - 2 * root - 256 < got <= need - less


def split_sum_network(slices):
    """A[m x 6, k x 11, s] and B[q x 4, k x 11, n x 2, s], closed with D[m x 6, n x 2]: a long sum in few tiles."""
    q, k, m, n = list(range(4)), list(range(4, 15)), list(range(15, 21)), list(range(21, 23))
    s = list(range(23, 23 + slices))
    rng = np.random.default_rng(47)
    draw = lambda ix: rng.standard_normal((2,) * len(ix)) + 1j * rng.standard_normal((2,) * len(ix))  # noqa: E731
    A, Bt, D = draw(m + k + s), draw(q + k + n + s), draw(m + n)
    net = TensorNetwork(4, [A, Bt, D], [tuple(m + k + s), tuple(q + k + n + s), tuple(m + n)], q, 23 + slices)
    return net, [(0, 1), (3, 2)], s


@pytest.mark.parametrize("batch", [2, 8])
def test_split_sums_go_slice_by_slice_first(batch):
    net, pairs, s = split_sum_network(3)
    words = np.arange(16, dtype=np.uint64)
    one, _ = figures(net, pairs, s, words, 1, 0)
    need, chunks = figures(net, pairs, s, words, batch, 0)
    assert chunks == 1 and need > one
    # a slice's results and its share of the last step's: all that every further slice of a batch has to take
    results = 16 * (8 * 2 ** 8 + 8)
    got, chunks = figures(net, pairs, s, words, batch, need - 1)
    assert chunks == 1 and got < need and got <= one + (batch - 1) * (results + 256)
