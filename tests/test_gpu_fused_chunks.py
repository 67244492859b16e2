"""Fused subtrees of key-chunked plans: a chunk that holds one key of a step reads that key's instance of a leaf,
which is not chunked and keeps all of its keys, so the gather map is needed at width one too.

Every plan runs in one chunk first, then under budgets that go down until a chunk holds a single key (or no smaller
workspace exists); the amplitudes keep their bits throughout.
"""

import numpy as np
import pytest

from gpu_util import rel_err, require_gpu, say

pytestmark = pytest.mark.gpu


def chunk_counts(make, ref_bits):
    """The chunk counts of ever smaller budgets, each plan's amplitudes compared bit for bit with ref_bits."""
    from paper_2212_04749_amd import binding as B
    seen, budget = [], 0
    while True:
        try:
            run = make(budget)
        except B.MatncError as e:
            assert e.code == B.MATNC_E_NOMEM
            return seen
        seen.append(int(run.info.n_chunks))
        budget = int(run.info.workspace_bytes) - 1
        a = run.amplitudes()
        run.close()
        assert np.array_equal(a, ref_bits), f"{seen[-1]} chunks"


@pytest.mark.parametrize("precision", ["c64", "chalf"])
def test_single_key_chunks_read_their_leaf_instance(precision):
    """One fused slice step between two leaves of two keys each: in four chunks every chunk has one key of it, and
    three of the four need instance 1 of a leaf."""
    require_gpu()
    from paper_2212_04749_amd import api
    from paper_2212_04749_amd.circuit_tn import TensorNetwork
    rng = np.random.default_rng(61)
    # qubits 0, 1 closed, 2 .. 11 open; bond 12, sliced bond 13
    ia, ib = [0, 12, 13, 2, 3, 4, 5, 6], [1, 12, 13, 7, 8, 9, 10, 11]
    A, B = (rng.standard_normal((2,) * 8) + 1j * rng.standard_normal((2,) * 8) for _ in range(2))
    net = TensorNetwork(12, [A, B], [tuple(ia), tuple(ib)], list(range(12)), 14)
    opens = tuple(range(2, 12))
    spec = api.PlanSpec([(0, 1)], [13], opens, 32)
    words = np.arange(4, dtype=np.uint64)

    def make(budget):
        return api.Contraction(net, spec, words, precision=precision, memory_budget=budget, half_nodes=0)

    run = make(0)
    say(f"fused chunks, two leaves {precision}: workspace {run.info.workspace_bytes}")
    assert run.info.n_chunks == 1 and run.info.n_launches_per_batch == 3  # the slice is one fused subtree
    full = run.amplitudes()
    run.close()
    # amplitude (word, open bits): open qubit t is bit t of the column
    ref = np.einsum("aksuvwxy,bksUVWXY->baYXWVUyxwvu", A, B).reshape(4, 1024)
    assert rel_err(full, ref) < 4 * 2.0 ** -23
    counts = chunk_counts(make, full)
    assert counts[0] == 1 and counts[-1] == 4


@pytest.mark.parametrize("depth,k,opens,cap,batch,seed,precision", [
    (8, 4, (), 8, 8, 21, "c64"), (12, 1024, (), 10, 2, 24, "c64"), (10, 200, (2, 9), 11, 8, 22, "c64"),
    (10, 200, (2, 9), 11, 8, 22, "chalf"),
])
def test_circuits_in_ever_more_chunks(depth, k, opens, cap, batch, seed, precision):
    require_gpu()
    from paper_2212_04749_amd import api, planner
    from paper_2212_04749_amd.circuit_tn import build_network
    from workload import GridSpec, random_circuit, uniform_bitstrings
    net = build_network(random_circuit(GridSpec(4, 4), depth, seed))
    words = uniform_bitstrings(16, k, seed + 1)
    pl = planner.find_plan(net, words, opens, cap, trials=4)
    spec = api.PlanSpec(pl.pairs, pl.sliced, opens, cap)

    def make(budget):
        return api.Contraction(net, spec, words, precision=precision, slice_batch=batch, memory_budget=budget)

    run = make(0)
    say(f"fused chunks 4x4 depth {depth} k {k} {precision}: workspace {run.info.workspace_bytes}")
    full = run.amplitudes()
    run.close()
    counts = chunk_counts(make, full)
    say(f"chunk counts {counts}")
    assert counts[0] == 1 and counts[-1] > 1
