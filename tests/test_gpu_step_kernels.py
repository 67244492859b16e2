"""Steps on the kernels that take bit positions by value: split-bfloat16 tiles,
small-K, long-sum and few-output kernels, at the edges of their ranges.

Reference: the complex128 definition of the permuted pairwise step.  Tolerance
of a sum of K products: each rounding of the FP32 accumulator is at most 2^-24
of a partial sum, whose size grows as sqrt(k) for independent operands; K of
them, independent, stay below 2^-23 sqrt(K) of the result's norm (plus 2^-23
for the operands' own products).
"""

import numpy as np
import pytest

from gpu_util import assert_close, bit_positions_to_index, rel_err, require_gpu, say
from test_gpu_contract import make_case, reference, run

pytestmark = pytest.mark.gpu


def plan_layout(rng, nm, nn, nk):
    """Contracted bits highest in both operands, rows and columns interleaved in the result."""
    at = sorted(rng.permutation(nm + nn)[:nm].tolist())
    return {"posA_m": list(range(nm)), "posA_k": list(range(nm, nm + nk)),
            "posB_n": list(range(nn)), "posB_k": list(range(nn, nn + nk)),
            "posC_m": at, "posC_n": [x for x in range(nm + nn) if x not in at]}


def tolerance(nk):
    return 2.0 ** -23 * (1 + np.sqrt(2.0 ** nk))


# (m, n, k bits, instances)
STEPS = [
    # split tiles: one k step, the smallest tile, every configuration of the library's own choice
    (7, 6, 3, 3), (6, 5, 4, 1), (13, 7, 6, 4), (14, 8, 5, 2), (16, 6, 4, 1),
    # more columns than rows (operands change places), with and without tiles
    (5, 9, 8, 3), (3, 12, 5, 2), (0, 11, 2, 4), (2, 7, 0, 5),
    # small K: blocks of 16 columns, instances above and below 256 rows, one output per lane and all columns
    (8, 7, 2, 3), (10, 5, 1, 2), (11, 6, 0, 1), (7, 7, 2, 9), (4, 3, 4, 2000), (0, 0, 0, 7),
    # long sums: 1..16 columns and more, one row, rows split over groups of lanes, K below and above 256
    (9, 4, 5, 3), (5, 5, 9, 2), (10, 1, 11, 5), (6, 0, 12, 1), (12, 2, 6, 2), (4, 4, 7, 3), (7, 3, 8, 40),
    # few outputs: a block per instance (256 and 512 lanes) and a wave per instance
    (0, 0, 13, 3), (3, 3, 9, 2), (1, 2, 5, 600), (0, 0, 9, 1500), (3, 1, 5, 1024), (2, 3, 7, 1027),
]


@pytest.mark.parametrize("layout", ["plan", "shuffled"])
@pytest.mark.parametrize("nm,nn,nk,batch", STEPS)
def test_library_choice(nm, nn, nk, batch, layout):
    torch = require_gpu()
    rng = np.random.default_rng(7000 + 100 * nm + 10 * nn + nk)
    pos, A, B = make_case(rng, nm, nn, nk, batch)
    if layout == "plan":
        pos = plan_layout(rng, nm, nn, nk)
    say(f"step {nm}/{nn}/{nk} x {batch} {layout}")
    got = run(torch, pos, A, B, nm, nn, nk, -1)
    assert rel_err(got, reference(pos, A, B, nm, nn, nk)) < tolerance(nk)


@pytest.mark.parametrize("scale_a,scale_b", [(1e-38, 1e8), (1e-41, 1e12), (1e18, 1e15), (1e-20, 1e-12)])
def test_split_tiles_keep_operand_bits_at_any_scale(scale_a, scale_b):
    """Denormal and tiny operands keep all their bits, sums above the scaled range are computed again in FP32."""
    torch = require_gpu()
    rng = np.random.default_rng(41)
    nm, nn, nk, batch = 9, 6, 5, 2
    pos, A, B = make_case(rng, nm, nn, nk, batch)
    A, B = (A * np.float32(scale_a)).astype(np.complex64), (B * np.float32(scale_b)).astype(np.complex64)
    say(f"split tile scales {scale_a:g} {scale_b:g}")
    got = run(torch, pos, A, B, nm, nn, nk, 101)
    assert rel_err(got, reference(pos, A, B, nm, nn, nk)) < tolerance(nk)


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, np.finfo(np.float32).max])
def test_split_tiles_non_finite(value):
    """One non-finite (or largest) component of A: the outputs of its row are what FP32 products give, the
    others do not change."""
    torch = require_gpu()
    rng = np.random.default_rng(43)
    nm, nn, nk = 8, 6, 4
    pos, A, B = make_case(rng, nm, nn, nk, 1)
    plain = run(torch, pos, A, B, nm, nn, nk, 101)
    am = bit_positions_to_index(pos["posA_m"], nm)
    ak = bit_positions_to_index(pos["posA_k"], nk)
    row, k = 77, 11
    parts = A.view(np.float32).reshape(1, -1, 2)
    parts[0, am[row] + ak[k], 0] = value
    say(f"split tile non-finite {value}")
    got = run(torch, pos, A, B, nm, nn, nk, 101)
    cm = bit_positions_to_index(pos["posC_m"], nm)[:, None] + bit_positions_to_index(pos["posC_n"], nn)[None, :]
    others = np.delete(cm, row, axis=0).reshape(-1)
    # (waves that hold the row run in FP32, so the rest of their tile may differ in the last bits)
    assert rel_err(got[0][others], plain[0][others]) < tolerance(nk)
    b = B[0][bit_positions_to_index(pos["posB_k"], nk)[k] + bit_positions_to_index(pos["posB_n"], nn)]
    if np.isfinite(value):
        ref = reference(pos, A, B, nm, nn, nk)[0][cm[row]]
        for g, r in ((got[0][cm[row]].real, ref.real), (got[0][cm[row]].imag, ref.imag)):
            top = float(np.finfo(np.float32).max)
            assert np.all(np.isinf(g[np.abs(r) > 1.0001 * top])) and np.all(np.isfinite(g[np.abs(r) < 0.9999 * top]))
    else:
        assert np.array_equal(got[0][cm[row]].real, value * b.real.astype(np.float64), equal_nan=True)
        assert np.array_equal(got[0][cm[row]].imag, value * b.imag.astype(np.float64), equal_nan=True)


@pytest.mark.parametrize("precision", ["c64", "chalf"])
def test_split_sums_with_and_without_room(precision):
    """A branch step with a long sum and few tiles (16 instances of 6/2/11 bits that share A) runs in parts, the
    same ones however the keys are chunked, and in one piece when the budget has no room for a single key's."""
    require_gpu()
    from paper_2212_04749_amd import api
    from paper_2212_04749_amd.circuit_tn import TensorNetwork
    rng = np.random.default_rng(47)
    # A[m x 6, k x 11], B[q x 4, k x 11, n x 2], D[m x 6, n x 2]
    q, k, m, n = list(range(4)), list(range(4, 15)), list(range(15, 21)), list(range(21, 23))
    draw = lambda ix: rng.standard_normal((2,) * len(ix)) + 1j * rng.standard_normal((2,) * len(ix))  # noqa: E731
    A, B, D = draw(m + k), draw(q + k + n), draw(m + n)
    net = TensorNetwork(4, [A, B, D], [tuple(m + k), tuple(q + k + n), tuple(m + n)], q, 23)
    spec = api.PlanSpec([(0, 1), (3, 2)], [], (), 32)
    words = np.arange(16, dtype=np.uint64)
    C = np.einsum("mk,qkn->qmn", A.reshape(64, 2048), B.reshape(16, 2048, 4))
    amps = np.einsum("qmn,mn->q", C, D.reshape(64, 4)).reshape(2, 2, 2, 2)
    ref = np.array([amps[w & 1, (w >> 1) & 1, (w >> 2) & 1, (w >> 3) & 1] for w in range(16)])
    def contract(budget):
        run = api.Contraction(net, spec, words, precision=precision, memory_budget=budget)
        assert run.info.n_fan_nodes == 1
        say(f"split sums {precision}: workspace {run.info.workspace_bytes}, {run.info.n_chunks} key chunks")
        a = run.amplitudes()
        assert np.array_equal(a, run.amplitudes())
        assert rel_err(a, ref) < tolerance(11) + tolerance(8)
        out = a, int(run.info.workspace_bytes), int(run.info.n_chunks)
        run.close()
        return out

    full, need, chunks = contract(0)
    assert chunks == 1
    while chunks < 16:  # smaller budgets: more key chunks, the same parts, the same bits
        a, need, chunks = contract(need - 1)
        assert np.array_equal(a, full)
    a, less, chunks = contract(need - 1)  # not even one key's parts fit: the sum in one piece
    assert less < need and not np.array_equal(a, full)


@pytest.mark.parametrize("precision,opens,cap,batch", [("c64", (), 4, 3), ("c64", (2, 9), 6, 2), ("chalf", (), 5, 4)])
def test_fused_slices(precision, opens, cap, batch):
    """Small circuits whose slices are fused subtrees, whole or in part: more slices than one launch takes, ranges that cut
    it anywhere, the one-by-one pass and the queue give the same bits; against the state vector."""
    torch = require_gpu()
    from oracle import statevector
    from paper_2212_04749_amd import api, planner
    from paper_2212_04749_amd.circuit_tn import build_network
    from workload import GridSpec, random_circuit, uniform_bitstrings
    circ = random_circuit(GridSpec(3, 4), 8, 51)
    words = uniform_bitstrings(12, 37, 52)
    net = build_network(circ)
    pl = planner.find_plan(net, words, opens, cap, trials=4, refine_top=0)
    spec = api.PlanSpec(pl.pairs, pl.sliced, opens, cap)
    run = api.Contraction(net, spec, words, precision=precision, slice_batch=batch)
    n = run.n_slices
    say(f"fused slices {precision}: {n} slices, {run.info.n_launches_per_batch} launches per batch")
    if not opens:  # one subtree per slice (with open legs the last steps are launches of their own)
        assert run.info.n_launches_per_batch == 3
    if not opens and precision == "c64":
        assert n > 1024
    full = run.execute()
    run.synchronize()
    full = full.cpu().numpy()
    parts = run.new_amplitudes()
    for lo, hi in ((0, 1), (1, n // 3), (n // 3, n // 3), (n // 3, n - 1), (n - 1, n)):
        run.execute(parts, lo, hi)
    run.synchronize()
    assert np.array_equal(full, parts.cpu().numpy())
    timed = run.new_amplitudes()
    run.execute_timed(timed, len(net.tensors) - 2)
    assert np.array_equal(full, timed.cpu().numpy())
    queue = api.Queue([run])
    for _ in range(2):
        amps, _ = queue.execute()
        torch.cuda.synchronize()
        assert np.array_equal(full, amps[0].cpu().numpy())
    queue.close()
    psi = statevector.final_state(circ)
    rows = []
    for w0 in words:
        for j in range(1 << len(opens)):
            word = int(w0)
            for t, q in enumerate(opens):
                word = (word & ~(1 << q)) | (((j >> t) & 1) << q)
            rows.append(word)
    assert_close(full[..., 0] + 1j * full[..., 1], statevector.amplitudes_from_state(psi, rows), 1e-5)
    run.close()


@pytest.mark.parametrize("precision", ["c64", "chalf"])
def test_invariant_steps_from_a_graph(precision):
    """An unsliced plan run again and again (its steps are replayed from a graph from the second time on), with other
    work between and new numbers in a tensor: the bits of a plan on the default stream, which never captures; and the
    same under a capture of the caller's, which leaves nothing in the cache."""
    torch = require_gpu()
    from paper_2212_04749_amd import api, planner
    from paper_2212_04749_amd.circuit_tn import build_network
    from workload import GridSpec, random_circuit, uniform_bitstrings
    net = build_network(random_circuit(GridSpec(4, 4), 10, 57))
    words = uniform_bitstrings(16, 40, 58)
    pl = planner.find_plan(net, words, (), 30, trials=4, refine_top=0)
    spec = api.PlanSpec(pl.pairs, pl.sliced, (), 30)
    eager = api.Contraction(net, spec, words, precision=precision, stream=torch.cuda.default_stream())
    run = api.Contraction(net, spec, words, precision=precision)
    assert run.n_slices == 1
    t = max(range(len(run.net.tensors)), key=lambda i: run.net.tensors[i].size)
    data = np.array(run.net.tensors[t])
    noise, amps = torch.zeros(1 << 20, device="cuda"), run.new_amplitudes()
    eager.amplitudes(), run.amplitudes()

    def want(scale):
        eager.set_tensor(t, data * scale)
        return eager.amplitudes()

    for scale in (1.0, 0.5, 0.75, -3.0, 1.0):
        noise += 1.0
        run.set_tensor(t, data * scale)
        got = run.amplitudes()
        run.reset_cache()
        torch.cuda.synchronize()
        noise += 1.0
        ref = want(scale)
        assert np.array_equal(got, ref) and np.array_equal(run.amplitudes(), ref)
    ref = want(2.0)
    run.set_tensor(t, data * 2.0)
    run.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=run.stream):
        amps.zero_()
        run.execute(amps)
    assert np.array_equal(run.amplitudes(), ref)  # the capture ran nothing, and the cache does not claim that it did
    for _ in range(3):
        noise += 1.0
        amps.fill_(7.0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        a = amps.cpu().numpy()
        assert np.array_equal(a[..., 0] + 1j * a[..., 1], ref.reshape(a.shape[:-1]))
        assert np.array_equal(run.amplitudes(), ref)
    torch.cuda.synchronize()
    run.close(), eager.close()


@pytest.mark.parametrize("batch", [1, 3])
def test_fused_slices_without_room(batch):
    """One amplitude of a plan whose slice is one subtree: a budget without room for more slices per launch than the
    slice batch is still enough, with the same bits."""
    require_gpu()
    from paper_2212_04749_amd import api, planner
    from paper_2212_04749_amd.circuit_tn import build_network
    from workload import GridSpec, random_circuit, uniform_bitstrings
    net = build_network(random_circuit(GridSpec(3, 4), 8, 51))
    words = uniform_bitstrings(12, 1, 52)
    pl = planner.find_plan(net, words, (), 5, trials=4, refine_top=0)
    spec = api.PlanSpec(pl.pairs, pl.sliced, (), 5)
    run = api.Contraction(net, spec, words, slice_batch=batch)
    need, n, full = int(run.info.workspace_bytes), run.n_slices, run.amplitudes()
    run.close()
    assert n > 32 * batch
    run = api.Contraction(net, spec, words, slice_batch=batch, memory_budget=need - 1)
    say(f"fused slices without room: {n} slices, {need} and {run.info.workspace_bytes} bytes")
    assert int(run.info.workspace_bytes) < need
    assert np.array_equal(run.amplitudes(), full) and np.array_equal(run.amplitudes(), full)
    run.close()
