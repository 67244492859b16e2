"""Long sums inside fused subtrees: no further from 64 bits than the long-sum kernel that runs them otherwise, and the
same bits in any slice batch and key chunk.

Tolerance: that kernel gives every lane of 256 / 2^(m bits) a run of L products and adds the lanes' sums one by one.
With roundings of 2.53e-8 of a value (rms; see test_gpu_split_accuracy) that is 2.53e-8 sqrt(E / K) of a sum of K
independent complex products, E = lanes (L^2 + L / 2) + L (2 + 3 + .. + lanes); 10% for the statistics.
"""

import numpy as np
import pytest

from gpu_util import rel_err, require_gpu, say
from test_gpu_split_accuracy import ROUNDING

pytestmark = pytest.mark.gpu


def network(rng, kb, keys, m, n, slices):
    """A[a.., s, k.., m..] and B[b.., s, n.., k..]: `keys` closed qubits each (one at 0 where keys is 0), m and n open
    qubits, sliced s.  Returns the network, sliced ids, open qubits, words and amplitudes."""
    from paper_2212_04749_amd.circuit_tn import TensorNetwork
    words = np.arange(1 << (2 * keys), dtype=np.uint64)
    keys = max(keys, 1)
    out = 2 * keys + m + n
    bond, sl = list(range(out, out + kb)), list(range(out + kb, out + kb + slices))
    qa, qb = list(range(keys)), list(range(keys, 2 * keys))
    om, on = list(range(2 * keys, 2 * keys + m)), list(range(2 * keys + m, out))
    ia, ib = qa + sl + bond + om, qb + sl + on + bond

    def draw(ix):
        z = rng.standard_normal((2,) * len(ix)) + 1j * rng.standard_normal((2,) * len(ix))
        return z.astype(np.complex64).astype(np.complex128)
    A, B = draw(ia), draw(ib)
    net = TensorNetwork(out, [A, B], [tuple(ia), tuple(ib)], list(range(out)), out + kb + slices)
    S, K, Q = 1 << slices, 1 << kb, 1 << keys
    amps = np.einsum("xskm,ysnk->xymn", A.reshape(Q, S, K, 1 << m), B.reshape(Q, S, 1 << n, K))
    return net, sl, tuple(range(2 * keys, out)), words, amps


def reversed_bits(n):
    x = np.arange(1 << n)
    return sum(((x >> t) & 1) << (n - 1 - t) for t in range(n)) if n else x


@pytest.mark.parametrize("kb,keys,m,n", [(5, 2, 0, 0), (7, 1, 0, 0), (10, 1, 0, 0), (12, 0, 0, 0), (6, 1, 2, 1), (5, 1, 4, 3),
                                         (8, 0, 4, 1)])
def test_long_sums_in_a_fused_step(kb, keys, m, n):
    require_gpu()
    from paper_2212_04749_amd import api
    err2 = ref2 = 0.0
    K = 1 << kb
    for seed in range(8 if keys or m else 32):
        rng = np.random.default_rng(1000 * kb + seed)
        net, sl, opens, words, amps = network(rng, kb, keys, m, n, 2)
        run = api.Contraction(net, api.PlanSpec([(0, 1)], sl, opens, 32), words, slice_batch=3)
        assert run.info.n_launches_per_batch == 3  # one fused subtree a slice
        got = run.execute()
        run.synchronize()
        got = got.cpu().numpy()
        parts = run.new_amplitudes()
        for s in range(run.n_slices):
            run.execute(parts, s, s + 1)
        run.synchronize()
        assert np.array_equal(parts.cpu().numpy(), got)
        run.close()
        got = got[..., 0] + 1j * got[..., 1]
        # word bit t is closed qubit t; the open qubits in ascending order, the first lowest
        w, o = reversed_bits(max(keys, 1)), reversed_bits(m)
        ref = np.empty_like(got)
        for word in range(1 << (2 * keys)):
            x, y = w[word & ((1 << keys) - 1)], w[word >> keys]
            for col in range(1 << (m + n)):
                ref[word, col] = amps[x, y, o[col & ((1 << m) - 1)], reversed_bits(n)[col >> m]]
        err2 += np.sum(np.abs(got - ref) ** 2)
        ref2 += np.sum(np.abs(ref) ** 2)
    lanes = min(256 >> max(m, n), K)
    L = K // lanes
    E = lanes * (L * L + L / 2) + L * (lanes * (lanes + 1) / 2 - 1)
    e, tol = np.sqrt(err2 / ref2), 1.1 * ROUNDING * np.sqrt(E / K)
    say(f"fused sums {m}/{n}/{kb}, {1 << (2 * keys)} keys: {e:.2e}, long-sum kernel {tol:.2e}")
    assert e < tol


def test_long_fused_sums_in_key_chunks():
    require_gpu()
    from paper_2212_04749_amd import api, binding as B
    net, sl, opens, words, _ = network(np.random.default_rng(5), 6, 2, 2, 2, 3)

    def make(budget):
        return api.Contraction(net, api.PlanSpec([(0, 1)], sl, opens, 32), words, slice_batch=4, memory_budget=budget)

    run = make(0)
    full, need = run.amplitudes(), int(run.info.workspace_bytes)
    run.close()
    chunks = []
    while True:
        try:
            run = make(need - 1)
        except B.MatncError:
            break
        need = int(run.info.workspace_bytes)
        chunks.append(int(run.info.n_chunks))
        assert np.array_equal(run.amplitudes(), full), chunks
        run.close()
    say(f"fused sums: chunks {chunks}")
    assert chunks
