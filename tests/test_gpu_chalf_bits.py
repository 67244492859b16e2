"""Complex-half plans with one and two FP16-stored tensors: their FP32-stored steps run on the FP32 matrix
instruction with its own order of additions, so the amplitudes are those of the stored runs bit for bit.

tests/golden/chalf_fp32_steps.json holds the float64 amplitude buffers (hexadecimal) of a 20-qubit circuit, unsliced
and in 128 slices, recorded when every FP32-stored step of a complex-half plan ran on that instruction.
"""

import json
import os

import numpy as np
import pytest

from gpu_util import assert_close, require_gpu, say

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "chalf_fp32_steps.json")


@pytest.mark.parametrize("which", range(4))
def test_fp32_steps_of_plans_with_fp16_tensors_keep_their_bits(which):
    require_gpu()
    from oracle import statevector
    from paper_2212_04749_amd import api
    from paper_2212_04749_amd.circuit_tn import build_network
    from workload import GridSpec, random_circuit, uniform_bitstrings
    with open(GOLDEN) as f:
        g = json.load(f)
    r = g["runs"][which]
    circ = random_circuit(GridSpec(g["rows"], g["cols"]), g["depth"], g["seed"])
    words = uniform_bitstrings(g["rows"] * g["cols"], g["k"], g["words_seed"])
    spec = api.PlanSpec([tuple(p) for p in r["pairs"]], r["sliced"], (), r["cap"])
    run = api.Contraction(build_network(circ), spec, words, precision="chalf", slice_batch=2,
                          half_nodes=r["half_nodes"])
    assert run.info.n_half_nodes == r["half_nodes"]
    say(f"chalf bits: {run.n_slices} slices, {run.info.n_half_nodes} FP16 tensors")
    amps = run.execute()
    run.synchronize()
    amps = amps.cpu().numpy().reshape(-1)
    want = np.array([float.fromhex(v) for v in r["amps"]])
    # each FP16 tensor rounds by 2^-11 of its largest entry or less
    ref = statevector.amplitudes_from_state(statevector.final_state(circ), [int(w) for w in words])
    assert_close(want[0::2] + 1j * want[1::2], ref, 2.0 ** -9)
    assert np.array_equal(amps, want)
    run.close()
