"""Keys of the tuning file: a step on the split-bfloat16 tiles and one on the FP32 instruction never share a choice."""

import json

import pytest

from gpu_util import assert_close, require_gpu, say
from oracle import statevector
from test_gpu_batching import build
from workload import GridSpec, random_circuit, uniform_bitstrings

pytestmark = pytest.mark.gpu


def last(key):
    return int(key.rsplit("/", 1)[1])


def test_split_and_fp32_steps_have_keys_of_their_own(tmp_path):
    require_gpu()
    from paper_2212_04749_amd import api
    circ = random_circuit(GridSpec(4, 5), 12, 21)
    words = uniform_bitstrings(20, 128, 22)
    ref = statevector.amplitudes(circ, words)
    path = str(tmp_path / "tune.json")
    run, spec = build(circ, words, 13, 4)
    run.autotune(reps=1, cache_path=path)
    with open(path) as f:
        split = json.load(f)
    say(f"tuning keys: {sorted(split)}")
    assert split and all(k.startswith("c64/f/") and last(k) >= 100 for k in split)
    # a file from before the split tiles: its choices stay there and decide nothing
    old = {k.rsplit("/", 1)[0] + f"/{last(k) % 100}": 2 for k in split}
    with open(path, "w") as f:
        json.dump(old, f)
    run.autotune(reps=1, cache_path=path)
    with open(path) as f:
        both = json.load(f)
    assert set(both) == set(old) | set(split) and all(both[k] == 2 for k in old)
    assert_close(run.amplitudes(), ref, 1e-5)
    # the same steps of a complex-half plan with FP16 tensors run on the FP32 instruction
    half = api.Contraction(run.net, spec, words, precision="chalf", slice_batch=4, half_nodes=2)
    half.autotune(reps=1, cache_path=path)
    with open(path) as f:
        keys = [k for k in json.load(f) if k.startswith("chalf/f/")]
    assert keys and all(last(k) < 100 for k in keys)
    half.close()
    run.close()
