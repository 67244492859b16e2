"""The split-bfloat16 tiles against 64 bits: no further off than an FP32 sum that rounds once for every real product.

Tolerance.  Rounding to nearest leaves a uniform error of at most half a unit of the last place; for a value anywhere
in a binade (log-uniform) that is 2^-23 sqrt(3 / (8 ln 2)) / sqrt(12) = 2.53e-8 of it (rms).  A sum of N independent
products rounded after each of them is off by that times sqrt(1 + 2 + .. + N) of a product, so by
2.53e-8 sqrt((N + 1) / 2) of the result; 5% are left for the statistics of a few thousand outputs.  A sum of one
product is one rounding: 2^-24 of it at most, and 2^-28 for what the smaller parts lose.
"""

import numpy as np
import pytest

from gpu_util import bit_positions_to_index, rel_err, require_gpu, say
from test_gpu_contract import run
from test_gpu_step_kernels import plan_layout

pytestmark = pytest.mark.gpu

ROUNDING = 2.0 ** -23 * np.sqrt(3 / (8 * np.log(2))) / np.sqrt(12)


def multiply(torch, rng, A, B, kernel):
    """A @ B through one pairwise step, and in 64 bits."""
    nm, nk = (int(np.log2(x)) for x in A.shape)
    nn = int(np.log2(B.shape[1]))
    A, B = A.astype(np.complex64), B.astype(np.complex64)
    pos = plan_layout(rng, nm, nn, nk)
    ix = {name: bit_positions_to_index(p, len(p)) for name, p in pos.items()}
    a, b = np.zeros((1, A.size), np.complex64), np.zeros((1, B.size), np.complex64)
    a[0][ix["posA_m"][:, None] + ix["posA_k"][None, :]] = A
    b[0][ix["posB_k"][:, None] + ix["posB_n"][None, :]] = B
    got = run(torch, pos, a, b, nm, nn, nk, kernel)[0]
    return got[ix["posC_m"][:, None] + ix["posC_n"][None, :]], A.astype(np.complex128) @ B.astype(np.complex128)


@pytest.mark.parametrize("nk,kernel", [(3, -1), (5, -1), (9, -1), (10, -1)] + [(7, 100 + c) for c in range(6)])
@pytest.mark.parametrize("operands", ["normal", "positive", "half zeros", "one per k step, real", "one, complex"])
def test_no_further_off_than_fp32_sums(operands, nk, kernel):
    torch = require_gpu()
    rng = np.random.default_rng(100 * nk + kernel)
    K = 1 << nk
    A = rng.standard_normal((512, K)) + 1j * rng.standard_normal((512, K))
    B = rng.standard_normal((K, 128)) + 1j * rng.standard_normal((K, 128))
    keep = np.ones(A.shape)
    products = 2 * K
    if operands == "positive":
        # (partial sums grow as j, not sqrt(j): the sum of their squares is N / 3 of the square of the result)
        A, B = np.abs(A.real) + 0j, np.abs(B.real) + 0j
        products = 2 * K / 3 - 1
    if operands == "half zeros":
        keep = rng.random(A.shape) < 0.5
        products = K
    if operands.startswith("one"):
        step = 8 if operands.startswith("one per") else K
        keep[:] = 0
        for s in range(0, K, step):
            keep[np.arange(512), s + rng.integers(0, step, 512)] = 1
        products = 2
        if operands.endswith("real"):
            A, B = A.real + 0j, B.real + 0j
            products = K // 8
    got, ref = multiply(torch, rng, A * keep, B, kernel)
    e, tol = rel_err(got, ref), 1.05 * ROUNDING * np.sqrt((products + 1) / 2)
    say(f"split accuracy {operands} k {nk} kernel {kernel}: {e:.2e}, FP32 sums {tol:.2e}")
    assert e < tol


@pytest.mark.parametrize("kernel", range(100, 106))
def test_a_single_product_is_rounded_once(kernel):
    torch = require_gpu()
    rng = np.random.default_rng(kernel)
    A, B = rng.standard_normal((512, 16)), rng.standard_normal((16, 128))
    A = A * (np.arange(16)[None, :] == rng.integers(0, 16, 512)[:, None])
    got, ref = multiply(torch, rng, A + 0j, B + 0j, kernel)
    assert np.all(np.abs(got.real - ref.real) <= (2.0 ** -24 + 2.0 ** -28) * np.abs(ref.real))
    assert not got.imag.any()


@pytest.mark.parametrize("kernel", [-1, 0] + list(range(100, 106)))
def test_plan_layout_at_an_8_byte_address(kernel):
    """Operands in a plan's layout whose addresses are not a multiple of 16 bytes: the same bits as at one that is."""
    torch = require_gpu()
    from paper_2212_04749_amd import api
    rng = np.random.default_rng(11)
    nm, nn, nk, batch = 9, 7, 4, 3
    pos = plan_layout(rng, nm, nn, nk)
    a, b = torch.randn(batch * (2 << (nm + nk)), device="cuda"), torch.randn(batch * (2 << (nn + nk)), device="cuda")
    out = []
    for shift in (0, 2):
        A, B = torch.zeros(a.numel() + 2, device="cuda"), torch.zeros(b.numel() + 2, device="cuda")
        C = torch.full((batch * (2 << (nm + nn)) + 2,), float("nan"), device="cuda")
        A[shift:shift + a.numel()], B[shift:shift + b.numel()] = a, b
        x, y = A[shift:shift + a.numel()], B[shift:shift + b.numel()]
        c = C[shift:shift + (batch * (2 << (nm + nn)))]
        assert x.data_ptr() % 16 == 4 * shift
        keep = api.contract_pair(x, y, c, pos, kernel=kernel)
        torch.cuda.synchronize()
        del keep
        out.append(c.cpu().numpy())
    assert np.isfinite(out[0]).all()
    assert np.array_equal(out[0], out[1])


@pytest.mark.parametrize("nm,nn,nk,batch", [(6, 5, 6, 3), (6, 5, 7, 3), (6, 6, 9, 2), (7, 6, 8, 1), (6, 5, 7, 600)])
@pytest.mark.parametrize("layout", ["plan", "shuffled"])
def test_few_tiles_with_several_k_steps_in_flight(nm, nn, nk, batch, layout):
    """Below and from the least sum on, and with more tiles than that is for: the bits of the next larger tile (none
    where m or n are too small for one), and the accuracy of FP32 sums."""
    torch = require_gpu()
    from test_gpu_contract import make_case, reference
    rng = np.random.default_rng(17 * nk + batch)
    pos, A, B = make_case(rng, nm, nn, nk, batch)
    if layout == "plan":
        pos = plan_layout(rng, nm, nn, nk)
    got = run(torch, pos, A, B, nm, nn, nk, 102)
    if nm > 6:
        assert np.array_equal(got, run(torch, pos, A, B, nm, nn, nk, 100))
    assert rel_err(got, reference(pos, A, B, nm, nn, nk)) < 1.05 * ROUNDING * np.sqrt(2.0 ** nk + 0.5)
