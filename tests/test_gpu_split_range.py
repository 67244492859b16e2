"""Split-bfloat16 tiles whose sums leave the range of the scaled operands (an operand above 2^104, a sum above 2^80):
the tile is computed again with operands scaled down, and only what that cannot give is summed one by one."""

import numpy as np
import pytest

from gpu_util import require_gpu, say
from test_gpu_split_accuracy import multiply
from test_gpu_step_kernels import plan_layout, tolerance

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel", range(100, 106))
@pytest.mark.parametrize("rows,cols", [(60, 60), (110, 0), (0, 110), (20, 100), (-60, 60)])
def test_rows_and_columns_of_very_different_size(rows, cols, kernel):
    """Row m of A is scaled by up to 2^+-rows, column n of B by up to 2^+-cols (-rows: one row of normal size among
    tiny ones): every output is as near to 64 bits as its own products allow."""
    torch = require_gpu()
    rng = np.random.default_rng(kernel + rows + cols)
    nk = 5
    A = rng.standard_normal((512, 1 << nk)) + 1j * rng.standard_normal((512, 1 << nk))
    B = rng.standard_normal((1 << nk, 128)) + 1j * rng.standard_normal((1 << nk, 128))
    sa = 2.0 ** rng.integers(-abs(rows), abs(rows) + 1, 512)
    sb = 2.0 ** rng.integers(-cols, cols + 1, 128)
    if rows < 0:
        sa[:] = 2.0 ** rows
        sa[77] = 1.0
    got, ref = multiply(torch, rng, A * sa[:, None], B * sb[None, :], kernel)
    # results below the smallest normal FP32 number have its absolute error
    unit = np.maximum(sa[:, None] * sb[None, :], 2.0 ** -120)
    e = np.abs(got - ref) / unit / np.sqrt(2.0 ** (nk + 2))
    say(f"split range {rows} {cols} kernel {kernel}: {np.sqrt(np.mean(e ** 2)):.2e} {e.max():.2e}")
    assert np.all(np.isfinite(got))
    assert np.sqrt(np.mean(e ** 2)) < tolerance(nk) and e.max() < 10 * tolerance(nk)


def test_large_operands_next_to_tiny_ones():
    """A's first column is 2^120 and B's first row 2^-130 (a denormal number): their products are of the size of the
    others, so nothing of them may get lost by the second scaling."""
    torch = require_gpu()
    rng = np.random.default_rng(3)
    A = rng.standard_normal((256, 32)) + 1j * rng.standard_normal((256, 32))
    B = rng.standard_normal((32, 64)) + 1j * rng.standard_normal((32, 64))
    A[:, 0] = 2.0 ** 120
    B[0, :] = 2.0 ** -130 * rng.integers(1, 1 << 18, 64)
    got, ref = multiply(torch, rng, A, B, 101)
    e = np.abs(got - ref) / np.sqrt(np.mean(np.abs(ref) ** 2))
    assert e.max() < 10 * tolerance(5)


def test_large_operands_run_on_the_matrix_units():
    """Operands of 1e13, every sum out of range: at most four times as long as in range (twice, and no more than one
    in thousands left to the vector units)."""
    torch = require_gpu()
    from paper_2212_04749_amd import api
    rng = np.random.default_rng(5)
    pos = plan_layout(rng, 12, 6, 9)
    A = torch.randn((64, 2 << 21), device="cuda")
    B = torch.randn((64, 2 << 15), device="cuda")
    C = torch.empty((64, 2 << 18), device="cuda")

    def ms(a, b):
        times = []
        for _ in range(5):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            keep = api.contract_pair(a, b, C, pos)
            e1.record()
            e1.synchronize()
            times.append(e0.elapsed_time(e1))
            del keep
        return min(times)

    plain = ms(A, B)
    large = ms(A * 1e13, B * 1e13)
    say(f"split range: {plain:.3f} ms in range, {large:.3f} ms out of it")
    assert large < 4 * plain
