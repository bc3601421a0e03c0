"""GPU parity at the edges of the kernels' dispatch rules and tiles, against the float64
oracle, with the bounds of test_gpu_parity (fp32 logits: loss 1e-5 relative, gradient 1e-5
absolute; 16-bit logits: loss 2e-3 relative, gradient 2e-3 relative + 1e-5, plus the bf16
rounding where the gradient is stored in bf16)."""
import sys

import pytest

from oracle import rnnt_ref as R
from paper_2303_10384_amd import workloads as W
from test_gpu_parity import pkg, run_case, tol_check, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def announce(request):
    sys.__stderr__.write("\n[gpu-test] %s\n" % request.node.nodeid)
    sys.__stderr__.flush()
    yield


def check(torch, pkg, B, T, U, V, seed, variant="rnnt", dtype="f32", grad_dtype=None, blank=0, sigma=1.5, full=False):
    logits, tl, ul, labels = W.small_case(B, T, U, V, seed, sigma=sigma, blank=blank, full=full)
    loss, grad, seen = run_case(torch, pkg, logits, tl, ul, labels, blank=blank, variant=variant, dtype=dtype,
                                grad_dtype=grad_dtype)
    loss_ref, grad_ref = R.rnnt_loss_grad(seen, labels, tl, ul, blank, variant)
    tol_check(loss, grad, loss_ref, grad_ref, dtype, tl, ul, grad_dtype=grad_dtype)


# a float32 gradient of 16-bit logits: chunks of four elements (rows shorter than a chunk, just
# below and at the 64-chunk rows of the wide form, a tensor ending inside a chunk)
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("V", [2, 3, 4, 5, 9, 254, 255, 257, 511, 1023])
def test_float32_gradient_of_half_logits(torch, pkg, dtype, V):  # noqa: F811
    check(torch, pkg, 3, 5, 6, V, seed=100 + V, dtype=dtype, grad_dtype="f32", blank=V - 1)


# blocks of the populate kernel: float32 rows of up to 128 KB a block (V = 128: 256 rows; 513: 63;
# 1023: 32), units at and past a block's end, and the row groups of equal coverage (V / 4 or V / 8
# interior chunks of 8, 16, 32, 64: two chunks for half the lanes)
@pytest.mark.parametrize("V,U,dtype", [(33, 255, "f32"), (33, 256, "f32"), (65, 300, "f32"), (128, 70, "f32"),
                                       (257, 126, "f32"), (257, 128, "f32"), (513, 62, "f32"), (513, 63, "f32"),
                                       (1023, 33, "f32"), (64, 40, "bf16"), (129, 40, "f16"), (257, 20, "bf16"),
                                       (513, 20, "f16")])
def test_populate_blocks_and_groups(torch, pkg, V, U, dtype):  # noqa: F811
    check(torch, pkg, 2, 5, U, V, seed=V + U, dtype=dtype, full=U % 2 == 0)


# few frames: blocks cut to a few rounds of their row groups (units just past a cut)
@pytest.mark.parametrize("V,U,dtype", [(1025, 16, "f32"), (1025, 33, "bf16"), (257, 65, "f16"), (513, 150, "bf16")])
def test_populate_blocks_of_few_frames(torch, pkg, V, U, dtype):  # noqa: F811
    check(torch, pkg, 1, 4, U, V, seed=V + U, dtype=dtype, full=True)
