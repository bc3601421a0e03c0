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
