"""GPU parity at the edges of the kernels' dispatch rules and tiles, against the float64
oracle, with the bounds of test_gpu_parity (fp32 logits: loss 1e-5 relative, gradient 1e-5
absolute; 16-bit logits: loss 2e-3 relative, gradient 2e-3 relative + 1e-5, plus the bf16
rounding where the gradient is stored in bf16)."""
import sys

import numpy as np
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


# rows taken in pieces (more than 320 interior chunks: V of about 1284 float32 and 2567 16-bit
# elements; pieces of 1024 and 2048): the edges of the rule and of the pieces, a block with fewer
# rows than waves, rows whose range moves far from the one before (a new shift), and a NaN row
@pytest.mark.parametrize("V,dtype", [(1283, "f32"), (1284, "f32"), (1287, "f32"), (2048, "f32"), (2051, "f32"),
                                     (3077, "f32"), (2567, "bf16"), (2568, "bf16"), (4096, "f16"), (6155, "bf16")])
def test_populate_rows_in_pieces(torch, pkg, V, dtype):  # noqa: F811
    check(torch, pkg, 2, 3, 5, V, seed=V, dtype=dtype, blank=V - 1)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_pieces_of_rows_far_apart(torch, pkg, dtype):  # noqa: F811
    V = 3000
    logits, tl, ul, labels = W.small_case(2, 4, 6, V, 5, sigma=1.5, full=True)
    # up to 60 nats between neighbouring rows, and the largest element of some rows in the last piece
    logits += np.random.default_rng(6).uniform(-30.0, 30.0, size=logits.shape[:3] + (1,)).astype(np.float32)
    logits[:, 1:3, ::2, V - 3] += 40.0
    logits[0, 2, 3, 17] = np.nan
    loss, grad, seen = run_case(torch, pkg, logits, tl, ul, labels, dtype=dtype)
    assert np.isnan(loss[0]) and not np.isnan(loss[1])
    loss_ref, grad_ref = R.rnnt_loss_grad(seen[1:], labels[1:], tl[1:], ul[1:], 0, "rnnt")
    tol_check(loss[1:], grad[1:], loss_ref, grad_ref, dtype)


# sweeps in scaled probabilities: columns of 64 units (NW waves and their exchange, up to six; 385
# units go to the log2 sweep), chunks of 8 diagonals (frames and units around a chunk's end), every
# lattice, utterances that end inside an earlier column
@pytest.mark.parametrize("variant", ["rnnt", "wrnnt", "wrnnt_allow_ignore"])
@pytest.mark.parametrize("T,U", [(1, 0), (1, 7), (2, 1), (9, 0), (8, 1), (3, 6), (5, 4), (6, 4), (17, 63), (16, 64),
                                 (30, 65), (25, 127), (9, 128), (40, 192), (3, 256), (12, 319), (70, 320), (11, 383),
                                 (6, 384), (300, 9), (90, 70)])
def test_sweep_columns_and_chunks(torch, pkg, variant, T, U):  # noqa: F811
    for full in (True, False):
        check(torch, pkg, 3, T, U, 6, seed=T * 1000 + U, variant=variant, full=full, sigma=2.0)


# logits so sharp that chunks are done again with an exponent per value (weights below 2^-200, steep
# neighbours) across columns, and -inf entries (arcs of probability 0, nodes no path reaches)
@pytest.mark.parametrize("variant", ["rnnt", "wrnnt", "wrnnt_allow_ignore"])
@pytest.mark.parametrize("T,U,sigma", [(30, 10, 30.0), (30, 10, 120.0), (41, 90, 60.0), (90, 140, 25.0)])
def test_sweep_of_sharp_logits(torch, pkg, variant, T, U, sigma):  # noqa: F811
    logits, tl, ul, labels = W.small_case(3, T, U, 7, int(T + U + sigma), sigma=1.0)
    logits *= np.random.default_rng(T).choice([0.2, 1.0], size=logits.shape[:3] + (1,)) * sigma
    logits = np.clip(logits, -160.0, 160.0).astype(np.float32)
    loss, grad, seen = run_case(torch, pkg, logits, tl, ul, labels, variant=variant)
    loss_ref, grad_ref = R.rnnt_loss_grad(seen, labels, tl, ul, 0, variant)
    # a softmax of logits of up to 160 nats: its float32 normaliser is 2^-17 of a log2 unit off
    assert np.all(np.abs(loss - loss_ref) <= 1e-5 * np.abs(loss_ref) + 1e-5)
    assert np.abs(grad - grad_ref).max() <= 2e-5


# an alignment's symbols raised by up to 20 nats (the falls and rises the one-sweep form is sized for, on
# both sides of its limits), utterances of fewer units than the padded shape: lanes without a node
@pytest.mark.parametrize("variant", ["rnnt", "wrnnt", "wrnnt_allow_ignore"])
@pytest.mark.parametrize("T,U,peak", [(60, 10, 8.0), (90, 20, 20.0), (70, 63, 12.0), (60, 110, 12.0), (40, 140, 20.0)])
def test_sweep_of_peaked_logits(torch, pkg, variant, T, U, peak):  # noqa: F811
    logits, tl, ul, labels = W.small_case(3, T, U, 29, T + U, sigma=2.0)
    rng = np.random.default_rng(U)
    for b in range(3):
        frame = np.append(np.sort(rng.integers(0, tl[b], size=ul[b])), 1 << 30)
        sym = np.where(np.arange(T)[:, None] >= frame, np.append(labels[b, :ul[b]], 0), 0)
        np.put_along_axis(logits[b, :, :ul[b] + 1], sym[..., None],
                          np.take_along_axis(logits[b, :, :ul[b] + 1], sym[..., None], 2) + np.float32(peak), 2)
    loss, grad, seen = run_case(torch, pkg, logits, tl, ul, labels, variant=variant)
    loss_ref, grad_ref = R.rnnt_loss_grad(seen, labels, tl, ul, 0, variant)
    # a loss is a sum of T + U weights, each off by its float32 normaliser's last bit (6e-8 of up to 32 nats)
    assert np.all(np.abs(loss - loss_ref) <= 1e-5 * np.abs(loss_ref) + 2e-6 * (T + U))
    assert np.abs(grad - grad_ref).max() <= 2e-5


def test_sweep_of_masked_symbols(torch, pkg):  # noqa: F811
    logits, tl, ul, labels = W.small_case(2, 20, 70, 6, 3, sigma=1.0, full=True)
    logits[0, 3:9, 2:60, 0] = -np.inf              # no blank there: the path must climb
    loss, grad, seen = run_case(torch, pkg, logits, tl, ul, labels)
    with np.errstate(divide="ignore", invalid="ignore"):
        loss_ref, grad_ref = R.rnnt_loss_grad(seen, labels, tl, ul, 0, "rnnt")
    tol_check(loss, grad, loss_ref, grad_ref, "f32")


def test_sweep_scales_past_the_stored_exponent(torch, pkg):  # noqa: F811
    logits, tl, ul, labels = W.small_case(3, 12, 70, 5, 9, sigma=1.0, full=True)
    logits[1] *= 3e6  # path probabilities below 2^-8300000: the log2 sweep of one wave
    loss, grad, seen = run_case(torch, pkg, logits, tl, ul, labels)
    loss_ref, grad_ref = R.rnnt_loss_grad(seen, labels, tl, ul, 0, "rnnt")
    assert np.all(np.abs(loss - loss_ref) <= 1e-5 * np.abs(loss_ref))
    for b in (0, 2):
        assert np.abs(grad[b] - grad_ref[b]).max() <= 1e-5
    assert np.all(np.isfinite(grad[1]))


# rows of more than 2^16 elements, flat (their sum relative to the largest element is past the inherited shift's
# limit) and in turn with rows of one dominant element; the bound of test_populate_kernel
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_flat_rows_of_many_elements(torch, pkg, dtype):  # noqa: F811
    B, T, U, V = 1, 2, 12, 140001
    rng = np.random.default_rng(1)
    logits = rng.normal(0.0, 0.05, size=(B, T, U + 1, V)).astype(np.float32)
    logits[0, 0, 1::3, 77] = 25.0
    logits[0, 1, 5] -= 60.0
    dev = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    lg = dev(logits).to(W.torch_dtype(dtype))
    lse = pkg.log_softmax_gather(lg, dev(np.ones((B, U), np.int32)), dev(np.array([T], np.int32)),
                                 dev(np.array([U], np.int32)), 0)[0].cpu().numpy()
    z = lg.double().cpu().numpy()
    m = z.max(axis=-1, keepdims=True)
    ref = (m + np.log(np.exp(z - m).sum(axis=-1, keepdims=True)))[..., 0]
    np.testing.assert_allclose(lse, ref, rtol=0, atol=1e-6)
