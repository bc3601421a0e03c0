"""The loss's sweep in scaled probabilities on networks far sharper than trained ones: weights of
2^-20 to 2^-199 on the best paths, where a score falls and is refilled within a few diagonals.
Against the float64 oracle with the bounds of test_gpu_parity: gradient 1e-5 absolute; loss 1e-5
relative, plus 6e-8 for each of the T + U weights of a path, whose float32 normalisers are that far
off (some losses here are next to 0, and the wild-card arcs even make them negative)."""
import sys

import numpy as np
import pytest

from oracle import rnnt_ref as R
from test_gpu_parity import pkg, run_case, tol_check, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def announce(request):
    sys.__stderr__.write("\n[gpu-test] %s\n" % request.node.nodeid)
    sys.__stderr__.flush()
    yield


def logits_of(x, y):
    """Logits of three symbols (blank 0, label 1, the rest) with p(blank) = 2^-x, p(label) = 2^-y."""
    x, y = np.asarray(x, float), np.asarray(y, float)
    rest = 1.0 - 2.0 ** -x - 2.0 ** -y
    return np.stack([-x * np.log(2.0), -y * np.log(2.0),
                     np.where(rest > 0, np.log(np.where(rest > 0, rest, 1.0)), -200.0)], axis=-1).astype(np.float32)


def check(torch, pkg, logits, tl, ul, variant="rnnt"):  # noqa: F811
    labels = np.ones((logits.shape[0], logits.shape[2] - 1), np.int32)
    tl, ul = np.asarray(tl, np.int32), np.asarray(ul, np.int32)
    loss, grad, seen = run_case(torch, pkg, logits, tl, ul, labels, variant=variant)
    loss_ref, grad_ref = R.rnnt_loss_grad(seen, labels, tl, ul, 0, variant)
    assert np.all(np.abs(loss - loss_ref) <= 1e-5 * np.abs(loss_ref) + 6e-8 * (tl + ul + 1)), (loss, loss_ref)
    assert np.abs(grad - grad_ref).max() <= 1e-5


# (x, y) of 24 frames of 5 nodes: p(blank) = 2^-x, p(label) = 2^-y.  The label posterior of node
# (12, 1) is 0.40, the product of alpha 2^-482, weight 2^-23 and beta 2^-593 of their lanes' scales
REFILLED = """
    1,100 1,199 1,1 1,199 1,1 | 1,199 1,199 1,1 1,1 1,1 | 100,1 1,199 1,199 1,1 1,1 | 50,1 199,141 199,199 1,1 1,1 |
    50,1 1,199 1,1 1,1 199,1 | 41,1 199,199 1,1 199,199 1,1 | 41,199 1,1 199,140 1,1 1,1 |
    41,199 199,199 199,1 199,1 91,1 | 41,199 1,199 1,1 199,1 100,1 | 41,199 1,199 1,1 1,1 41,1 |
    1,199 199,199 1,1 199,1 50,1 | 1,199 1,1 1,199 1,1 1,1 | 1,199 1,1 1,1 1,199 20,1 | 1,1 1,199 1,1 1,199 21,1 |
    50,1 1,1 199,199 199,199 1,1 | 100,1 199,199 1,199 1,199 1,1 | 1,1 199,1 199,199 1,199 21,1 |
    100,199 1,1 1,1 1,199 41,1 | 100,199 1,1 199,1 199,199 21,1 | 100,1 199,50 100,199 1,1 1,1 |
    199,1 100,199 199,1 199,1 100,1 | 1,1 1,199 1,1 1,1 50,1 | 1,1 1,199 1,1 1,1 50,1 | 1,1 1,199 1,199 1,1 1,1"""


def test_score_refilled_inside_a_chunk(torch, pkg):  # noqa: F811
    cells = np.array([[tuple(map(int, c.split(","))) for c in row.split()] for row in REFILLED.split("|")])
    check(torch, pkg, logits_of(cells[..., 0], cells[..., 1])[None], [24], [4])


# lattices drawn from a few steep weights, so that most nodes lie hundreds of binary orders off the
# best path and the best path itself takes unlikely arcs
@pytest.mark.parametrize("variant", ["rnnt", "wrnnt", "wrnnt_allow_ignore"])
@pytest.mark.parametrize("seed", range(8))
def test_steep_random_lattices(torch, pkg, variant, seed):  # noqa: F811
    rng = np.random.default_rng(700 + seed)
    T, U, B = int(rng.integers(9, 40)), int(rng.integers(1, 9)), 12
    steep = [1, 1, 1, 20, 50, 100, 199][: int(rng.integers(4, 8))]
    x = rng.choice(steep, size=(B, T, U + 1))
    y = rng.choice(steep, size=(B, T, U + 1))
    tl = rng.integers(max(1, T // 2), T, size=B, endpoint=True)
    ul = rng.integers(0, U, size=B, endpoint=True)
    check(torch, pkg, logits_of(x, y), tl, ul, variant)


# the same over several columns of 64 units (and their exchange), with weights down to the log2 form
# (below 2^-1000) and arcs of probability 0; utterances that end inside an earlier column
@pytest.mark.parametrize("variant", ["rnnt", "wrnnt", "wrnnt_allow_ignore"])
@pytest.mark.parametrize("T,U", [(30, 40), (40, 63), (30, 70), (90, 64), (41, 127), (14, 150), (50, 190), (9, 255),
                                 (12, 300), (70, 383)])
def test_steep_lattices_over_columns(torch, pkg, variant, T, U):  # noqa: F811
    rng = np.random.default_rng(T * 1000 + U)
    B = 5
    x, y = np.empty((2, B, T, U + 1))
    for b, steep in enumerate([[1, 1, 2, 3, 30], [1, 1, 20, 50, 100, 199], [1, 1, 1, 400, 900], [1, 1, 990, 1010, 2500],
                               [1, 1, 1, 1, 60, np.inf]]):
        x[b] = rng.choice(steep, size=(T, U + 1))
        y[b] = rng.choice(steep, size=(T, U + 1))
    x[4, :, -1], y[4, 0] = 1.0, 1.0  # a path is left
    tl, ul = np.full(B, T), np.full(B, U)
    tl[1:4] = rng.integers(max(1, T // 2), T, size=3, endpoint=True)
    ul[1:4] = rng.integers(U // 2, U, size=3, endpoint=True)
    with np.errstate(divide="ignore", invalid="ignore"):
        check(torch, pkg, logits_of(x, y), tl, ul, variant)


# an alignment's symbols raised by up to 60 nats: past what a chunk's scales hold
@pytest.mark.parametrize("variant", ["rnnt", "wrnnt", "wrnnt_allow_ignore"])
@pytest.mark.parametrize("T,U,peak", [(90, 20, 40.0), (70, 63, 60.0), (100, 80, 30.0), (60, 110, 40.0), (90, 150, 25.0),
                                      (60, 260, 45.0)])
def test_sharp_alignments(torch, pkg, variant, T, U, peak):  # noqa: F811
    rng = np.random.default_rng(U)
    logits = rng.normal(0.0, 2.0, size=(3, T, U + 1, 7)).astype(np.float32)
    tl = np.array([T, T - 7, max(1, T // 2)], np.int32)
    ul = np.array([U, U // 2, U - 1], np.int32)
    labels = rng.integers(1, 7, size=(3, U)).astype(np.int32)
    for b in range(3):
        frame = np.append(np.sort(rng.integers(0, tl[b], size=ul[b])), 1 << 30)
        sym = np.where(np.arange(T)[:, None] >= frame, np.append(labels[b, :ul[b]], 0), 0)
        np.put_along_axis(logits[b, :, :ul[b] + 1], sym[..., None],
                          np.take_along_axis(logits[b, :, :ul[b] + 1], sym[..., None], 2) + np.float32(peak), 2)
    loss, grad, seen = run_case(torch, pkg, logits, tl, ul, labels, variant=variant)
    loss_ref, grad_ref = R.rnnt_loss_grad(seen, labels, tl, ul, 0, variant)
    # a loss is a sum of T + U weights, each off by its float32 normaliser's last bit (2e-6 of up to 64 nats)
    assert np.all(np.abs(loss - loss_ref) <= 1e-5 * np.abs(loss_ref) + 4e-6 * (T + U))
    assert np.abs(grad - grad_ref).max() <= 4e-5


# a NaN logit anywhere in an utterance: its loss and gradient are NaN, the others' are not
@pytest.mark.parametrize("variant", ["rnnt", "wrnnt", "wrnnt_allow_ignore"])
@pytest.mark.parametrize("T,U", [(30, 20), (60, 100), (20, 300)])
def test_nan_stays_in_its_utterance(torch, pkg, variant, T, U):  # noqa: F811
    rng = np.random.default_rng(U)
    logits = rng.normal(0.0, 2.0, size=(4, T, U + 1, 6)).astype(np.float32)
    for b, (t, u) in enumerate([(0, 0), (T // 2, U // 2), (T - 1, U)]):
        logits[b, t, u, 3] = np.nan
    labels = rng.integers(1, 6, size=(4, U)).astype(np.int32)
    tl, ul = np.full(4, T, np.int32), np.full(4, U, np.int32)
    loss, grad, seen = run_case(torch, pkg, logits, tl, ul, labels, variant=variant)
    assert np.all(np.isnan(loss[:3])) and np.all(np.isnan(grad[:3]))
    loss_ref, grad_ref = R.rnnt_loss_grad(seen[3:], labels[3:], tl[3:], ul[3:], 0, variant)
    tol_check(loss[3:], grad[3:], loss_ref, grad_ref, "f32", tl[3:], ul[3:])


# path probabilities below 2^-4194304: scores in log2 units, one wave a sweep, in every lattice and over columns
@pytest.mark.parametrize("variant", ["rnnt", "wrnnt", "wrnnt_allow_ignore"])
@pytest.mark.parametrize("T,U", [(12, 20), (30, 63), (12, 70), (40, 150), (20, 383)])
def test_scores_in_log2_units(torch, pkg, variant, T, U):  # noqa: F811
    rng = np.random.default_rng(T + U)
    logits = rng.normal(0.0, 1.0, size=(3, T, U + 1, 5)).astype(np.float32)
    logits[1] *= 3e6
    labels = rng.integers(1, 5, size=(3, U)).astype(np.int32)
    tl, ul = np.array([T, T, T - 3], np.int32), np.array([U, U, U // 2], np.int32)
    loss, grad, seen = run_case(torch, pkg, logits, tl, ul, labels, variant=variant)
    loss_ref, grad_ref = R.rnnt_loss_grad(seen, labels, tl, ul, 0, variant)
    assert np.all(np.abs(loss - loss_ref) <= 1e-5 * np.abs(loss_ref))
    for b in (0, 2):
        assert np.abs(grad[b] - grad_ref[b]).max() <= 1e-5
    assert np.all(np.isfinite(grad[1]))


# path probabilities below 2^-4194304: scores in log2 units, one wave a sweep, in every lattice and over columns
@pytest.mark.parametrize("variant", ["rnnt", "wrnnt", "wrnnt_allow_ignore"])
@pytest.mark.parametrize("T,U", [(12, 20), (30, 63), (12, 70), (40, 150), (20, 383)])
def test_scores_in_log2_units(torch, pkg, variant, T, U):  # noqa: F811
    rng = np.random.default_rng(T + U)
    logits = rng.normal(0.0, 1.0, size=(3, T, U + 1, 5)).astype(np.float32)
    logits[1] *= 3e6
    labels = rng.integers(1, 5, size=(3, U)).astype(np.int32)
    tl, ul = np.array([T, T, T - 3], np.int32), np.array([U, U, U // 2], np.int32)
    loss, grad, seen = run_case(torch, pkg, logits, tl, ul, labels, variant=variant)
    loss_ref, grad_ref = R.rnnt_loss_grad(seen, labels, tl, ul, 0, variant)
    assert np.all(np.abs(loss - loss_ref) <= 1e-5 * np.abs(loss_ref))
    for b in (0, 2):
        assert np.abs(grad[b] - grad_ref[b]).max() <= 1e-5
    assert np.all(np.isfinite(grad[1]))


# the closing blank masked with a finite number, down to float32's lowest: the loss is that number where
# every path takes the arc, and untouched where paths may leave it out (allow-ignore, T > 1)
@pytest.mark.parametrize("variant", ["rnnt", "wrnnt", "wrnnt_allow_ignore"])
@pytest.mark.parametrize("T,U", [(1, 0), (3, 2), (9, 3), (17, 0)])
def test_masked_closing_blank(torch, pkg, variant, T, U):  # noqa: F811
    masks = [-1e4, -1e6, -1e10, -1e30, float(np.finfo(np.float32).min)]
    logits = np.random.default_rng(T).normal(size=(len(masks), T, U + 1, 5)).astype(np.float32)
    logits[:, T - 1, U, 0] = masks
    labels = np.ones((len(masks), U), np.int32)
    tl, ul = np.full(len(masks), T, np.int32), np.full(len(masks), U, np.int32)
    loss, grad, seen = run_case(torch, pkg, logits, tl, ul, labels, variant=variant)
    loss_ref, grad_ref = R.rnnt_loss_grad(seen, labels, tl, ul, 0, variant)
    tol_check(loss, grad, loss_ref, grad_ref, "f32", tl, ul)
