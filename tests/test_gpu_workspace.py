"""Calls that are given no workspace: under a stream capture, and where torch has no memory left."""
import ctypes
import sys

import numpy as np
import pytest

from paper_2303_10384_amd import workloads as W
from test_gpu_parity import pkg, to_dev, torch  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def announce(request):
    sys.__stderr__.write("\n[gpu-test] %s\n" % request.node.nodeid)
    sys.__stderr__.flush()
    yield


def inputs(torch):  # noqa: F811
    logits, tl, ul, labels = W.small_case(6, 20, 9, 48, seed=8, sigma=2.0)
    return [to_dev(torch, a) for a in (logits, labels, tl, ul)]


class Capture:
    """A capture that torch did not begin: HIP's own calls on a torch stream."""

    def __init__(self, torch):  # noqa: F811
        self.hip = ctypes.CDLL("libamdhip64.so")
        self.stream = torch.cuda.Stream()
        self.raw = ctypes.c_void_p(self.stream.cuda_stream)

    def check(self, code):
        assert code == 0, code

    def record(self, torch, fn):  # noqa: F811
        graph, self.exec = ctypes.c_void_p(), ctypes.c_void_p()
        with torch.cuda.stream(self.stream):
            self.check(self.hip.hipStreamBeginCapture(self.raw, 2))  # relaxed
            fn()
            self.check(self.hip.hipStreamEndCapture(self.raw, ctypes.byref(graph)))
        self.check(self.hip.hipGraphInstantiate(ctypes.byref(self.exec), graph, None, None, ctypes.c_size_t(0)))

    def replay(self):
        self.check(self.hip.hipGraphLaunch(self.exec, self.raw))


def test_capture_that_torch_did_not_begin(torch, pkg):  # noqa: F811
    lg, labels, tl, ul = inputs(torch)
    grad, loss = torch.empty_like(lg), torch.empty(6, dtype=torch.float32, device="cuda")

    def call():
        pkg.rnnt_loss(lg, labels, tl, ul, variant="wrnnt", grad_out=grad, loss_out=loss)

    call()
    torch.cuda.synchronize()
    loss_ref, grad_ref = loss.clone(), grad.clone()
    c = Capture(torch)
    c.record(torch, call)
    n = pkg.loss_workspace_bytes(6, 20, 9, 48)
    # blocks of the workspace's size, allocated after the capture on its stream: a replay must not write them
    with torch.cuda.stream(c.stream):
        others = [torch.full((n,), 7, dtype=torch.uint8, device="cuda") for _ in range(4)]
    torch.cuda.synchronize()
    for _ in range(3):
        grad.fill_(float("nan"))
        loss.fill_(float("nan"))
        torch.cuda.synchronize()
        c.replay()
        torch.cuda.synchronize()
        assert torch.equal(loss, loss_ref) and torch.equal(grad, grad_ref)
        assert all(bool((o == 7).all()) for o in others)
        call()  # eager work between the replays
        torch.cuda.synchronize()


def test_torch_graph_without_a_workspace(torch, pkg):  # noqa: F811
    lg, labels, tl, ul = inputs(torch)
    loss_ref, grad_ref = pkg.rnnt_loss(lg, labels, tl, ul)
    grad, loss = torch.empty_like(lg), torch.empty_like(loss_ref)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        pkg.rnnt_loss(lg, labels, tl, ul, grad_out=grad, loss_out=loss)
    for _ in range(3):
        grad.fill_(float("nan"))
        loss.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(loss, loss_ref) and torch.equal(grad, grad_ref)
        pkg.rnnt_loss(lg, labels, tl, ul, grad_out=grad, loss_out=loss)
        torch.cuda.synchronize()


def test_no_memory_left_in_torch(torch, pkg, monkeypatch):  # noqa: F811
    """torch's allocator refusing the workspace is not an error of the call: the library's own checks come
    first, and it takes a workspace of its own."""
    lg, labels, tl, ul = inputs(torch)
    loss_ref, grad_ref = pkg.rnnt_loss(lg, labels, tl, ul)
    grad, loss = torch.empty_like(lg), torch.empty_like(loss_ref)
    empty = torch.empty

    def no_bytes(*args, **kw):
        if kw.get("dtype") is torch.uint8:
            raise torch.OutOfMemoryError("no memory left")
        return empty(*args, **kw)

    monkeypatch.setattr(torch, "empty", no_bytes)
    pkg.rnnt_loss(lg, labels, tl, ul, grad_out=grad, loss_out=loss)
    assert torch.equal(loss, loss_ref) and torch.equal(grad, grad_ref)
    xr = lg.clone().requires_grad_(True)
    pkg.RNNTLoss(reduction="sum")(xr, labels, tl, ul).backward()
    assert np.array_equal(xr.grad.cpu().numpy(), grad_ref.cpu().numpy())
    with pytest.raises(pkg.RNNTError, match="blank"):
        pkg.rnnt_loss(lg, labels, tl, ul, blank=99, grad_out=grad, loss_out=loss)
