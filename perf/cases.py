"""Timed workloads of the loss library: what a program has it do, through the package's
public entry points.

A case is a dict of plain values; listed() names the fixed ones and draw() makes more
from the ranges they stand for.  prepare() builds what the caller's program holds before
the call (logits of a joint network, labels, lengths, a planned lattice, buffers it
keeps), run() is one call, exact() the same results in float64 from plain torch.

Keys of a case
  path      the entry point: "loss" (rnnt_loss), "train" (RNNTLoss, forward and backward),
            "noalloc" (rnnt_loss_noalloc), "align" (viterbi_align), "arc" (arc_loss)
  B, T, U, V  padded shape: logits (B, T, U+1, V)
  dtype     logits: "f32", "bf16", "f16";  grad: dtype of the gradient, or "none" (loss only)
  variant   "rnnt", "wrnnt", "wrnnt_allow_ignore"
  lengths   "full", "variable" (0.5-1 of T, 0.3-1 of U), "text_drop" (all frames, 0.6-1 of U);
            drawn from len_seed, so a case has the same lengths for every input seed
  sigma     the logits are N(0, sigma^2), the stand-in for a joint network's outputs
  peak      added to the symbol of a random alignment in every row (a trained network); 0: none
  blank     index of the blank
  keep      the caller keeps workspace and outputs between calls (a training loop)
  reduction reduction of RNNTLoss
"""
import math

import numpy as np
import torch

import paper_2303_10384_amd as rnnt
from paper_2303_10384_amd import topologies

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
BYTES = {"f32": 4, "bf16": 2, "f16": 2, "none": 0}
MAX_ELEMS = 64 * 500 * 151 * 1025  # the largest listed case's logits
EXACT_ELEMS = 1_000_000_000        # above this the float64 result takes too long


def _case(name, path, B, T, U, V, dtype="f32", grad=None, variant="rnnt", lengths="variable", len_seed=0, sigma=3.0,
          peak=0.0, blank=0, keep=False, reduction="none"):
    return {"name": name, "path": path, "B": B, "T": T, "U": U, "V": V, "dtype": dtype,
            "grad": dtype if grad is None else grad, "variant": variant, "lengths": lengths, "len_seed": len_seed,
            "sigma": sigma, "peak": peak, "blank": blank, "keep": keep, "reduction": reduction}


def listed():
    return [
        # the smallest call (the smoke test's shape): two short utterances, nothing kept by the caller
        _case("tiny", "loss", 2, 20, 8, 16, lengths="full", sigma=1.0),
        # a training step on characters through the autograd module (forward and backward)
        _case("char_train", "train", 16, 150, 40, 29, sigma=2.0, len_seed=1, reduction="mean"),
        # characters of utterances of about 15 s: hundreds of units to a lattice, few symbols to a row
        _case("char_long", "loss", 16, 400, 300, 32, sigma=2.0, peak=3.0, len_seed=2),
        # the benchmark's training batch on word pieces, buffers kept from step to step
        _case("bpe", "loss", 32, 250, 80, 1025, len_seed=3, keep=True),
        # the same batch in a mixed-precision training step through the autograd module
        _case("bpe_amp_train", "train", 32, 250, 80, 1025, dtype="bf16", len_seed=4, reduction="mean"),
        # W-Transducer training on transcripts with words dropped at both ends
        _case("wrnnt", "loss", 32, 250, 80, 1025, variant="wrnnt", lengths="text_drop", len_seed=5, keep=True),
        # the largest batch: 64 long utterances in bfloat16
        _case("large", "loss", 64, 500, 150, 1025, dtype="bf16", len_seed=6, keep=True),
        # validation with a trained network: losses only, half precision
        _case("eval", "loss", 32, 300, 60, 513, dtype="f16", grad="none", sigma=2.0, peak=8.0, len_seed=7),
        # a vocabulary of several thousand units, half-precision logits and a float32 gradient
        _case("wide_vocab", "loss", 8, 200, 50, 5003, dtype="bf16", grad="f32", variant="wrnnt_allow_ignore",
              sigma=2.0, peak=4.0, len_seed=8),
        # forced alignment of a batch with a trained network
        _case("align", "align", 32, 250, 80, 1025, grad="none", peak=8.0, len_seed=9),
        # forced alignment of one utterance while a user waits
        _case("align_one", "align", 1, 180, 45, 257, dtype="f16", grad="none", lengths="full", sigma=2.0, peak=8.0),
        # the training lattices given as arc lists (any other topology takes this path too)
        _case("arc", "arc", 32, 250, 80, 1025, len_seed=10, keep=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any path, sizes spread over the listed cases' ranges."""
    path = rng.choice(["loss", "loss", "loss", "train", "train", "noalloc", "align", "align", "arc"])
    while True:
        B = _log_int(rng, 1, 64)
        T = _log_int(rng, 12, 600)
        U = min(_log_int(rng, 4, 320), 2 * T)
        V = _log_int(rng, 16, 6000)
        dtype = rng.choice(["f32", "f32", "bf16", "f16"])
        variant = rng.choice(["rnnt", "rnnt", "wrnnt", "wrnnt_allow_ignore"])
        grad = dtype
        if path == "align":
            grad = "none"
        elif path in ("loss", "noalloc", "arc"):
            grad = rng.choice([dtype, dtype, "f32", "none"])
        elems = B * T * (U + 1) * V
        if path == "train" and elems > 32 * 250 * 81 * 1025:
            continue
        if path == "arc" and B * T * (U + 1) > 32 * 250 * 81:
            continue
        if path == "noalloc" and rnnt.loss_workspace_bytes(B, T, U, V) > (64 << 20):
            continue
        if elems <= MAX_ELEMS // 4:
            break
    lengths = rng.choice(["variable", "variable", "full"]) if variant == "rnnt" else "text_drop"
    return _case("", path, B, T, U, V, dtype=dtype, grad=grad, variant=variant, lengths=lengths,
                 len_seed=rng.randrange(1 << 20), sigma=round(rng.uniform(1.0, 3.0), 2),
                 peak=rng.choice([0.0, 3.0, 8.0]), blank=rng.choice([0, 0, V - 1]),
                 keep=rng.random() < 0.5, reduction=rng.choice(["none", "sum", "mean"]) if path == "train" else "none")


# ---------------------------------------------------------------- inputs

def _lengths(case):
    """(frames, units) of every utterance, utterance 0 at the padded shape."""
    B, T, U = case["B"], case["T"], case["U"]
    rng = np.random.Generator(np.random.PCG64([77, case["len_seed"], B, T, U]))
    if case["lengths"] == "full":
        return np.full(B, T, np.int32), np.full(B, U, np.int32)
    if case["lengths"] == "variable":
        tl = rng.integers(math.ceil(0.5 * T), T, size=B, endpoint=True)
        ul = rng.integers(math.ceil(0.3 * U), U, size=B, endpoint=True)
    else:
        tl = np.full(B, T)
        ul = rng.integers(math.ceil(0.6 * U), U, size=B, endpoint=True)
    tl[0], ul[0] = T, U
    return tl.astype(np.int32), ul.astype(np.int32)


def _labels(case, rng):
    """Units other than the blank, (B, U)."""
    y = rng.integers(0, case["V"] - 1, size=(case["B"], case["U"]))
    return (y + (y >= case["blank"])).astype(np.int32)


def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _inputs(case, seed):
    """(logits, labels, frames, units) of one seed, the last three as numpy arrays."""
    B, T, U, V = case["B"], case["T"], case["U"], case["V"]
    dev, dtype = _device(), DTYPES[case["dtype"]]
    rng = np.random.Generator(np.random.PCG64([11, seed]))
    labels = _labels(case, rng)
    tl, ul = _lengths(case)
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(rng.integers(1 << 40)))
    logits = torch.empty((B, T, U + 1, V), dtype=dtype, device=dev)
    if dtype == torch.float32:
        logits.normal_(0.0, case["sigma"], generator=gen)
    else:
        for b in range(B):  # drawn in float32, then rounded
            logits[b] = torch.empty((T, U + 1, V), device=dev).normal_(0.0, case["sigma"], generator=gen)
    if case["peak"]:
        # an alignment per utterance: unit u+1 comes at frame f[u]; a row before it favours the
        # blank, a row from it on favours the unit
        f = np.sort(rng.integers(0, tl[:, None], size=(B, U)), axis=1)
        f = np.concatenate([f, np.full((B, 1), 1 << 30)], axis=1)
        sym = np.where(np.arange(T)[None, :, None] >= f[:, None, :],
                       np.concatenate([labels, np.full((B, 1), case["blank"])], axis=1)[:, None, :], case["blank"])
        index = torch.from_numpy(sym.astype(np.int64)).to(dev).unsqueeze(-1)
        logits.scatter_add_(3, index, torch.full(index.shape, case["peak"], dtype=dtype, device=dev))
    return logits, labels, tl, ul


def prepare(case, seed):
    logits, labels, tl, ul = _inputs(case, seed)
    dev = logits.device
    s = {"path": case["path"], "variant": case["variant"], "blank": case["blank"], "logits": logits,
         "labels": torch.from_numpy(labels).to(dev), "tl": torch.from_numpy(tl).to(dev),
         "ul": torch.from_numpy(ul).to(dev), "need_grad": case["grad"] != "none"}
    gdt = DTYPES[case["grad"]] if s["need_grad"] else None
    s["grad_dtype"] = gdt
    s["workspace"] = s["grad_out"] = s["loss_out"] = s["outputs"] = None
    B, T, U, V = case["B"], case["T"], case["U"], case["V"]
    if case["path"] == "train":
        logits.requires_grad_(True)
        s["module"] = rnnt.RNNTLoss(case["blank"], case["variant"], case["reduction"])
    if case["path"] == "arc":
        lattices = topologies.batch_grid_lattices(tl, ul, labels, case["blank"], case["variant"])
        s["plan"] = rnnt.arc_plan(lattices, T, U, V, case["blank"], device=dev)
    if case["keep"] or case["path"] == "noalloc":
        s["loss_out"] = torch.empty(B, dtype=torch.float32, device=dev)
        if s["need_grad"]:
            s["grad_out"] = torch.empty(logits.shape, dtype=gdt, device=dev)
    if case["keep"]:
        size = {"loss": lambda: rnnt.loss_workspace_bytes(B, T, U, V),
                "align": lambda: rnnt.viterbi_workspace_bytes(B, T, U, V),
                "arc": lambda: rnnt.arc_loss_workspace_bytes(s["plan"])}.get(case["path"])
        if size:
            s["workspace"] = torch.empty(size(), dtype=torch.uint8, device=dev)
        if case["path"] == "align":
            s["outputs"] = (torch.empty(B, dtype=torch.float32, device=dev),
                            torch.empty((B, U), dtype=torch.int32, device=dev),
                            torch.empty((B, 2), dtype=torch.int32, device=dev))
    return s


def run(s):
    if s["path"] == "train":
        loss = s["module"](s["logits"], s["labels"], s["tl"], s["ul"])
        upstream = None if loss.dim() == 0 else torch.ones_like(loss)
        (grad,) = torch.autograd.grad(loss, s["logits"], upstream)
        return loss.detach(), grad
    if s["path"] == "noalloc":
        out = rnnt.rnnt_loss_noalloc(s["logits"], s["labels"], s["tl"], s["ul"], s["loss_out"], s["grad_out"],
                                     blank=s["blank"], variant=s["variant"])
    elif s["path"] == "align":
        return rnnt.viterbi_align(s["logits"], s["labels"], s["tl"], s["ul"], blank=s["blank"], variant=s["variant"],
                                  workspace=s["workspace"], outputs=s["outputs"])
    elif s["path"] == "arc":
        out = rnnt.arc_loss(s["logits"], s["tl"], s["ul"], s["plan"], need_grad=s["need_grad"],
                            workspace=s["workspace"], grad_out=s["grad_out"], loss_out=s["loss_out"],
                            grad_dtype=s["grad_dtype"])
    else:
        out = rnnt.rnnt_loss(s["logits"], s["labels"], s["tl"], s["ul"], blank=s["blank"], variant=s["variant"],
                             need_grad=s["need_grad"], workspace=s["workspace"], grad_out=s["grad_out"],
                             loss_out=s["loss_out"], grad_dtype=s["grad_dtype"])
    return out if s["need_grad"] else out[:1]


# ---------------------------------------------------------------- what a pass cannot do without

def work(case):
    tl, ul = _lengths(case)
    rows = int(np.sum(tl.astype(np.int64) * (ul + 1)))  # the rows an utterance has; padding is not read
    elems = rows * case["V"]
    padded = case["B"] * case["T"] * (case["U"] + 1) * case["V"]
    small = 4 * case["B"] * (case["U"] + 2) + 4 * case["B"]  # labels, lengths, losses
    if case["path"] == "align":
        small += 4 * case["B"] * (case["U"] + 2)
    if case["path"] == "arc":
        small += 24 * 2 * rows  # about two arcs to a node, as the caller lists them
    # a row's normaliser: scale, exponential and sum; its gradient: the same exponential, one product
    flops = elems * (3 + (3 if case["grad"] != "none" else 0)) + 20 * rows
    return {"bytes": elems * BYTES[case["dtype"]] + padded * BYTES[case["grad"]] + small, "flops": flops}


def tolerance(case):
    """About four times the error measured against exact() over listed and drawn cases."""
    if case["path"] == "align":
        # scores are float64 sums of the chosen arcs, stored in float32; frames are whole numbers that
        # only a tie between float32-rounded normalisers could move
        return {"rel": 4e-7, "differ": 0.002}
    if case["grad"] == "bf16":
        return {"rel": 5e-3, "max": 1.6e-2}  # the stored gradient's own rounding: 1.3e-3, at most 3.9e-3
    if case["grad"] == "f16":
        return {"rel": 8e-4, "max": 2e-3}    # 2.1e-4, at most 4.9e-4
    return {"rel": 4e-6, "max": 1e-3}        # float32 sums: 8e-7, at most 1.8e-4 (a trained network's peaks)


# ---------------------------------------------------------------- the same in float64

def _log_probs(case, logits, labels):
    """Natural-log weights of the blank and label arcs, (B, T, U+1) float64."""
    B, T, U1, V = logits.shape
    lpb = torch.empty((B, T, U1), dtype=torch.float64, device=logits.device)
    lpl = torch.full_like(lpb, -math.inf)
    y = torch.from_numpy(labels.astype(np.int64)).to(logits.device)
    for b in range(B):
        z = logits[b].double()
        lse = torch.logsumexp(z, dim=-1)
        lpb[b] = z[..., case["blank"]] - lse
        idx = y[b].view(1, U1 - 1, 1).expand(T, U1 - 1, 1)
        lpl[b, :, :-1] = z[:, :-1].gather(2, idx).squeeze(2) - lse[:, :-1]
    return lpb, lpl


def _shear(x, fill):
    """(B, T, U1) -> (T+U, B, U1): diagonal d holds cell (d-u, u) in column u."""
    B, T, U1 = x.shape
    d = torch.arange(T + U1 - 1, device=x.device)[:, None]
    t = d - torch.arange(U1, device=x.device)[None]
    ok = (t >= 0) & (t < T)
    out = x[:, t.clamp(0, T - 1), torch.arange(U1, device=x.device)[None]]
    return torch.where(ok[None], out, torch.full_like(out, fill)).transpose(0, 1).contiguous()


def _unshear(x, T):
    """The inverse of _shear."""
    D, B, U1 = x.shape
    t = torch.arange(T, device=x.device)[:, None]
    u = torch.arange(U1, device=x.device)[None]
    return x[t + u, :, u].permute(2, 0, 1).contiguous()


def _lattice(case, lpb, lpl, tl, ul):
    """ln P of every utterance and the posteriors of the blank and label arcs."""
    B, T, U1 = lpb.shape
    dev, var = lpb.device, case["variant"]
    ninf = -math.inf
    Tb = torch.from_numpy(tl.astype(np.int64)).to(dev)
    Ub = torch.from_numpy(ul.astype(np.int64)).to(dev)
    t = torch.arange(T, device=dev)[None, :, None]
    u = torch.arange(U1, device=dev)[None, None]
    valid = (t < Tb[:, None, None]) & (u <= Ub[:, None, None])
    top = valid & (u == Ub[:, None, None])
    last = t == (Tb - 1)[:, None, None]
    close = lpb[torch.arange(B, device=dev), Tb - 1, Ub]
    pb = _shear(torch.where(valid & ~last, lpb, torch.full_like(lpb, ninf)), ninf)
    pl = _shear(torch.where(valid & ~top, lpl, torch.full_like(lpl, ninf)), ninf)
    D = pb.shape[0]
    skip0 = _shear((valid & (u == 0) & (t >= 1)).double(), 0.0) > 0  # (t, 0), t >= 1
    skip_top = _shear((top & ~last).double(), 0.0) > 0               # (t, U), t <= T-2
    alpha = torch.full((D, B, U1), ninf, dtype=torch.float64, device=dev)
    alpha[0, :, 0] = 0.0
    pad = torch.full((B, 1), ninf, dtype=torch.float64, device=dev)
    zero = torch.zeros((), dtype=torch.float64, device=dev)
    for d in range(1, D):
        a = torch.logaddexp(alpha[d - 1] + pb[d - 1], torch.cat([pad, (alpha[d - 1] + pl[d - 1])[:, :-1]], 1))
        if var != "rnnt":
            a = torch.where(skip0[d], torch.logaddexp(a, zero), a)
        alpha[d] = a
    alpha = _unshear(alpha, T)
    end = alpha[torch.arange(B, device=dev), Tb - 1, Ub]
    jump = torch.logsumexp(torch.where(top & ~last, alpha, torch.full_like(alpha, ninf)).flatten(1), dim=1)
    if var == "wrnnt":
        end = torch.logaddexp(end, jump)
        alpha[torch.arange(B, device=dev), Tb - 1, Ub] = end
    ln_p = end + close
    if var == "wrnnt_allow_ignore":
        ln_p = torch.logaddexp(ln_p, jump)
    # backward: the final node (T-1, U) starts at the closing blank
    is_end = _shear((top & last).double(), 0.0) > 0
    beta = torch.full((D + 1, B, U1), ninf, dtype=torch.float64, device=dev)
    jump_to = close if var == "wrnnt" else torch.zeros_like(close)
    for d in range(D - 1, -1, -1):
        b_next = beta[d + 1]
        x = torch.logaddexp(pb[d] + b_next, pl[d] + torch.cat([b_next[:, 1:], pad], 1))
        x = torch.where(is_end[d], close[:, None].expand_as(x), x)
        if var != "rnnt":
            x = torch.where(skip_top[d], torch.logaddexp(x, jump_to[:, None].expand_as(x)), x)
        beta[d] = x
    beta = _unshear(beta[:D], T)
    b_down = torch.cat([beta[:, 1:], torch.full_like(beta[:, :1], ninf)], 1)
    b_down = torch.where(top & last, torch.zeros_like(b_down), b_down)
    b_right = torch.cat([beta[:, :, 1:], torch.full_like(beta[:, :, :1], ninf)], 2)
    no_blank = ~valid | (last & ~top)
    occ_b = torch.where(no_blank, zero, torch.exp(alpha + lpb + b_down - ln_p[:, None, None]))
    occ_l = torch.where(~valid | top, zero, torch.exp(alpha + lpl + b_right - ln_p[:, None, None]))
    return ln_p, occ_b, occ_l


def _gradient(case, logits, labels, tl, ul, occ_b, occ_l):
    B, T, U1, V = logits.shape
    grad = torch.zeros(logits.shape, dtype=torch.float64, device=logits.device)
    y = torch.from_numpy(labels.astype(np.int64)).to(logits.device)
    for b in range(B):
        Tb, Ub1 = int(tl[b]), int(ul[b]) + 1
        g = torch.softmax(logits[b, :Tb, :Ub1].double(), dim=-1)
        ob, ol = occ_b[b, :Tb, :Ub1], occ_l[b, :Tb, :Ub1]
        g *= (ob + ol)[..., None]
        g[..., case["blank"]] -= ob
        if Ub1 > 1:
            idx = y[b, :Ub1 - 1].view(1, -1, 1).expand(Tb, Ub1 - 1, 1)
            g[:, :-1].scatter_add_(2, idx, -ol[:, :-1, None])
        grad[b, :Tb, :Ub1] = g
    return grad


def _best_paths(case, lpb, lpl, tl, ul):
    """Scores, unit frames and spans of the best paths (ties: blank, label, initial jump, final jump)."""
    B, U = case["B"], case["U"]
    score = np.zeros(B)
    frames = np.full((B, U), -1, np.int32)
    span = np.zeros((B, 2), np.int32)
    var = case["variant"]
    lpb, lpl = lpb.cpu().numpy(), lpl.cpu().numpy()
    for b in range(B):
        Tb, Ub = int(tl[b]), int(ul[b])
        pb, pl = lpb[b, :Tb, :Ub + 1], lpl[b, :Tb, :Ub + 1]
        delta = np.full((Tb, Ub + 1), -math.inf)
        by_label = np.zeros((Tb, Ub + 1), bool)
        jumped = np.zeros(Tb, bool)
        delta[0, 0] = 0.0
        for d in range(1, Tb + Ub):
            u = np.arange(max(0, d - Tb + 1), min(d, Ub) + 1)
            t = d - u
            from_blank = np.where(t > 0, delta[t - 1, u] + pb[t - 1, u], -math.inf)
            from_label = np.where(u > 0, delta[t, u - 1] + pl[t, u - 1], -math.inf)
            by_label[t, u] = from_label > from_blank
            delta[t, u] = np.maximum(from_label, from_blank)
            if var != "rnnt" and u[0] == 0 and delta[d, 0] < 0.0:
                delta[d, 0], jumped[d] = 0.0, True
        t_end = Tb - 1
        best = delta[Tb - 1, Ub] + pb[Tb - 1, Ub]
        if var != "rnnt" and Tb >= 2:
            ts = int(np.argmax(delta[:Tb - 1, Ub]))
            jump = delta[ts, Ub] + (pb[Tb - 1, Ub] if var == "wrnnt" else 0.0)
            if jump > best:
                best, t_end = jump, ts
        t, u = t_end, Ub
        while t > 0 or u > 0:
            if u == 0 and jumped[t]:
                break
            if u > 0 and (t == 0 or by_label[t, u]):
                u -= 1
                frames[b, u] = t
            else:
                t -= 1
        score[b] = best
        span[b] = t, t_end
    return [torch.from_numpy(x) for x in (score, frames, span)]


def exact(case, seed):
    elems = case["B"] * case["T"] * (case["U"] + 1) * case["V"]
    if elems > EXACT_ELEMS:
        return None
    logits, labels, tl, ul = _inputs(case, seed)
    lpb, lpl = _log_probs(case, logits, labels)
    if case["path"] == "align":
        return tuple(_best_paths(case, lpb, lpl, tl, ul))
    ln_p, occ_b, occ_l = _lattice(case, lpb, lpl, tl, ul)
    loss, scale = -ln_p, 1.0
    if case["reduction"] == "mean" and case["path"] == "train":
        loss, scale = loss.mean(), 1.0 / case["B"]
    elif case["reduction"] == "sum" and case["path"] == "train":
        loss = loss.sum()
    if case["grad"] == "none":
        return (loss,)
    return loss, _gradient(case, logits, labels, tl, ul, occ_b, occ_l).mul_(scale)
