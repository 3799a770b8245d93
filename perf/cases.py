"""The work that a training program hands to this library, as cases that can be timed and compared.

Three kinds of work, each through the entry points of `paper_2509_13232_amd.binding`:

  step    the prompt side of one iteration: draw prompts by priority, advantages of their
          responses, tracker update (optionally the advantage diagnostics);
  head    the token side over hidden states and the LM head: log-probs alone ("forward"), loss then
          gradients as an autograd framework calls them ("two_calls"), or both at once ("one_call");
  logits  the token side where the logits already exist: loss, then their gradient.

Sizes are those of `workloads.CONFIGS`, of the tests and of bench.py, and odd ones between them.
"""
from __future__ import annotations

import ctypes
import math

import numpy as np
import torch

from paper_2509_13232_amd import binding as spo
from paper_2509_13232_amd import workloads as wl

DEV = "cuda"
EPS_LOW, EPS_HIGH = 0.2, 0.28      # clip range of the training configurations
D_HALF, RHO_MIN, RHO_MAX, EPS_EXPLORE = 0.25, 0.875, 0.96, 0.05
HIDDEN, VOCAB = 4096, 151936       # the large LM head of the configurations


def _step(name, N, B, replace=False, repeats=False, diagnostics=False):
    return dict(name=name, kind="step", N=N, B=B, replace=replace, repeats=repeats, diagnostics=diagnostics)


def _head(name, path, dtype, T, B, H, V, mask=0.0, hv=False, dw="fp32", accumulate=False, noise=0.1):
    """mask: share of tokens masked in spans; hv: the head as [H, V]; dw: type of d_W; noise: std of old - current log-prob."""
    return dict(name=name, kind="head", path=path, dtype=dtype, T=T, B=B, H=H, V=V, mask=mask, hv=hv, dw=dw,
                accumulate=accumulate, noise=noise)


def _logits(name, dtype, T, B, V, mask=0.0):
    return dict(name=name, kind="logits", dtype=dtype, T=T, B=B, V=V, mask=mask)


def listed():
    return [
        # the prompt side of the smallest run (16 prompts, 8 responses): nothing but latency and launches
        _step("step_tiny", 16, 8),
        # the prompt side over 2^20 tracked prompts, 4096 distinct ones drawn
        _step("step_million", 1 << 20, 4096),
        # the same for batches that repeat prompts: draws with replacement, updates in batch order, the
        # advantage statistics of a large batch, and the diagnostics that a run logs
        _step("step_repeats", 20000, 40000, replace=True, repeats=True, diagnostics=True),
        # the smallest training step, in fp32: 8 responses of 64 tokens
        _head("head_tiny_fp32", "two_calls", "fp32", 512, 8, 128, 1000, noise=0.05),
        # an odd little batch of a model that keeps its head as [H, V]: tool output masked, d_W summed over mini-batches
        _head("head_ragged_hv", "one_call", "bf16", 713, 5, 256, 3000, mask=0.25, hv=True, accumulate=True),
        # the small model's step: 64 responses of 128 tokens over the full vocabulary
        _head("head_small_model", "one_call", "bf16", 8192, 64, 1024, VOCAB),
        # log-probs of a few short responses (evaluation, the behaviour policy's own log-probs)
        _head("head_score", "forward", "bf16", 1191, 4, HIDDEN, VOCAB),
        # a mini-batch inside an autograd framework: loss, later its gradients, in the weights' own type
        _head("head_mini_batch", "two_calls", "bf16", 17043, 8, HIDDEN, VOCAB, dw="bf16"),
        # a mini-batch of long tool-integrated responses, a fifth of the tokens masked
        _head("head_long_masked", "one_call", "bf16", 46511, 2, HIDDEN, VOCAB, mask=0.2, noise=0.2),
        # the whole batch of the headline benchmark
        _head("head_full_batch", "one_call", "bf16", 284780, 128, HIDDEN, VOCAB),
        # logits that a model's own head has formed, as bench.py sizes them
        _logits("logits_bf16", "bf16", 8192, 4, VOCAB),
        # fp32 logits over a vocabulary of odd size, a few hundred tokens, some of them masked
        _logits("logits_odd_fp32", "fp32", 713, 5, 100003, mask=0.25),
    ]


# ------------------------------------------------------------------ drawn cases
def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_step(rng):
    replace = rng.random() < 0.4
    N = _log_uniform(rng, 16, 1 << 20)
    B = _log_uniform(rng, 8, 40000 if replace else max(8, min(4096, N // 2)))
    return _step("", N, B, replace, replace, rng.random() < 0.3)


def _draw_head(rng):
    if rng.random() < 0.3:
        dtype, T, H, V = "fp32", _log_uniform(rng, 16, 4096), 64 * _log_uniform(rng, 1, 16), _log_uniform(rng, 500, 32000)
    else:
        dtype, T, H, V = "bf16", _log_uniform(rng, 16, 65536), 64 * _log_uniform(rng, 2, 64), _log_uniform(rng, 1000, VOCAB)
        if rng.random() < 0.4:
            V = VOCAB
    path = rng.choice(["forward", "two_calls", "one_call", "one_call"])
    dw = "bf16" if rng.random() < 0.25 else "fp32"
    return _head("", path, dtype, T, max(1, min(128, T // _log_uniform(rng, 16, 4096))), H, V,
                 mask=rng.choice([0.0, 0.0, 0.2]), hv=rng.random() < 0.25, dw=dw,
                 accumulate=dw == "fp32" and path != "forward" and rng.random() < 0.3, noise=rng.choice([0.05, 0.1, 0.2]))


def _draw_logits(rng):
    V = _log_uniform(rng, 1000, VOCAB) if rng.random() < 0.6 else VOCAB
    T = _log_uniform(rng, 4, min(16384, (1 << 30) // V))
    return _logits("", rng.choice(["bf16", "fp32"]), T, max(1, min(64, T // 128)), V, mask=rng.choice([0.0, 0.2]))


def draw(rng):
    case = rng.choice([_draw_step, _draw_head, _draw_head, _draw_logits])(rng)
    del case["name"]
    return case


# ------------------------------------------------------------------ inputs
def _dtype(name):
    return {"fp32": torch.float32, "bf16": torch.bfloat16}[name]


def _lengths(T, B, rng):
    """B response lengths that add up to T, the longest some ten times the shortest."""
    w = rng.uniform(0.1, 1.0, B)
    cuts = np.floor(np.cumsum(w) / w.sum() * T).astype(np.int64)
    cuts[-1] = T
    return np.diff(np.concatenate([[0], cuts]))


def _old_logp(logp, noise):
    """Log-probs under the behaviour policy: the current ones plus noise, no ratio so close to a clip
    bound that a rounding error decides the branch."""
    old = logp + noise
    for _ in range(3):
        ratio = torch.exp(logp - old)
        near = ((ratio / (1.0 - EPS_LOW) - 1.0).abs() < 2e-3) | ((ratio / (1.0 + EPS_HIGH) - 1.0).abs() < 2e-3)
        old = torch.where(near, old + 0.01, old)
    return old


def _target_logp(rows, target, chunk):
    """log-softmax of `rows(s, e)` at the targets, a chunk of tokens at a time."""
    T = target.numel()
    out = torch.empty(T, dtype=torch.float32, device=DEV)
    for s in range(0, T, chunk):
        e = min(T, s + chunk)
        z, zy = rows(s, e)
        out[s:e] = zy - torch.logsumexp(z.float(), dim=1)
    return out


def _responses(case, seed):
    """What a token batch carries besides its hidden states or logits."""
    T, B = case["T"], case["B"]
    rng = np.random.default_rng([seed, 21])
    cu = wl.cu_seqlens(_lengths(T, B, rng))
    adv = rng.standard_normal(B)
    adv = (adv - adv.mean()) / adv.std() if B > 1 else np.ones(1)
    mask = None
    if case["mask"]:
        span = (max(1, min(32, T // 16)), max(2, min(512, T // 4)))
        mask = wl.loss_mask(wl.scaled(wl.CONFIGS["C4"], mask_frac=case["mask"], mask_span=span), T, seed)
    target = wl.target_tokens(T, case["V"], seed)
    to = lambda x: torch.as_tensor(np.ascontiguousarray(x)).to(DEV)  # noqa: E731
    return to(target), None if mask is None else to(mask), to(adv.astype(np.float32)), to(cu)


def _prepare_step(case, seed):
    N, B = case["N"], case["B"]
    cfg = wl.scaled(wl.CONFIGS["C5"], N=N, B=B)
    a, b = wl.tracker_state(cfg, seed)
    rng = np.random.default_rng([seed, 22])
    to = lambda x: torch.as_tensor(np.asarray(x, np.float32)).to(DEV)  # noqa: E731
    L = spo.lib()
    s = dict(kind="step", B=B, alpha=to(a), beta=to(b), reward=to(rng.random(B) < 0.4), kl=to(rng.exponential(0.02, B)),
             replace=case["replace"], repeats=case["repeats"], diagnostics=case["diagnostics"], seed=int(seed), iteration=0)
    space = lambda n: torch.empty(max(256, int(n)), dtype=torch.uint8, device=DEV)  # noqa: E731
    s["ws_sample"] = space(L.spo_sample_prompts_workspace_bytes(N, B))
    s["ws_adv"] = space(L.spo_advantages_workspace_bytes(B))
    s["ws_update"] = space(L.spo_tracker_update_workspace_bytes(N)) if case["repeats"] else None
    return s


def _prepare_head(case, seed):
    T, H, V = case["T"], case["H"], case["V"]
    hidden = wl.hidden_states(T, H, case["dtype"], DEV, seed)
    W = wl.lm_head(V, H, case["dtype"], 0.02, DEV, seed)
    target, mask, adv, cu = _responses(case, seed)

    def rows(s, e):
        h, y = hidden[s:e], target[s:e].long()
        return h @ W.t(), (h.float() * W[y].float()).sum(dim=1)

    logp = _target_logp(rows, target, max(256, (1 << 28) // V))
    old = _old_logp(logp, torch.as_tensor(wl.logp_noise(T, case["noise"], seed)).to(DEV))
    if case["hv"]:
        W = W.t().contiguous()
    desc = spo.make_desc(hidden, W, target, old, mask, adv, cu, EPS_LOW, EPS_HIGH, spo.SPO_W_HV if case["hv"] else spo.SPO_W_VH)
    s = dict(kind="head", path=case["path"], desc=desc, d_W=None, ws=None, ws_fwd=None, accumulate=case["accumulate"])
    # what a program keeps from step to step: the workspaces and the weight gradient
    space = lambda n: torch.empty(max(256, int(n)), dtype=torch.uint8, device=DEV)  # noqa: E731
    if case["path"] == "one_call":
        s["ws"] = space(spo.spo_pg_loss_fwd_bwd_workspace_bytes(desc))
    else:
        s["ws_fwd"] = space(spo.lib().spo_pg_loss_fwd_workspace_bytes(ctypes.byref(desc[0])))
        if case["path"] == "two_calls":
            s["ws"] = space(spo.spo_pg_loss_bwd_workspace_bytes(desc))
    if case["path"] != "forward":
        s["d_W"] = torch.zeros(W.shape, dtype=_dtype(case["dw"]), device=DEV)
    return s


def _prepare_logits(case, seed):
    T, V = case["T"], case["V"]
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) + 31)
    logits = torch.empty((T, V), dtype=_dtype(case["dtype"]), device=DEV)
    for s in range(0, T, 1024):
        e = min(T, s + 1024)
        logits[s:e] = torch.randn((e - s, V), generator=g, device=DEV) * 2.0
    target, mask, adv, cu = _responses(case, seed)

    def rows(s, e):
        z = logits[s:e].float()
        return z, z.gather(1, target[s:e].long()[:, None])[:, 0]

    logp = _target_logp(rows, target, 512)
    old = _old_logp(logp, torch.as_tensor(wl.logp_noise(T, 0.1, seed)).to(DEV))
    desc = spo.make_desc(None, None, target, old, mask, adv, cu, EPS_LOW, EPS_HIGH, logits=logits)
    space = lambda n: torch.empty(max(256, int(n)), dtype=torch.uint8, device=DEV)  # noqa: E731
    return dict(kind="logits", desc=desc, ws_fwd=space(spo.lib().spo_pg_loss_fwd_workspace_bytes(ctypes.byref(desc[0]))),
                ws=space(spo.spo_pg_loss_bwd_workspace_bytes(desc)))


def prepare(case, seed):
    return {"step": _prepare_step, "head": _prepare_head, "logits": _prepare_logits}[case["kind"]](case, int(seed))


# ------------------------------------------------------------------ one pass
def _run_step(s):
    a, b = s["alpha"], s["beta"]
    s["iteration"] += 1
    idx = spo.spo_sample_prompts(a, b, s["B"], EPS_EXPLORE, s["seed"], s["iteration"], s["replace"], workspace=s["ws_sample"])
    raw, adv, stats = spo.spo_advantages(a, b, idx, s["reward"], workspace=s["ws_adv"])
    spo.spo_tracker_update(a, b, idx, s["reward"], s["kl"], D_HALF, RHO_MIN, RHO_MAX, ids_unique=not s["repeats"],
                           workspace=s["ws_update"])
    out = dict(idx=idx, raw=raw, adv=adv, stats=stats, alpha=a, beta=b)
    if s["diagnostics"]:
        out["diagnostics"] = spo.spo_advantage_diagnostics(raw, s["reward"])
    return out


def _run_head(s):
    desc = s["desc"]
    if s["path"] == "one_call":
        loss, logp, lse, stats, dx, dw = spo.spo_pg_loss_fwd_bwd(desc, 1.0, d_W=s["d_W"], accumulate_dW=s["accumulate"],
                                                                 workspace=s["ws"])
        return dict(loss=loss, logp=logp, lse=lse, stats=stats, d_hidden=dx, d_W=dw)
    loss, logp, lse, stats = spo.spo_pg_loss_fwd(desc, workspace=s["ws_fwd"])
    out = dict(loss=loss, logp=logp, lse=lse, stats=stats)
    if s["path"] == "two_calls":
        out["d_hidden"], out["d_W"] = spo.spo_pg_loss_bwd(desc, logp, lse, 1.0, d_W=s["d_W"], accumulate_dW=s["accumulate"],
                                                          workspace=s["ws"])
    return out


def _run_logits(s):
    loss, logp, lse, stats = spo.spo_pg_loss_fwd(s["desc"], workspace=s["ws_fwd"])
    return dict(loss=loss, logp=logp, lse=lse, stats=stats, d_logits=spo.spo_pg_loss_bwd(s["desc"], logp, lse, 1.0, workspace=s["ws"]))


def run(state):
    return {"step": _run_step, "head": _run_head, "logits": _run_logits}[state["kind"]](state)


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    if case["kind"] == "step":
        # the tracker is read once for the weights; per response: id, reward, KL in, two advantages out,
        # the prompt's two counters read and rewritten
        return {"bytes": 8 * case["N"] + 36 * case["B"], "flops": 0}
    T, V, elt = case["T"], case["V"], 4 if case["dtype"] == "fp32" else 2
    live = T * (1.0 - case["mask"])          # tokens that can carry a gradient
    if case["kind"] == "logits":
        # read for the log-sum-exp, read again (masked rows are not) for the gradient, which is written
        return {"bytes": elt * V * (2 * T + live), "flops": 0}
    H, head = case["H"], case["H"] * V
    if case["path"] == "forward":
        return {"bytes": elt * (T * H + head), "flops": 2.0 * T * head}
    # logits of every token, dHidden and dW of the tokens that can carry a gradient; the backward of
    # the two calls has only the log-sum-exps to go by and forms the logits once more
    contractions = 2.0 if case["path"] == "one_call" else 3.0
    dw = (4 if case["dw"] == "fp32" else 2) * (2 if case["accumulate"] else 1)
    return {"bytes": elt * (2 * T * H + head) + dw * head, "flops": 2.0 * head * (T + contractions * live)}


def tolerance(case):
    # about four times the distance to the same pass in fp64 (in brackets)
    if case["kind"] == "step":
        # statistics in fp64, one rounding to fp32 each
        return {"rel": 3e-7, "max": 1e-6}
    if case["kind"] == "logits":
        # bf16 gradients (1.5e-3, 4e-3 at most); fp32 exponentials of long rows (5e-7, 3e-6 at most)
        return {"rel": 5e-3, "max": 2e-2} if case["dtype"] == "bf16" else {"rel": 1e-5, "max": 1e-4}
    if case["path"] == "forward":
        # 32-bit sums over the hidden size and the vocabulary; the loss is a sum of both signs (3e-7)
        return {"rel": 1e-5, "max": 1e-4}
    # bf16 logit gradients and operands (2.4e-3; single entries of d_W, sums of both signs, up to 0.17)
    return {"rel": 1e-2, "max": 0.5}
