"""The binding's plain calls (csrc/calls.cpp) against the general way through ctypes: the same bits, and the same errors."""
import numpy as np
import pytest
import torch

from paper_2509_13232_amd import workloads as wl
from pg_cases import Case, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def spo():
    from paper_2509_13232_amd import binding
    binding.lib()
    return binding


class Nothing:
    """Stands in for the extension: no call is plain."""

    def __getattr__(self, name):
        return lambda *a: None


def both_ways(spo, monkeypatch, call):
    """What `call` gives by the plain way, which has to be taken, and by the general one."""
    real, taken = spo._plain_calls(), []

    class Watch:
        def __getattr__(self, name):
            def f(*a):
                out = getattr(real, name)(*a)
                taken.append(out is not None)
                return out
            return f

    res = []
    for way in (Watch(), Nothing()):
        with monkeypatch.context() as m:
            m.setattr(spo, "_calls", way)
            res.append(call())
    torch.cuda.synchronize()
    assert taken and all(taken)
    return res


def same(a, b):
    if isinstance(a, (tuple, list)):
        assert type(a) is type(b) and len(a) == len(b)
        for x, y in zip(a, b):
            same(x, y)
    elif a is None:
        assert b is None
    else:
        assert a.dtype == b.dtype and a.shape == b.shape and a.device == b.device and torch.equal(a, b)


def space(n):
    return torch.empty(max(256, int(n)), dtype=torch.uint8, device="cuda")


@pytest.mark.parametrize("unique", [True, False])
@pytest.mark.parametrize("replace", [True, False])
def test_prompt_step(spo, monkeypatch, unique, replace):
    say(f"plain calls of a prompt step, unique={unique} replace={replace}")
    N, B = 500, 40
    rng = np.random.default_rng(3)
    f = lambda lo, hi, n: torch.as_tensor(rng.uniform(lo, hi, n).astype(np.float32)).cuda()
    a0, b0, r, kl = f(.5, 50, N), f(.5, 50, N), f(0, 1, B).round(), f(0, .1, B)
    L = spo.lib()
    ws, wt, wa = (space(x) for x in (L.spo_sample_prompts_workspace_bytes(N, B), L.spo_tracker_update_workspace_bytes(N),
                                     L.spo_advantages_workspace_bytes(B)))
    def step():
        a, b = a0.clone(), b0.clone()
        idx, info = spo.spo_sample_prompts(a, b, B, 0.05, 1 << 63, -3, replace, workspace=ws, return_info=True)
        adv = spo.spo_advantages(a, b, idx, r, 1, 1e-6, workspace=wa)
        assert spo.spo_tracker_update(a, b, idx, r, kl, 0.25, 0.875, 0.96, ids_unique=unique, workspace=None if unique else wt) is None
        return idx, info, adv, a, b, spo.spo_advantage_diagnostics(adv[0], r, 0, 1)
    same(*both_ways(spo, monkeypatch, step))


@pytest.mark.parametrize("w_layout", [0, 1])
@pytest.mark.parametrize("dw_dtype", [torch.float32, torch.bfloat16])
def test_loss(spo, monkeypatch, oracle, w_layout, dw_dtype):
    say(f"plain calls of the loss, layout={w_layout} d_W {dw_dtype}")
    case = Case(wl.scaled(wl.CONFIGS["C2"], name="plain", H=128, V=600), [30, 90])
    case.set_old_from_oracle(oracle)
    desc = case.to_gpu(spo, w_layout)
    shape = (128, 600) if w_layout else (600, 128)
    wf = space(spo.lib().spo_pg_loss_fwd_workspace_bytes(desc[0]))
    wb, wo = space(spo.spo_pg_loss_bwd_workspace_bytes(desc, 256)), space(spo.spo_pg_loss_fwd_bwd_workspace_bytes(desc))
    def loss():
        dw = [torch.ones(shape, dtype=dw_dtype, device="cuda") for _ in range(2)]
        add = dw_dtype == torch.float32
        fwd = spo.spo_pg_loss_fwd(desc, workspace=wf)
        back = spo.spo_pg_loss_bwd(desc, fwd[1], fwd[2], 2, d_W=dw[0], accumulate_dW=add, chunk_tokens=256, workspace=wb)
        one = spo.spo_pg_loss_fwd_bwd(desc, -0.5, d_W=dw[1], accumulate_dW=add, workspace=wo)
        assert back[1] is dw[0] and one[5] is dw[1]
        return fwd, back, one
    same(*both_ways(spo, monkeypatch, loss))


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_logits(spo, monkeypatch, dtype):
    say(f"plain calls of the logits-in form, {dtype}")
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    z = torch.randn((50, 777), generator=g, device="cuda").to(dtype)
    i32 = lambda x: torch.as_tensor(x, dtype=torch.int32).cuda()
    desc = spo.make_desc(None, None, i32(np.arange(50) * 7), torch.full((50,), -6.0, device="cuda"), None,
                         torch.tensor([1.0, -1.0], device="cuda"), i32([0, 20, 50]), 0.2, 0.28, logits=z)
    wf, wb = space(spo.lib().spo_pg_loss_fwd_workspace_bytes(desc[0])), space(spo.spo_pg_loss_bwd_workspace_bytes(desc))
    def loss():
        fwd = spo.spo_pg_loss_fwd(desc, workspace=wf)
        return fwd, spo.spo_pg_loss_bwd(desc, fwd[1], fwd[2], 1.0, workspace=wb)
    same(*both_ways(spo, monkeypatch, loss))


def test_errors_are_those_of_the_general_way(spo, monkeypatch):
    say("plain calls: errors")
    a, b = torch.ones(64, device="cuda"), torch.ones(64, device="cuda")
    ws = space(spo.lib().spo_sample_prompts_workspace_bytes(64, 8))
    idx, r = torch.zeros(8, dtype=torch.int32, device="cuda"), torch.zeros(8, device="cuda")
    calls = [
        lambda: spo.spo_sample_prompts(a, b, 65, workspace=ws),                       # more than there are
        lambda: spo.spo_sample_prompts(a, b, -1, workspace=ws),
        lambda: spo.spo_sample_prompts(a, b, 8, workspace=ws[1:]),
        lambda: spo.spo_sample_prompts(a, b[:-1], 8, workspace=ws),
        lambda: spo.spo_sample_prompts(a.double(), b, 8, workspace=ws),
        lambda: spo.spo_sample_prompts(a.cpu(), b, 8, workspace=ws),
        lambda: spo.spo_sample_prompts(a, b, 8, 1.5, workspace=ws),
        lambda: spo.spo_sample_prompts(a, b, 8, 10 ** 400, workspace=ws),             # an int that no double holds
        lambda: spo.spo_advantages(a, b, idx, r, 0, -10 ** 400),
        lambda: spo.spo_advantage_diagnostics(r, r, 0, 10 ** 400),
        lambda: spo.spo_tracker_update(a, b, idx, r, r, 10 ** 400, 0.875, 0.96),
        lambda: spo.spo_advantages(a, b, idx.long(), r),
        lambda: spo.spo_advantages(a, b, idx, r, ddof=2),
        lambda: spo.spo_advantages(a, b, idx, r, workspace=ws[8:]),
        lambda: spo.spo_advantage_diagnostics(r, r[:-1]),
        lambda: spo.spo_advantage_diagnostics(r, r, 0.5, 0.1),
        lambda: spo.spo_tracker_update(a, b, idx, r, r, -1.0, 0.875, 0.96),
        lambda: spo.spo_tracker_update(a, b, idx, r, r[::2], 0.25, 0.875, 0.96),
        lambda: spo.spo_tracker_update(a, b, idx, r, r, 0.25, 0.875, 0.96, ids_unique=False, workspace=ws[:0]),
    ]
    case = Case(wl.scaled(wl.CONFIGS["C2"], name="plain", H=128, V=600), [30, 90])
    case.old = np.full(case.T, -6.0, np.float32)
    desc = case.to_gpu(spo)
    logp = torch.full((case.T,), -6.0, device="cuda")
    wb, wo = space(spo.spo_pg_loss_bwd_workspace_bytes(desc)), space(spo.spo_pg_loss_fwd_bwd_workspace_bytes(desc))
    for d_W in (torch.zeros(599, 128, device="cuda"), torch.zeros(128, 600, device="cuda").t(), torch.zeros(600, 128)):  # short, across, on the host
        calls += [lambda d_W=d_W: spo.spo_pg_loss_bwd(desc, logp, logp, d_W=d_W, workspace=wb),
                  lambda d_W=d_W: spo.spo_pg_loss_fwd_bwd(desc, d_W=d_W, workspace=wo)]
    for i, call in enumerate(calls):
        seen = []
        for way in (spo._plain_calls(), Nothing()):
            with monkeypatch.context() as m:
                m.setattr(spo, "_calls", way)
                with pytest.raises(Exception) as e:
                    call()
                seen.append((type(e.value), str(e.value), getattr(e.value, "status", None)))
        assert seen[0] == seen[1], (i, seen)


@pytest.mark.parametrize("under", ["grad", "jvp", "functionalize", "vmap"])
def test_calls_under_a_transform_take_the_general_way(spo, monkeypatch, under):
    # outputs made under a transform may have no memory to write to: what then happens (an error, or a result) is the
    # general way's business
    say(f"plain calls under {under}")
    raw, r = torch.linspace(-1, 1, 24, device="cuda"), torch.ones(24, device="cuda")
    x = torch.ones(2, device="cuda")
    seen = []

    def f(t):
        try:
            d = spo.spo_advantage_diagnostics(raw, r)
            seen[-1].append("result" if torch._C._functorch.is_functorch_wrapped_tensor(d) else d.cpu().tolist())
        except Exception as e:
            seen[-1].append((type(e), str(e), getattr(e, "status", None)))
        return t.sum()

    F = torch.func
    run = {"grad": lambda: F.grad(f)(x), "jvp": lambda: F.jvp(f, (x,), (x,)), "functionalize": lambda: F.functionalize(f)(x),
           "vmap": lambda: F.vmap(f)(x[None])}[under]
    real = spo._plain_calls()
    for way in (real, Nothing()):
        seen.append([])
        with monkeypatch.context() as m:
            m.setattr(spo, "_calls", way)
            run()
    torch.cuda.synchronize()
    assert seen[0] and seen[0] == seen[1], seen
    # afterwards calls are plain again, and other threads run
    assert real.advantage_diagnostics(raw, r, 1e-4, 0.02) is not None
