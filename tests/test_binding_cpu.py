"""The checks that the binding makes on the host before the library is called (no GPU needed): tensors of the device are
stood in for, the library by a recorder that must not be reached."""
import types

import pytest
import torch

from paper_2509_13232_amd import binding as spo


class OnDevice:
    """A tensor that says it is on the GPU."""

    is_cuda = True

    def __init__(self, t):
        self._t = t

    def __getattr__(self, name):
        return getattr(self._t, name)


class Recorder:
    def __init__(self, called):
        self._called = called

    def __getattr__(self, name):
        def f(*a):
            if name.endswith("_bytes"):
                return 256
            self._called.append(name)
            return 0
        return f


@pytest.fixture
def reached(monkeypatch):
    """Names of the library's functions that were called."""
    called = []
    monkeypatch.setattr(spo, "lib", lambda: Recorder(called))
    monkeypatch.setattr(spo, "_calls", types.SimpleNamespace(**{
        n: (lambda *a: None) for n in ("sample_prompts", "advantages", "advantage_diagnostics", "tracker_update", "pg_loss_fwd",
                                       "pg_loss_bwd", "pg_loss_fwd_bwd")}))
    monkeypatch.setattr(spo, "_stream", lambda: 0)
    return called


def _desc(w_layout, T=20, H=64, V=100):
    dev = lambda *shape, dtype=torch.float32: OnDevice(torch.zeros(shape, dtype=dtype))
    W = dev(V, H, dtype=torch.bfloat16) if w_layout == spo.SPO_W_VH else dev(H, V, dtype=torch.bfloat16)
    return spo.make_desc(dev(T, H, dtype=torch.bfloat16), W, dev(T, dtype=torch.int32), dev(T), None, dev(1), dev(2, dtype=torch.int32),
                         0.2, 0.28, w_layout), dev(T), dev(T)


@pytest.mark.parametrize("w_layout", [spo.SPO_W_VH, spo.SPO_W_HV])
@pytest.mark.parametrize("one_call", [False, True])
def test_a_given_d_W_holds_the_head(reached, w_layout, one_call):
    desc, logp, lse = _desc(w_layout)
    shape = (100, 64) if w_layout == spo.SPO_W_VH else (64, 100)

    def call(d_W, **kw):
        if one_call:
            return spo.spo_pg_loss_fwd_bwd(desc, d_W=d_W, **kw)
        return spo.spo_pg_loss_bwd(desc, logp, lse, d_W=d_W, **kw)

    for bad in (OnDevice(torch.zeros(shape[::-1]).t()),           # the head's shape, the other order in memory
                OnDevice(torch.zeros(shape[0], 2 * shape[1])[:, ::2]),
                torch.zeros(shape)):                              # not on the GPU
        with pytest.raises(TypeError, match="d_W"):
            call(bad)
    for bad in (OnDevice(torch.zeros(shape[0] - 1, shape[1])), OnDevice(torch.zeros(0)), OnDevice(torch.zeros(1, dtype=torch.bfloat16))):
        with pytest.raises(ValueError, match="d_W"):
            call(bad)
    assert not reached
    call(OnDevice(torch.zeros(shape)))
    call(OnDevice(torch.zeros(100 * 64)))                         # any shape with the elements in order,
    call(OnDevice(torch.zeros(shape[0] + 28, shape[1])))          # and a buffer that is longer
    call(OnDevice(torch.zeros(1)), want_d_W=False)                # not looked at
    assert len(reached) == 4


def test_calls_without_a_workspace_do_not_ask_for_a_plain_call(reached, monkeypatch):
    asked = []

    class Asked:
        def __getattr__(self, name):
            return lambda *a: asked.append(name)

    monkeypatch.setattr(spo, "_calls", Asked())
    f, i = OnDevice(torch.zeros(16)), OnDevice(torch.zeros(4, dtype=torch.int32))
    r, ws = OnDevice(torch.zeros(4)), OnDevice(torch.zeros(512, dtype=torch.uint8))
    ws.data_ptr = lambda: 256
    desc, logp, lse = _desc(spo.SPO_W_VH)
    d_W = OnDevice(torch.zeros(100, 64))
    spo.spo_sample_prompts(f, f, 4)
    spo.spo_tracker_update(f, f, i, r, r, 0.25, 0.875, 0.96, ids_unique=False)
    spo.spo_pg_loss_fwd(desc)
    for w, g in ((None, d_W), (ws, None), (None, None)):
        spo.spo_pg_loss_bwd(desc, logp, lse, d_W=g, workspace=w)
        spo.spo_pg_loss_fwd_bwd(desc, d_W=g, workspace=w)
    assert len(reached) == 9 and not asked
    # those that might be plain do
    spo.spo_sample_prompts(f, f, 4, workspace=ws)
    spo.spo_advantages(f, f, i, r)
    spo.spo_tracker_update(f, f, i, r, r, 0.25, 0.875, 0.96)
    spo.spo_pg_loss_fwd(desc, workspace=ws)
    spo.spo_pg_loss_bwd(desc, logp, lse, d_W=d_W, workspace=ws)
    spo.spo_pg_loss_fwd_bwd(desc, d_W=d_W, workspace=ws)
    assert asked == ["sample_prompts", "advantages", "tracker_update", "pg_loss_fwd", "pg_loss_bwd", "pg_loss_fwd_bwd"]
