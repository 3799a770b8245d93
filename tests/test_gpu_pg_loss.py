"""GPU parity of the clipped policy-gradient loss (fused LM-head form and
logits-in form, forward and backward) against the fp64 oracle, through the C ABI.

Tolerances: lse / logp absolute 2e-4 (bf16 inputs, fp32 accumulation), loss 2e-3
relative, gradients 1e-2 relative L2; fp32 inputs: lse / logp absolute 2e-5."""
import numpy as np
import pytest
import torch

from paper_2509_13232_amd import workloads as wl
from pg_cases import Case, check_forward, f64, rel_l2, say

pytestmark = pytest.mark.gpu
GRAD_TOL = 1e-2


@pytest.fixture(scope="module")
def spo():
    from paper_2509_13232_amd import binding
    binding.lib()
    assert torch.cuda.is_available()
    return binding


MID = wl.scaled(wl.CONFIGS["C2"], name="mid", H=256, V=3000, mask_span=(4, 40))
MID_LENGTHS = [37, 300, 1, 255, 120]  # T = 713: three token tiles, ragged tail; V: 11 tiles + 184


@pytest.fixture(params=[False, True], ids=["fwd_then_bwd", "one_call"])
def one_call(request):
    """The two ways to the gradients: spo_pg_loss_fwd followed by spo_pg_loss_bwd (the logits are
    formed twice), or spo_pg_loss_fwd_bwd (formed once and kept, piece by piece, as fp16)."""
    return request.param


def run_fwd_bwd(spo, case, w_layout=0, chunk_tokens=0, dx_dtype=torch.float32, dw_dtype=torch.float32,
                one_call=False):
    desc = case.to_gpu(spo, w_layout)
    if one_call:
        *fwd, dx, dw = spo.spo_pg_loss_fwd_bwd(desc, 1.0, d_hidden_dtype=dx_dtype, d_W_dtype=dw_dtype,
                                               chunk_tokens=chunk_tokens)
        fwd = tuple(fwd)
    else:
        fwd = spo.spo_pg_loss_fwd(desc)
        dx, dw = spo.spo_pg_loss_bwd(desc, fwd[1], fwd[2], 1.0, d_hidden_dtype=dx_dtype, d_W_dtype=dw_dtype,
                                     chunk_tokens=chunk_tokens)
    torch.cuda.synchronize()
    if w_layout == 1:
        dw = dw.t()
    return fwd, dx, dw


@pytest.mark.parametrize("w_layout", [0, 1])
def test_tiny_spo_step_fp32(spo, oracle, w_layout, one_call):
    cfg = wl.CONFIGS["C1"]
    say(f"fused fp32 C1 T=512 H=128 V=1000 w_layout={w_layout} one_call={one_call}")
    case = Case(cfg)
    assert case.T == 512
    case.set_old_from_oracle(oracle)
    fwd, dx, dw = run_fwd_bwd(spo, case, w_layout=w_layout, one_call=one_call)
    check_forward(case, oracle, fwd, atol_logp=2e-5)
    rb = oracle.pg_loss_bwd(*case.oracle_inputs(), *case.eps)
    assert rel_l2(f64(dx), rb["d_hidden"]) < GRAD_TOL
    assert rel_l2(f64(dw), rb["d_W"]) < GRAD_TOL


@pytest.mark.parametrize("w_layout", [0, 1])
@pytest.mark.parametrize("w_scale,mask_frac", [(1.0, 0.0), (1.0, 0.25), (30.0, 0.25)])
def test_fused_bf16_matches_oracle(spo, oracle, w_layout, w_scale, mask_frac, one_call):
    say(f"fused bf16 mid T=713 H=256 V=3000 w_layout={w_layout} w_scale={w_scale} mask={mask_frac} one_call={one_call}")
    case = Case(MID, MID_LENGTHS, w_scale=w_scale, mask_frac=mask_frac)
    case.set_old_from_oracle(oracle)
    fwd, dx, dw = run_fwd_bwd(spo, case, w_layout, one_call=one_call)
    ref = check_forward(case, oracle, fwd)
    assert 0 < ref["active"].sum() < case.T          # both branches of the min occur
    rb = oracle.pg_loss_bwd(*case.oracle_inputs(), *case.eps)
    assert rel_l2(f64(dx), rb["d_hidden"]) < GRAD_TOL
    assert rel_l2(f64(dw), rb["d_W"]) < GRAD_TOL
    # the softmax part alone (gradient minus the rank-one target term), which a flat
    # softmax hides inside the total: bounded by the bf16 rounding of the logit
    # gradients of both parts
    g = rb["g"]
    Wd, Hd = f64(case.W), f64(case.hidden)
    onehot_dx = g[:, None] * Wd[case.target]
    soft_ref = rb["d_hidden"] - onehot_dx
    soft_gpu = f64(dx) - onehot_dx
    # (a target entry of dZ is rounded to bf16 once: at most 2^-9 of it)
    bound = GRAD_TOL * np.linalg.norm(soft_ref) + 1.1 * 2.0 ** -9 * np.linalg.norm(onehot_dx)
    assert np.linalg.norm(soft_gpu - soft_ref) <= bound
    if w_scale > 1.0:   # peaked softmax: the softmax part is as large as the target part
        assert np.linalg.norm(soft_ref) > 0.3 * np.linalg.norm(onehot_dx)
        assert rel_l2(soft_gpu, soft_ref) < 2 * GRAD_TOL
    # rows of masked tokens are exactly zero; softmax rows sum to one
    if case.mask is not None:
        assert not dx[torch.as_tensor(case.mask == 0)].any()
    col = f64(dw).sum(axis=0)
    assert np.abs(col).max() <= 2e-2 * np.abs(f64(dw)).sum(axis=0).max()
    del Hd


def test_backward_chunks_and_output_dtypes(spo, oracle, one_call):
    say(f"fused bf16 mid, chunk_tokens=256 (3 chunks), bf16 outputs, one_call={one_call}")
    case = Case(MID, MID_LENGTHS, mask_frac=0.25)
    case.set_old_from_oracle(oracle)
    rb = oracle.pg_loss_bwd(*case.oracle_inputs(), *case.eps)
    f1, dx1, dw1 = run_fwd_bwd(spo, case, chunk_tokens=256, one_call=one_call)
    f2, dx2, dw2 = run_fwd_bwd(spo, case, chunk_tokens=0, one_call=one_call)
    check_forward(case, oracle, f1)
    assert torch.allclose(f1[1], f2[1], atol=1e-5, rtol=0)            # a token's log-prob does not depend on the pieces
    assert rel_l2(f64(dx1), rb["d_hidden"]) < GRAD_TOL and rel_l2(f64(dw1), rb["d_W"]) < GRAD_TOL
    assert rel_l2(f64(dx1), f64(dx2)) < 1e-5           # rows depend on the chunking only through the order of fp32 sums
    assert rel_l2(f64(dw1), f64(dw2)) < 1e-5           # fp32 partial sums in another order
    _, dx3, dw3 = run_fwd_bwd(spo, case, chunk_tokens=512, dx_dtype=torch.bfloat16, dw_dtype=torch.bfloat16,
                              one_call=one_call)
    assert dx3.dtype == torch.bfloat16 and dw3.dtype == torch.bfloat16
    assert rel_l2(f64(dx3), rb["d_hidden"]) < GRAD_TOL and rel_l2(f64(dw3), rb["d_W"]) < GRAD_TOL


@pytest.mark.parametrize("mask_frac", [None, 0.25], ids=["no_mask", "masked"])
def test_one_call_with_only_one_of_the_two_gradients(spo, oracle, mask_frac):
    # d_hidden alone, d_W alone, neither (loss and log-probs only): the one call skips what is not asked for
    say(f"one call, single outputs, mask={mask_frac}")
    case = Case(MID, MID_LENGTHS, mask_frac=mask_frac)
    case.set_old_from_oracle(oracle)
    desc = case.to_gpu(spo)
    rb = oracle.pg_loss_bwd(*case.oracle_inputs(), *case.eps)
    *fwd, dx, dw = spo.spo_pg_loss_fwd_bwd(desc, 1.0, d_hidden_dtype=torch.float32, want_d_W=False)
    torch.cuda.synchronize()
    check_forward(case, oracle, tuple(fwd))
    assert dw is None and rel_l2(f64(dx), rb["d_hidden"]) < GRAD_TOL
    *fwd, dx, dw = spo.spo_pg_loss_fwd_bwd(desc, 1.0, want_d_hidden=False)
    torch.cuda.synchronize()
    check_forward(case, oracle, tuple(fwd))
    assert dx is None and rel_l2(f64(dw), rb["d_W"]) < GRAD_TOL
    *fwd, dx, dw = spo.spo_pg_loss_fwd_bwd(desc, 1.0, want_d_hidden=False, want_d_W=False)
    torch.cuda.synchronize()
    check_forward(case, oracle, tuple(fwd))
    assert dx is None and dw is None
    # grad_loss scales both gradients
    _, _, _, _, dx2, dw2 = spo.spo_pg_loss_fwd_bwd(desc, -2.5, d_hidden_dtype=torch.float32)
    torch.cuda.synchronize()
    assert rel_l2(f64(dx2), -2.5 * rb["d_hidden"]) < GRAD_TOL and rel_l2(f64(dw2), -2.5 * rb["d_W"]) < GRAD_TOL


@pytest.mark.parametrize("w_layout", [0, 1])
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_head_gradient_on_ragged_shapes(spo, oracle, w_layout, dtype, one_call):
    # dW contracts over tokens from rows of dZ and of the hidden states: a vocabulary that is
    # neither a multiple of the tile nor of the 8-element pieces the rows are fetched in, a
    # hidden size below one tile, a token count with a ragged last tile.  Element-wise check:
    # a misplaced column or a piece fetched past the end of a row shows up in single entries.
    say(f"fused {dtype} ragged T=300 H=192 V=1003 w_layout={w_layout} one_call={one_call}")
    cfg = wl.scaled(MID, name="ragged", H=192, V=1003, dtype=dtype)
    case = Case(cfg, [130, 170])
    case.set_old_from_oracle(oracle)
    fwd, dx, dw = run_fwd_bwd(spo, case, w_layout, one_call=one_call)
    check_forward(case, oracle, fwd, atol_logp=2e-4 if dtype == "bf16" else 2e-5)
    rb = oracle.pg_loss_bwd(*case.oracle_inputs(), *case.eps)
    assert dw.shape == (1003, 192)
    assert rel_l2(f64(dx), rb["d_hidden"]) < GRAD_TOL and rel_l2(f64(dw), rb["d_W"]) < GRAD_TOL
    scale = np.abs(rb["d_W"]).max()
    np.testing.assert_allclose(f64(dw), rb["d_W"], atol=2e-2 * scale, rtol=0)
    # every vocabulary row's gradient against its own size (the target rows dominate the total)
    rows = np.linalg.norm(f64(dw) - rb["d_W"], axis=1)
    assert (rows <= 5e-2 * np.linalg.norm(rb["d_W"], axis=1) + 1e-3 * scale).all()


@pytest.mark.parametrize("lengths,V,H,w_layout,chunk", [
    ([1], 5, 64, 0, 0),              # one token, vocabulary below one fetch piece
    ([1], 5, 64, 1, 0),
    ([200, 55], 63, 128, 1, 0),      # one short of a k-block of the vocabulary, one short of a token tile
    ([129, 128], 65, 64, 0, 256),    # one past both, two chunks
    ([500, 12], 1023, 192, 1, 256),  # one short of four vocabulary tiles
    ([150, 150], 2049, 256, 0, 0),   # one past eight vocabulary tiles
    ([40], 300, 320, 1, 0),          # hidden size between one and two tiles
])
def test_corner_shapes_match_oracle(spo, oracle, lengths, V, H, w_layout, chunk, one_call):
    # sizes that sit on, just below and just above the tile, block and fetch-piece boundaries of
    # the contraction kernels, forward and both gradients against the oracle
    say(f"fused bf16 corner T={sum(lengths)} H={H} V={V} w_layout={w_layout} chunk={chunk} one_call={one_call}")
    cfg = wl.scaled(MID, name="corner", H=H, V=V)
    case = Case(cfg, lengths)
    case.set_old_from_oracle(oracle)
    fwd, dx, dw = run_fwd_bwd(spo, case, w_layout, chunk_tokens=chunk, one_call=one_call)
    check_forward(case, oracle, fwd)
    rb = oracle.pg_loss_bwd(*case.oracle_inputs(), *case.eps)
    assert dw.shape == (V, H) and dx.shape == (sum(lengths), H)
    if np.any(rb["d_hidden"]):
        assert rel_l2(f64(dx), rb["d_hidden"]) < GRAD_TOL and rel_l2(f64(dw), rb["d_W"]) < GRAD_TOL
        scale = np.abs(rb["d_W"]).max()
        np.testing.assert_allclose(f64(dw), rb["d_W"], atol=2e-2 * scale, rtol=0)
    else:   # every token ended on the clipped branch
        assert not dx.any() and not dw.any()


@pytest.mark.parametrize("w_layout,chunk", [(0, 0), (1, 512)])
def test_last_round_of_dW_tiles_cut_along_the_tokens(spo, oracle, w_layout, chunk, one_call):
    # 33 x 8 = 264 tiles of d_W on 256 compute units: the 8 tiles of the last round are launched on
    # their own, each cut into 8 runs of tokens whose partial tiles are added in order (with chunk =
    # 512 two launches add into d_W; 900 tokens are 16 k-steps: two per part in the first chunk, one or
    # none in the second).  Every entry against the oracle, the tiles of the last round on their own.
    V, H = 8200, 2048
    say(f"fused bf16 T=900 H={H} V={V} w_layout={w_layout} chunk={chunk} one_call={one_call}: d_W tail tiles")
    cfg = wl.scaled(MID, name="tail", H=H, V=V)
    case = Case(cfg, [400, 500])
    case.set_old_from_oracle(oracle)
    fwd, dx, dw = run_fwd_bwd(spo, case, w_layout, chunk_tokens=chunk, one_call=one_call)
    check_forward(case, oracle, fwd)
    rb = oracle.pg_loss_bwd(*case.oracle_inputs(), *case.eps)
    got = f64(dw)
    assert rel_l2(f64(dx), rb["d_hidden"]) < GRAD_TOL and rel_l2(got, rb["d_W"]) < GRAD_TOL
    scale = np.abs(rb["d_W"]).max()
    np.testing.assert_allclose(got, rb["d_W"], atol=2e-2 * scale, rtol=0)
    # in the row-major order of 256 x 256 tiles of the kernel's output ([V, H], or [H, V] for w_layout 1)
    # the last 8 tiles are the last tile row: vocabulary entries from 8192 on, or hidden units from 1792 on
    tail = (slice(8192, V), slice(None)) if w_layout == 0 else (slice(None), slice(1792, H))
    assert np.abs(rb["d_W"][tail]).max() > 0
    assert rel_l2(got[tail], rb["d_W"][tail]) < 2 * GRAD_TOL


@pytest.mark.parametrize("mask_frac", [None, 0.02], ids=["no_mask", "masked"])
def test_last_round_of_dHidden_tiles_cut_along_the_vocabulary(spo, oracle, mask_frac, one_call):
    # ~8300 rows x 2048 hidden units: 33 x 8 = 264 tiles of d_hidden on 256 compute units, so the 8 tiles
    # of the last round (the last 52 tokens) are cut into 8 runs of the vocabulary (9 k-steps: five parts
    # have work).  Without a mask the one call knows the tile count on the host; otherwise the number of
    # active tokens, and with it whether and where to cut, is known on the device only.
    # (token counts chosen so that the rows the contraction runs over, all tokens or the ~97-99 % with a
    # gradient, fall into the 33rd row tile)
    T = 8300 if (one_call and mask_frac is None) else 8400 if mask_frac is None else 8560
    say(f"fused bf16 T={T} H=2048 V=520 mask={mask_frac} one_call={one_call}: d_hidden tail tiles")
    cfg = wl.scaled(MID, name="dxtail", H=2048, V=520)
    case = Case(cfg, [4000, T - 4000], mask_frac=mask_frac)
    case.set_old_from_oracle(oracle)
    fwd, dx, dw = run_fwd_bwd(spo, case, one_call=one_call)
    ref = check_forward(case, oracle, fwd)
    rb = oracle.pg_loss_bwd(*case.oracle_inputs(), *case.eps)
    n_active = int(np.count_nonzero(rb["g"]))
    rows = T if (one_call and mask_frac is None) else n_active
    assert 8192 < rows <= 8448, rows        # 33 row tiles: a last round of 8 tiles
    got = f64(dx)
    assert rel_l2(got, rb["d_hidden"]) < GRAD_TOL and rel_l2(f64(dw), rb["d_W"]) < GRAD_TOL
    per_row = np.linalg.norm(got - rb["d_hidden"], axis=1)
    scale = np.linalg.norm(rb["d_hidden"], axis=1)
    assert (per_row <= 2 * GRAD_TOL * scale + 1e-12).all()     # every token's row, those of the cut tiles included
    assert not got[scale == 0].any()


@pytest.mark.parametrize("T,H,V", [
    (600, 1344, 11200),    # 44 x 6 tiles of d_W in bands of 24: the 8 cut tiles are the end of the last, half a band
    (11300, 1344, 520)])   # 45 x 6 of d_hidden: 14 cut tiles, two thirds of a patch of 4 x 6 and a row of 6
def test_cut_tiles_where_bands_divide_no_round(spo, oracle, T, H, V, one_call):
    say(f"fused bf16 T={T} H={H} V={V} one_call={one_call}: cut tiles in the order of the launch")
    case = Case(wl.scaled(MID, name="bands", H=H, V=V), [T // 3, T - T // 3])
    case.set_old_from_oracle(oracle)
    fwd, dx, dw = run_fwd_bwd(spo, case, one_call=one_call)
    rb = oracle.pg_loss_bwd(*case.oracle_inputs(), *case.eps)
    for got, ref in ((f64(dx), rb["d_hidden"]), (f64(dw), rb["d_W"])):
        assert rel_l2(got, ref) < GRAD_TOL
        np.testing.assert_allclose(got, ref, atol=2e-2 * np.abs(ref).max(), rtol=0)


DEEP = wl.scaled(wl.CONFIGS["C2"], name="deep", H=320, V=1100)
DEEP_LENGTHS = [9000, 7000, 12001, 5000, 6999]  # T = 40000: 157 token tiles, three chunks of 16384


@pytest.mark.timeout(600)
@pytest.mark.parametrize("w_layout,w_scale", [(0, 1.0), (1, 1.0), (0, 30.0)])
def test_dense_deep_token_contraction_of_dW(spo, oracle, w_layout, w_scale, one_call):
    # The head gradient contracts over tokens.  Here nothing is masked, so every chunk of 16384
    # tokens is one launch with 256 steps of the contraction, and the three chunks add into the
    # same fp32 d_W (read-modify-write across launches), as in the benchmark configuration.
    # Every entry of d_W and d_hidden is compared with the oracle; the softmax part of d_W
    # (d_W minus the rank-one terms of the sampled tokens) is compared on its own, because with
    # flat logits it hides inside the total; w_scale = 30 makes it as large as the target part.
    say(f"fused bf16 deep T=40000 H=320 V=1100 chunk=16384 w_layout={w_layout} w_scale={w_scale} one_call={one_call}")
    case = Case(DEEP, DEEP_LENGTHS, w_scale=w_scale)
    assert case.T == 40000 and case.mask is None
    case.set_old_from_oracle(oracle)
    fwd, dx, dw = run_fwd_bwd(spo, case, w_layout, chunk_tokens=16384, one_call=one_call)
    ref = check_forward(case, oracle, fwd)
    assert ref["active"].sum() > 2 * 16384                   # three chunks of active tokens
    rb = oracle.pg_loss_bwd(*case.oracle_inputs(), *case.eps)
    got_dw, got_dx = f64(dw), f64(dx)
    assert rel_l2(got_dx, rb["d_hidden"]) < GRAD_TOL and rel_l2(got_dw, rb["d_W"]) < GRAD_TOL
    scale = np.abs(rb["d_W"]).max()
    np.testing.assert_allclose(got_dw, rb["d_W"], atol=2e-2 * scale, rtol=0)
    rows = np.linalg.norm(got_dw - rb["d_W"], axis=1)        # no vocabulary row hides in the norm
    assert (rows <= 2 * GRAD_TOL * np.linalg.norm(rb["d_W"], axis=1) + 1e-3 * scale).all()
    # softmax part: subtract sum over the tokens that sampled v of g_t h_t
    g, Hd = rb["g"], f64(case.hidden)
    onehot_dw = np.zeros_like(rb["d_W"])
    np.add.at(onehot_dw, case.target, g[:, None] * Hd)
    soft_ref, soft_gpu = rb["d_W"] - onehot_dw, got_dw - onehot_dw
    # bf16 rounding of a target entry of dZ is at most 2^-9 of it, independently per token
    bound = GRAD_TOL * np.linalg.norm(soft_ref) + 1.1 * 2.0 ** -9 * np.linalg.norm(onehot_dw)
    assert np.linalg.norm(soft_gpu - soft_ref) <= bound
    if w_scale > 1.0:
        assert np.linalg.norm(soft_ref) > 0.3 * np.linalg.norm(onehot_dw)
        assert rel_l2(soft_gpu, soft_ref) < 2 * GRAD_TOL
    # the same gradients from one chunk that holds every token: only the order of the fp32 sums differs
    # (of dW over the chunks, of dHidden over the parts a small chunk's vocabulary contraction is cut into)
    _, dx1, dw1 = run_fwd_bwd(spo, case, w_layout, chunk_tokens=0, one_call=one_call)
    assert rel_l2(f64(dx1), got_dx) < 1e-5 and rel_l2(f64(dw1), got_dw) < 1e-4
    _, dx2, dw2 = run_fwd_bwd(spo, case, w_layout, chunk_tokens=16384, one_call=one_call)
    assert torch.equal(dx2, dx) and torch.equal(dw2, dw if w_layout == 0 else dw)   # same call, same bits


@pytest.mark.parametrize("keep,chunk", [(256, 256), (257, 256), (1, 0), (300, 512), (511, 256)])
def test_backward_runs_over_active_tokens_only(spo, oracle, keep, chunk, one_call):
    # A sparse loss mask: the backward gathers the tokens that carry a gradient and works on
    # that list, `keep` of them here, chosen to end exactly on, one past, and far from the
    # boundaries of token tiles and chunks.  Rows of all other tokens must be exact zeros.
    say(f"fused bf16 mid, {keep} unmasked tokens, chunk_tokens={chunk} one_call={one_call}")
    case = Case(MID, MID_LENGTHS)
    case.set_old_from_oracle(oracle)
    rng = np.random.default_rng(keep)
    live = np.sort(rng.choice(case.T, keep, replace=False))
    case.mask = np.zeros(case.T, np.uint8)
    case.mask[live] = 1
    fwd, dx, dw = run_fwd_bwd(spo, case, chunk_tokens=chunk, one_call=one_call)
    check_forward(case, oracle, fwd)
    rb = oracle.pg_loss_bwd(*case.oracle_inputs(), *case.eps)
    assert rel_l2(f64(dx), rb["d_hidden"]) < GRAD_TOL and rel_l2(f64(dw), rb["d_W"]) < GRAD_TOL
    dead = np.setdiff1d(np.arange(case.T), live)
    assert not dx[torch.as_tensor(dead, device="cuda")].any()
    # a clipped token is dropped from the list like a masked one
    zero_rows = np.flatnonzero(~rb["d_hidden"].any(axis=1))
    assert not dx[torch.as_tensor(zero_rows, device="cuda")].any()


@pytest.mark.parametrize("T,V,chunk", [
    (1000, 17900, 0),      # 4 token tiles, all divided by splits (a multiple of 8)
    (2304, 10200, 0),      # 9: eight by token tile, one by splits
    (4700, 3000, 0),       # 19 over 12 vocabulary tiles: more token tiles than splits, splits no multiple of 8
    (8900, 4000, 6144)])   # 35 in pieces of 24 and 11, each with its own splits; the masked ones run on fewer
def test_token_tiles_and_splits_over_the_chip(spo, oracle, T, V, chunk, one_call):
    say(f"fused bf16 T={T} H=64 V={V} chunk={chunk} one_call={one_call}: token tiles x splits")
    case = Case(wl.scaled(MID, name="splits", H=64, V=V), [T // 3, T - T // 3], mask_frac=0.3 if T > 4000 else None)
    case.set_old_from_oracle(oracle)
    fwd, dx, dw = run_fwd_bwd(spo, case, chunk_tokens=chunk, one_call=one_call)
    check_forward(case, oracle, fwd)
    rb = oracle.pg_loss_bwd(*case.oracle_inputs(), *case.eps)
    assert rel_l2(f64(dx), rb["d_hidden"]) < GRAD_TOL and rel_l2(f64(dw), rb["d_W"]) < GRAD_TOL
    per_row = np.linalg.norm(f64(dx) - rb["d_hidden"], axis=1)
    assert (per_row <= 2 * GRAD_TOL * np.linalg.norm(rb["d_hidden"], axis=1) + 1e-12).all()


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("w_layout", [0, 1])
@pytest.mark.parametrize("T,H,V,mask_frac", [
    (1, 64, 1, None), (3, 64, 63, None),          # less than a tile of the head
    (257, 128, 1032, None),                       # a head of whole tiles and one vector, rows on 16-byte boundaries
    (300, 64, 1001, 0.3),                         # rows off 16-byte boundaries
    (4096, 64, 320, 0.2), (4097, 64, 320, 0.2)])  # most tokens whose factors are formed beside the head, and the next
def test_inputs_prepared_in_one_launch(spo, oracle, dtype, w_layout, T, H, V, mask_frac, one_call):
    say(f"prepared inputs {dtype} T={T} H={H} V={V} layout={w_layout} mask={mask_frac} one_call={one_call}")
    case = Case(wl.scaled(MID, name="prep", H=H, V=V, dtype=dtype), [T] if T < 3 else [T // 3, T - T // 3], mask_frac=mask_frac)
    case.set_old_from_oracle(oracle)
    fwd, dx, dw = run_fwd_bwd(spo, case, w_layout=w_layout, one_call=one_call)
    check_forward(case, oracle, fwd)
    rb = oracle.pg_loss_bwd(*case.oracle_inputs(), *case.eps)
    # a vocabulary of one: the softmax is 1 and every gradient 0, in fp32 up to the rounding of one exponential
    tol = lambda ref: GRAD_TOL * np.linalg.norm(ref) + (1e-5 if V == 1 else 0.0)
    assert np.linalg.norm(f64(dx) - rb["d_hidden"]) <= tol(rb["d_hidden"])
    assert np.linalg.norm(f64(dw) - rb["d_W"]) <= tol(rb["d_W"])


@pytest.mark.parametrize("w_layout", [0, 1])
@pytest.mark.parametrize("T,H,V", [
    (440, 1344, 2500),     # 10 x 6 tiles of d_W: bands of 4, 4, 2 tile rows, patches 6 wide; 7 steps: not cut
    (700, 1344, 2500),     # the same, cut into parts
    (300, 2368, 8000)])    # 32 x 10: a round of the chip and 64 tiles, patches 8 and 2 wide
def test_every_tile_of_dW_is_written(spo, oracle, T, H, V, w_layout, one_call):
    say(f"tiles of d_W, T={T} H={H} V={V} layout={w_layout} one_call={one_call}")
    case = Case(wl.scaled(MID, name="tiles", H=H, V=V), [T // 3, T - T // 3])
    case.set_old_from_oracle(oracle)
    desc = case.to_gpu(spo, w_layout)
    dw = torch.full((V, H) if w_layout == 0 else (H, V), float("nan"), device="cuda")
    if one_call:
        dx = spo.spo_pg_loss_fwd_bwd(desc, 1.0, d_hidden_dtype=torch.float32, d_W=dw)[4]
    else:
        _, logp, lse, _ = spo.spo_pg_loss_fwd(desc)
        dx, _ = spo.spo_pg_loss_bwd(desc, logp, lse, 1.0, d_hidden_dtype=torch.float32, d_W=dw)
    torch.cuda.synchronize()
    rb = oracle.pg_loss_bwd(*case.oracle_inputs(), *case.eps)
    got = f64(dw.t() if w_layout else dw)
    np.testing.assert_allclose(got, rb["d_W"], atol=2e-2 * np.abs(rb["d_W"]).max(), rtol=0)
    assert rel_l2(got, rb["d_W"]) < GRAD_TOL and rel_l2(f64(dx), rb["d_hidden"]) < GRAD_TOL


@pytest.mark.parametrize("T,H,V,mask_frac", [
    (20, 64, 20000, None),     # 1 tile of d_hidden, 313 steps: 19 parts, the last ones shorter or empty
    (290, 448, 16500, 0.2),    # 4 tiles, 258 steps: 16 parts
    (700, 4096, 8300, None)])  # 48 tiles: five parts, what the chip has room for
def test_dHidden_in_parts_along_the_vocabulary(spo, oracle, T, H, V, mask_frac, one_call):
    say(f"parts of d_hidden, T={T} H={H} V={V} mask={mask_frac} one_call={one_call}")
    case = Case(wl.scaled(MID, name="parts", H=H, V=V), [T // 3, T - T // 3], mask_frac=mask_frac)
    case.set_old_from_oracle(oracle)
    fwd, dx, dw = run_fwd_bwd(spo, case, one_call=one_call)
    rb = oracle.pg_loss_bwd(*case.oracle_inputs(), *case.eps)
    got, scale = f64(dx), np.linalg.norm(rb["d_hidden"], axis=1)
    assert rel_l2(got, rb["d_hidden"]) < GRAD_TOL and rel_l2(f64(dw), rb["d_W"]) < GRAD_TOL
    assert (np.linalg.norm(got - rb["d_hidden"], axis=1) <= 2 * GRAD_TOL * scale + 1e-12).all()
    assert not got[scale == 0].any()


@pytest.mark.parametrize("w_layout", [0, 1])
@pytest.mark.parametrize("T,H,V,chunk", [
    (300, 64, 1001, 0), (700, 1344, 2500, 0),    # one chunk: rounded as it is stored, rows off 8-byte boundaries; cut tiles
    (700, 64, 1001, 256)])                       # three chunks: summed in fp32 first
def test_bf16_dW_is_the_fp32_one_rounded(spo, oracle, T, H, V, chunk, w_layout, one_call):
    say(f"bf16 d_W, T={T} H={H} V={V} chunk={chunk} layout={w_layout} one_call={one_call}")
    case = Case(wl.scaled(MID, name="dw16", H=H, V=V), [T // 3, T - T // 3], mask_frac=0.2)
    case.set_old_from_oracle(oracle)
    _, _, dw32 = run_fwd_bwd(spo, case, w_layout, chunk_tokens=chunk, one_call=one_call)
    _, _, dw16 = run_fwd_bwd(spo, case, w_layout, chunk_tokens=chunk, one_call=one_call, dw_dtype=torch.bfloat16)
    assert torch.equal(dw16, dw32.to(torch.bfloat16))
    rb = oracle.pg_loss_bwd(*case.oracle_inputs(), *case.eps)
    assert rel_l2(f64(dw16), rb["d_W"]) < GRAD_TOL


def torch_reference(case):
    """Loss, log-probs and gradients in fp64 by torch's autograd, on the GPU (shapes that take the oracle minutes)."""
    d = "cuda"
    h, w = case.hidden.to(d, torch.float64).requires_grad_(), case.W.to(d, torch.float64).requires_grad_()
    y = torch.as_tensor(case.target).to(d).long()
    old = torch.as_tensor(case.old).to(d, torch.float64)
    m = torch.ones(case.T, dtype=torch.float64, device=d) if case.mask is None else torch.as_tensor(case.mask).to(d, torch.float64)
    adv = torch.repeat_interleave(torch.as_tensor(case.adv).to(d, torch.float64), torch.as_tensor(np.diff(case.cu)).to(d))
    logp = torch.log_softmax(h @ w.t(), dim=1).gather(1, y[:, None])[:, 0]
    ratio = torch.exp(logp - old)
    obj = torch.minimum(ratio * adv, ratio.clamp(1 - case.eps[0], 1 + case.eps[1]) * adv)
    loss = -(m * obj).sum() / m.sum()
    loss.backward()
    return loss.item(), logp.detach(), h.grad, w.grad


@pytest.mark.parametrize("T,H,V", [
    (1000, 2112, 20008),   # large tiles in all contractions: 4 x 79 tiles of logits, 8.25 across d_hidden
    (2300, 2112, 12003),   # the same, rows of a head [H,V] that start anywhere: copied
    (900, 2048, 8200),     # large tiles for the logits and d_W, small ones for d_hidden
    (700, 4096, 8300)])    # small, large, small
@pytest.mark.parametrize("w_layout", [0, 1])
@pytest.mark.parametrize("mask_frac", [None, 0.2], ids=["no_mask", "masked"])
def test_tiles_of_both_sizes(spo, T, H, V, w_layout, mask_frac, one_call):
    say(f"fused bf16 T={T} H={H} V={V} layout={w_layout} mask={mask_frac} one_call={one_call}: large and small tiles")
    case = Case(wl.scaled(MID, name="both", H=H, V=V), [T // 3, T - T // 3], mask_frac=mask_frac)
    case.old = np.zeros(T, np.float32)
    logp = torch_reference(case)[1].cpu().numpy()
    case.old = (logp + case.noise).astype(np.float32)
    for _ in range(3):  # no ratio near a clip bound
        r = np.exp(logp - case.old)
        case.old[(np.abs(r / (1 - case.eps[0]) - 1) < 2e-3) | (np.abs(r / (1 + case.eps[1]) - 1) < 2e-3)] += np.float32(0.01)
    loss, logp, gx, gw = torch_reference(case)
    fwd, dx, dw = run_fwd_bwd(spo, case, w_layout, one_call=one_call)
    assert abs(fwd[0].item() - loss) <= 2e-3 * abs(loss) + 1e-7
    assert (fwd[1].double() - logp).abs().max() < 2e-4
    for got, ref in ((dx, gx), (dw, gw)):
        assert float((got.double() - ref).norm() / ref.norm()) < GRAD_TOL
        assert float((got.double() - ref).abs().max()) <= 2e-2 * float(ref.abs().max())


@pytest.mark.parametrize("H", [384, 448])  # logits of the active tokens formed twice; stored and turned into gradients
@pytest.mark.parametrize("T,chunk", [(713, 0), (2600, 1024)])
@pytest.mark.parametrize("w_layout", [0, 1])
def test_masked_batches_with_and_without_stored_logits(spo, T, H, chunk, w_layout):
    say(f"fused bf16 T={T} H={H} V=3000 layout={w_layout} chunk={chunk}: logits of a masked batch")
    case = Case(wl.scaled(MID, name="again", H=H, V=3000), [T // 3, T - T // 3], mask_frac=0.2)
    case.old = np.zeros(T, np.float32)
    case.old = (torch_reference(case)[1].cpu().numpy() + 0.1 * case.noise).astype(np.float32)  # no ratio near a clip bound
    loss, logp, gx, gw = torch_reference(case)
    fwd, dx, dw = run_fwd_bwd(spo, case, w_layout, one_call=True, chunk_tokens=chunk)
    assert abs(fwd[0].item() - loss) <= 2e-3 * abs(loss) + 1e-7
    assert (fwd[1].double() - logp).abs().max() < 2e-4
    for got, ref in ((dx, gx), (dw, gw)):
        assert float((got.double() - ref).norm() / ref.norm()) < GRAD_TOL
        assert float((got.double() - ref).abs().max()) <= 2e-2 * float(ref.abs().max())


@pytest.mark.parametrize("T,H,V,dtype,mask_frac", [
    (1000, 64, 17904, "bf16", None),    # small tiles, a contraction of one step: three tiles per workgroup
    (1000, 128, 17904, "bf16", None),   # of two steps
    (300, 448, 33000, "bf16", 0.2),     # logits stored from small tiles, two of them per workgroup
    (300, 64, 40000, "fp32", 0.2),      # the same, six steps of a split contraction
    (713, 128, 40000, "bf16", None),    # large tiles, two steps, two tiles
    (1000, 512, 60000, "bf16", 0.2)])   # logits stored from large tiles, several of them
@pytest.mark.parametrize("w_layout", [0, 1])
def test_runs_of_tiles_that_are_stored(spo, T, H, V, dtype, mask_frac, w_layout):
    # the next tile's operands are requested in the last step of a tile, whose stores are still on their way then
    say(f"one call, {dtype} T={T} H={H} V={V} mask={mask_frac} layout={w_layout}: runs of tiles")
    case = Case(wl.scaled(MID, name="runs", H=H, V=V, dtype=dtype), [T // 3, T - T // 3], mask_frac=mask_frac)
    case.old = np.zeros(T, np.float32)
    case.old = (torch_reference(case)[1].cpu().numpy() + 0.1 * case.noise).astype(np.float32)  # no ratio near a clip bound
    loss, logp, gx, gw = torch_reference(case)
    fwd, dx, dw = run_fwd_bwd(spo, case, w_layout, one_call=True)
    assert abs(fwd[0].item() - loss) <= 2e-3 * abs(loss) + 1e-7
    assert (fwd[1].double() - logp).abs().max() < 2e-4
    for got, ref in ((dx, gx), (dw, gw)):
        assert float((got.double() - ref).norm() / ref.norm()) < GRAD_TOL
        assert float((got.double() - ref).abs().max()) <= 2e-2 * float(ref.abs().max())


@pytest.mark.parametrize("T,H,V", [
    (100, 64, 40),          # one stage of 40 entries
    (300, 128, 104),        # two
    (713, 256, 3000),       # small tiles, the vocabulary in parts
    (1000, 2112, 20008),    # large tiles
    (700, 4096, 8307)])     # rows of a head [H,V] that start anywhere: copied
@pytest.mark.parametrize("w_layout", [0, 1])
@pytest.mark.parametrize("mask_frac", [None, 0.2], ids=["no_mask", "masked"])
def test_infinite_weights_stay_in_their_column(spo, T, H, V, w_layout, mask_frac, one_call):
    # A head may ban a token: one feature is 1 everywhere and its weight is -inf.  d_hidden of that feature is then NaN (a
    # probability of 0 times -inf), and so are the banned ids' rows of d_W (rows that pad the batch); all else is what a very
    # large finite weight gives.  The banned ids are those whose weights lie beside what a last stage that is not whole
    # reads in place of entries past the vocabulary.
    say(f"fused bf16 T={T} H={H} V={V} layout={w_layout} mask={mask_frac} one_call={one_call}: infinite weights")
    case = Case(wl.scaled(MID, name="ban", H=H, V=V), [T // 3, T - T // 3], mask_frac=mask_frac)
    feature, banned = H - 1, [0, V - 1]
    case.hidden[:, feature] = 1.0
    case.target[:] = 1 + case.target % (V - 2)
    case.W[banned] = 0.0
    case.old = np.zeros(T, np.float32)
    case.W[banned, feature] = -3e38
    case.old = (torch_reference(case)[1].cpu().numpy() + 0.1 * case.noise).astype(np.float32)
    res = []
    for ban in (-3e38, -np.inf):
        case.W[banned, feature] = ban
        res.append(run_fwd_bwd(spo, case, w_layout, one_call=one_call))
    (fwd, dx, dw), (fwd_inf, dx_inf, dw_inf) = res
    assert all(torch.equal(a, b) for a, b in zip(fwd, fwd_inf)) and torch.equal(dw[1:V - 1], dw_inf[1:V - 1])
    assert torch.isfinite(dx).all() and torch.equal(dx[:, :feature], dx_inf[:, :feature])


@pytest.mark.parametrize("T,H,V,mask_frac", [(512, 128, 1000, None), (713, 256, 3000, 0.25)])
def test_workspaces_down_to_what_large_tiles_need(spo, oracle, T, H, V, mask_frac):
    # small tiles have more partial results; a workspace without that room is served by large ones
    say(f"fused bf16 T={T} H={H} V={V} mask={mask_frac}: smallest workspaces")
    case = Case(wl.scaled(MID, name="room", H=H, V=V), [T // 3, T - T // 3], mask_frac=mask_frac)
    case.set_old_from_oracle(oracle)
    desc = case.to_gpu(spo)
    import ctypes
    L, d = spo.lib(), desc[0]
    buf = torch.empty(L.spo_pg_loss_fwd_bwd_workspace_bytes(ctypes.byref(d), 0), dtype=torch.uint8, device="cuda")
    f = lambda n: torch.empty(n, dtype=torch.float32, device="cuda")
    out = [f(1), f(T), f(T), f(4)]
    dx, dw = f(T * H), f(V * H)
    def fwd(n):
        return L.spo_pg_loss_fwd(ctypes.byref(d), *[o.data_ptr() for o in out], buf.data_ptr(), n, None)
    def both(n):
        return L.spo_pg_loss_fwd_bwd(ctypes.byref(d), 1.0, *[o.data_ptr() for o in out], dx.data_ptr(), 0, dw.data_ptr(), 0, 0, 0,
                                     buf.data_ptr(), n, None)
    for call, size in ((fwd, L.spo_pg_loss_fwd_workspace_bytes(ctypes.byref(d))), (both, buf.numel())):
        assert call(size) == 0
        torch.cuda.synchronize()
        want = [t.clone() for t in (*out, dx, dw)] if call is both else [t.clone() for t in out]
        lo, hi = 0, size    # refused, accepted
        while hi - lo > 256:
            mid = (lo + hi) // 512 * 256
            if call(mid) == 0:
                hi = mid
            else:
                lo = mid
        assert hi < size and call(hi) == 0
        torch.cuda.synchronize()
        for a, b in zip(want, (*out, dx, dw)):
            assert float((a - b).norm()) <= 1e-3 * float(a.norm()) + 1e-9


@pytest.mark.parametrize("V", [1, 3, 6, 257, 510, 1003])   # rows of d_W [H,V] that end inside a run of 4 or 8 columns
@pytest.mark.parametrize("H", [64, 320])                    # a tile with a quarter of its rows; one and a quarter
def test_dW_rows_that_end_anywhere(spo, oracle, V, H):
    # the same sums in either layout of the head (rows of H values are whole runs): stored as fp32, as bf16, and added
    # to.  Sums in fp32 in the same order: equal up to the last place of the largest (2^-23 of it, and of a product).
    T = 90
    say(f"fused bf16 T={T} H={H} V={V}: ends of d_W's rows")
    case = Case(wl.scaled(MID, name="ends", H=H, V=V), [T // 3, T - T // 3])
    case.set_old_from_oracle(oracle)
    _, _, ref = run_fwd_bwd(spo, case, 0)
    tol = 4 * 2.0 ** -23 * float(ref.abs().max()) + 1e-30
    _, _, got = run_fwd_bwd(spo, case, 1)
    assert (got - ref).abs().max() <= tol
    _, _, got16 = run_fwd_bwd(spo, case, 1, dw_dtype=torch.bfloat16)
    assert torch.equal(got16, got.to(torch.bfloat16))
    # guards before and behind the array
    buf = torch.full((H * V + 9,), 7.0, dtype=torch.float32, device="cuda")
    dw = buf[4:4 + H * V].view(H, V)
    desc = case.to_gpu(spo, 1)
    _, logp, lse, _ = spo.spo_pg_loss_fwd(desc)
    spo.spo_pg_loss_bwd(desc, logp, lse, 1.0, d_W=dw, accumulate_dW=True)
    torch.cuda.synchronize()
    assert bool((buf[:4] == 7.0).all()) and bool((buf[4 + H * V:] == 7.0).all())
    assert (dw - (got.t() + 7.0)).abs().max() <= 8 * 2.0 ** -23 * 7.0 + tol


def test_cu_seqlens_may_start_anywhere(spo, oracle):
    # a mini-batch cut out of a packed batch keeps the batch's offsets: only differences count
    say("fused bf16 mid, cu_seqlens shifted by a constant")
    case = Case(MID, MID_LENGTHS, mask_frac=0.25)
    case.set_old_from_oracle(oracle)
    a = run_fwd_bwd(spo, case)
    case.cu = (case.cu.astype(np.int64) + 123456).astype(np.int32)
    b = run_fwd_bwd(spo, case)
    assert torch.equal(a[0][0], b[0][0]) and torch.equal(a[0][1], b[0][1])
    assert torch.equal(a[1], b[1]) and torch.equal(a[2], b[2])


def test_results_are_bitwise_reproducible(spo, oracle, one_call):
    say(f"fused bf16 mid, determinism, one_call={one_call}")
    case = Case(MID, MID_LENGTHS)
    case.set_old_from_oracle(oracle)
    a = run_fwd_bwd(spo, case, chunk_tokens=256, one_call=one_call)
    b = run_fwd_bwd(spo, case, chunk_tokens=256, one_call=one_call)
    assert torch.equal(a[0][0], b[0][0]) and torch.equal(a[0][1], b[0][1])
    assert torch.equal(a[1], b[1]) and torch.equal(a[2], b[2])


def test_mini_batches_accumulate_into_dW(spo, oracle, one_call):
    # two mini-batches of whole responses, the batch-wide normalised advantages,
    # gradients accumulated into one d_W (one optimiser step per mini-batch is the
    # caller's business; the kernel only has to add)
    say(f"fused bf16 mid, two mini-batches, accumulate_dW, one_call={one_call}")
    case = Case(MID, MID_LENGTHS)
    case.set_old_from_oracle(oracle)
    h, w, tg, old, mk, ad, cu = case.oracle_inputs()
    d = "cuda"
    hidden, W = case.hidden.to(d), case.W.to(d)
    target = torch.as_tensor(case.target).to(d)
    oldg = torch.as_tensor(case.old).to(d)
    adv = torch.as_tensor(case.adv).to(d)
    cug = torch.as_tensor(case.cu).to(d)
    dW = torch.zeros_like(W, dtype=torch.float32)
    ref_dw = np.zeros_like(w)
    for (b0, b1) in ((0, 2), (2, 5)):
        t0, t1 = int(cu[b0]), int(cu[b1])
        desc = spo.make_desc(hidden[t0:t1], W, target[t0:t1], oldg[t0:t1], None, adv[b0:b1],
                             cug[b0:b1 + 1], *case.eps)
        if one_call:
            loss, _, _, _, dx, _ = spo.spo_pg_loss_fwd_bwd(desc, 1.0, d_hidden_dtype=torch.float32, d_W=dW,
                                                           accumulate_dW=True)
        else:
            loss, logp, lse, _ = spo.spo_pg_loss_fwd(desc)
            dx, _ = spo.spo_pg_loss_bwd(desc, logp, lse, 1.0, d_hidden_dtype=torch.float32, d_W=dW,
                                        accumulate_dW=True)
        torch.cuda.synchronize()
        sub_cu = (cu[b0:b1 + 1] - cu[b0]).astype(np.int32)
        rf = oracle.pg_loss_fwd(h[t0:t1], w, tg[t0:t1], old[t0:t1], None, ad[b0:b1], sub_cu, *case.eps)
        rb = oracle.pg_loss_bwd(h[t0:t1], w, tg[t0:t1], old[t0:t1], None, ad[b0:b1], sub_cu, *case.eps)
        assert abs(loss.item() - rf["loss"]) <= 2e-3 * abs(rf["loss"]) + 1e-7
        assert rel_l2(f64(dx), rb["d_hidden"]) < GRAD_TOL
        ref_dw += rb["d_W"]
    assert rel_l2(f64(dW), ref_dw) < GRAD_TOL


def test_degenerate_inputs(spo, oracle, one_call):
    say(f"fused: all tokens masked, one_call={one_call}")
    case = Case(MID, [40, 60], mask_frac=0.5)
    case.set_old_from_oracle(oracle)
    case.mask = np.zeros(case.T, np.uint8)
    fwd, dx, dw = run_fwd_bwd(spo, case, one_call=one_call)
    assert fwd[0].item() == 0.0 and not dx.any() and not dw.any()
    ref = oracle.pg_loss_fwd(*case.oracle_inputs(), *case.eps)
    np.testing.assert_allclose(f64(fwd[1]), ref["logp"], atol=2e-4)     # log-probs are still produced
    say("fused: one token, vocabulary smaller than a tile")
    tiny = wl.scaled(MID, name="tiny", H=64, V=100)
    case = Case(tiny, [1], adv=[1.5])
    case.set_old_from_oracle(oracle)
    fwd, dx, dw = run_fwd_bwd(spo, case, one_call=one_call)
    check_forward(case, oracle, fwd)
    rb = oracle.pg_loss_bwd(*case.oracle_inputs(), *case.eps)
    assert rel_l2(f64(dx), rb["d_hidden"]) < GRAD_TOL and rel_l2(f64(dw), rb["d_W"]) < GRAD_TOL
    say("fused: empty responses inside the batch")
    case = Case(MID, [0, 70, 0, 0, 33, 0])
    case.set_old_from_oracle(oracle)
    fwd, dx, dw = run_fwd_bwd(spo, case, one_call=one_call)
    check_forward(case, oracle, fwd)
    rb = oracle.pg_loss_bwd(*case.oracle_inputs(), *case.eps)
    assert rel_l2(f64(dx), rb["d_hidden"]) < GRAD_TOL and rel_l2(f64(dw), rb["d_W"]) < GRAD_TOL
    say("fused: no tokens at all")
    case = Case(MID, [0, 0])
    case.old = np.zeros(0, np.float32)
    desc = case.to_gpu(spo)
    dW = torch.full((MID.V, MID.H), 7.0, device="cuda")
    if one_call:
        loss, logp, lse, stats, _, _ = spo.spo_pg_loss_fwd_bwd(desc, 1.0, d_W=dW, want_d_hidden=False)
    else:
        loss, logp, lse, stats = spo.spo_pg_loss_fwd(desc)
        spo.spo_pg_loss_bwd(desc, logp, lse, 1.0, d_W=dW, want_d_hidden=False)
    torch.cuda.synchronize()
    assert loss.item() == 0.0 and stats[0].item() == 0.0 and not dW.any()


@pytest.mark.parametrize("dtype,V", [("bf16", 3000), ("bf16", 1001), ("fp32", 3000), ("fp32", 1001)])
def test_logits_in_matches_oracle(spo, oracle, dtype, V):
    say(f"logits-in {dtype} T=713 V={V}")
    cfg = wl.scaled(MID, V=V, dtype=dtype)
    case = Case(cfg, MID_LENGTHS, mask_frac=0.25)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    # the logits a model would hand over, rounded to the storage type: they are the input
    logits = (case.hidden.float() @ case.W.float().t() * 4.0).to(tdt)
    lg64 = f64(logits)
    h, w, tg, _, mk, ad, cu = case.oracle_inputs()
    logp = oracle.pg_loss_fwd(None, None, tg, np.zeros(case.T), mk, ad, cu, *case.eps, logits=lg64)["logp"]
    old = (logp + case.noise).astype(np.float32)
    ratio = np.exp(logp - old)
    near = (np.abs(ratio - 0.8) < 2e-3) | (np.abs(ratio - 1.28) < 3e-3)
    old[near] += np.float32(0.01)
    case.old = old
    ref = oracle.pg_loss_fwd(None, None, tg, old.astype(np.float64), mk, ad, cu, *case.eps, logits=lg64)
    rb = oracle.pg_loss_bwd(None, None, tg, old.astype(np.float64), mk, ad, cu, *case.eps, logits=lg64)
    desc = case.to_gpu(spo, logits=logits.cuda())
    fwd = spo.spo_pg_loss_fwd(desc)
    dl = spo.spo_pg_loss_bwd(desc, fwd[1], fwd[2], 1.0)
    torch.cuda.synchronize()
    check_forward(case, oracle, fwd, ref=ref, atol_logp=2e-5 if dtype == "fp32" else 2e-4,
                  rtol_loss=2e-3)
    assert rel_l2(f64(dl), rb["d_logits"]) < (1e-5 if dtype == "fp32" else GRAD_TOL)
    assert not dl[torch.as_tensor(case.mask == 0)].any()


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("T,V,offset", [
    (5, 1, 0), (5, 7, 0), (9, 9, 3),              # rows shorter than one 16-byte vector, or just longer
    (7, 1024, 0), (7, 1025, 0), (6, 4097, 1),     # a row to a wavefront, and the first rows past that
    (3, 16384, 0), (3, 33001, 5),                 # segments of one round, whole and ragged, and rows off a 16-byte boundary
    (2100, 2055, 1)])                             # enough rows for two rounds per segment
def test_logits_in_row_edges(spo, oracle, dtype, T, V, offset):
    say(f"logits-in {dtype} T={T} V={V} offset={offset}")
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator().manual_seed(T * 131 + V)
    logits = (torch.randn((T, V), generator=g) * 3.0).to(tdt)
    rng = np.random.default_rng([T, V])
    tg = rng.integers(0, V, T).astype(np.int32)
    adv = np.array([0.7, -1.3], np.float32)
    cu = np.array([0, T // 2, T], np.int32)
    lg64 = f64(logits)
    logp = oracle.pg_loss_fwd(None, None, tg, np.zeros(T), None, adv.astype(np.float64), cu, 0.2, 0.28, logits=lg64)["logp"]
    old = (logp + rng.choice([-0.1, 0.1, 0.5], T)).astype(np.float32)     # ratios 1.105, 0.905, 0.61: off the bounds
    ref = oracle.pg_loss_fwd(None, None, tg, old.astype(np.float64), None, adv.astype(np.float64), cu, 0.2, 0.28, logits=lg64)
    rb = oracle.pg_loss_bwd(None, None, tg, old.astype(np.float64), None, adv.astype(np.float64), cu, 0.2, 0.28, logits=lg64)
    buf = torch.zeros(T * V + offset, dtype=tdt, device="cuda")
    buf[offset:] = logits.cuda().flatten()
    t = lambda x: torch.as_tensor(x).cuda()
    desc = spo.make_desc(None, None, t(tg), t(old), None, t(adv), t(cu), 0.2, 0.28, logits=buf[offset:].view(T, V))
    loss, lp, lse, _ = spo.spo_pg_loss_fwd(desc)
    dl = spo.spo_pg_loss_bwd(desc, lp, lse, 1.0)
    torch.cuda.synchronize()
    # fp32 sums of at most 33001 exponentials: a few 1e-7 relative
    np.testing.assert_allclose(f64(lse), ref["lse"], atol=1e-5, rtol=0)
    np.testing.assert_allclose(f64(lp), ref["logp"], atol=1e-5, rtol=0)
    assert abs(loss.item() - ref["loss"]) <= 1e-5
    if V > 1:   # entry by entry: one rounding to the storage type (bf16: 2^-9), differences near zero against the row's scale
        scale = np.abs(rb["d_logits"]) + 1e-3 * np.abs(rb["d_logits"]).max(axis=1, keepdims=True)
        assert (np.abs(f64(dl) - rb["d_logits"]) <= (2e-4 if dtype == "fp32" else 5e-3) * scale).all()


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("T,V,offset", [
    (2100, 2560, 0), (2100, 2561, 1), (2100, 5120, 3), (2100, 5121, 0),   # longest rows of single wavefronts, and the next
    (2100, 8192, 0), (2100, 8193, 1),             # a workgroup's row in one round, and in two
    (1100, 16392, 1),                             # halves of a row
    (59000, 2300, 0)])                            # wavefronts' rows that no cache holds
def test_logits_in_segments(spo, oracle, dtype, T, V, offset):
    test_logits_in_row_edges(spo, oracle, dtype, T, V, offset)


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("T,V", [(9, 7), (9, 1000), (9, 1001), (9, 6001), (2100, 8193), (9, 33001)])
def test_logits_far_from_zero(spo, dtype, T, V):
    # rows masked throughout with a large finite value, alone or but for one entry, and rows far off zero: the
    # log-sum-exp is that of the differences, to the rounding of the row's largest logit
    say(f"logits far from zero {dtype} T={T} V={V}")
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    rng = np.random.default_rng([T, V])
    z = rng.standard_normal((T, V)) * 3
    z[0], z[1], z[2], z[3] = -9.9e29, -9.9e29, -1e9, -1e9   # (what lies below -1e30 counts as -inf)
    z[1, V // 2] = 2.0
    z[3, V - 1] = 1e9
    z[4] += 3e4
    z[5] -= 1e5
    z[6, ::2] = -9.9e29
    logits = torch.as_tensor(z, dtype=torch.float32).to(tdt)
    z64 = f64(logits)
    top = z64.max(axis=1)
    want = top + np.log(np.exp(z64 - top[:, None]).sum(axis=1))
    t = lambda x: torch.as_tensor(x).cuda()
    tg = z64.argmax(axis=1).astype(np.int32)
    desc = spo.make_desc(None, None, t(tg), torch.zeros(T, device="cuda"), None, t(np.ones(1, np.float32)),
                         t(np.array([0, T], np.int32)), 0.2, 0.28, logits=logits.cuda())
    _, lp, lse, _ = spo.spo_pg_loss_fwd(desc)
    torch.cuda.synchronize()
    # one rounding of max + log(sum) to fp32, and a few 1e-7 of the sum
    np.testing.assert_allclose(f64(lse), want, rtol=2.0 ** -23, atol=1e-5)
    err = np.abs(f64(lp) - (z64[np.arange(T), tg] - want))
    assert (err <= 2.0 ** -23 * np.abs(want) + 1e-5).all()


@pytest.mark.parametrize("T,B,offset", [
    (63, 3, 0), (64, 3, 1), (65, 1, 15),            # one workgroup of tokens, whole and one more; masks off 16-byte boundaries
    (5000, 1023, 3), (5000, 1024, 0),               # response offsets kept in LDS, and too many for it
    (32768, 5, 7), (32769, 5, 2)])                  # longest mask that every workgroup counts, and the next
def test_token_kernels_edges(spo, oracle, T, B, offset):
    say(f"per-token kernels T={T} B={B} mask offset={offset}")
    V = 8
    rng = np.random.default_rng([T, B])
    logits = (rng.standard_normal((T, V)) * 2).astype(np.float32)
    tg = rng.integers(0, V, T).astype(np.int32)
    adv = rng.standard_normal(B).astype(np.float32)
    cu = np.concatenate([[0], np.sort(rng.integers(0, T + 1, B - 1)), [T]]).astype(np.int32)   # some responses empty
    mask = (rng.random(T) < 0.7).astype(np.uint8)
    o = lambda old: oracle.pg_loss_fwd(None, None, tg, old, mask, adv.astype(np.float64), cu, 0.2, 0.28, logits=logits.astype(np.float64))
    old = (o(np.zeros(T))["logp"] + rng.choice([-0.1, 0.1, 0.5], T)).astype(np.float32)
    ref = o(old.astype(np.float64))
    rb = oracle.pg_loss_bwd(None, None, tg, old.astype(np.float64), mask, adv.astype(np.float64), cu, 0.2, 0.28,
                            logits=logits.astype(np.float64))
    t = lambda x: torch.as_tensor(x).cuda()
    buf = torch.ones(T + offset, dtype=torch.uint8, device="cuda")
    buf[offset:] = t(mask)
    desc = spo.make_desc(None, None, t(tg), t(old), buf[offset:], t(adv), t(cu), 0.2, 0.28, logits=t(logits))
    loss, lp, lse, stats = spo.spo_pg_loss_fwd(desc)
    dl = spo.spo_pg_loss_bwd(desc, lp, lse, 1.0)
    torch.cuda.synchronize()
    np.testing.assert_allclose(f64(lp), ref["logp"], atol=1e-5, rtol=0)
    st = f64(stats)
    m = mask.astype(bool)
    assert st[0] == ref["M"] and abs(st[1] - (1 - ref["active"][m].mean())) < 1e-6 and abs(st[2] - ref["ratio"][m].mean()) < 1e-4
    assert abs(loss.item() - ref["loss"]) <= 1e-5
    assert rel_l2(f64(dl), rb["d_logits"]) < 1e-5 and not dl[t(mask) == 0].any()


@pytest.mark.parametrize("T,V", [
    *[(T, V) for T in (1, 64, 65, 129, 200, 320)   # 1 to 5 blocks of 64 tokens, a workgroup each
      for V in (8, 20000, 60000)],                 # rows in 1, 5 and 15 segments: 1, 2 and 4 wavefronts per block
    (4033, 8), (4225, 20000), (4097, 60000),       # from 64 blocks on 4, 2 and 1 per workgroup, the last one ragged
    (131073, 8), (140000, 8), (262145, 8)])        # 4, 8 and 16 blocks per workgroup
def test_token_blocks_per_workgroup(spo, oracle, T, V):
    say(f"token blocks T={T} V={V}")
    rng = np.random.default_rng([T, V, 6])
    logits = (rng.standard_normal((T, V)) * 2).astype(np.float32)
    tg, adv = rng.integers(0, V, T).astype(np.int32), np.array([0.7, -1.3], np.float32)
    cu, mask = np.array([0, T // 3, T], np.int32), (np.arange(T) % 5 != 1).astype(np.uint8)
    args = lambda old: (None, None, tg, old, mask, adv.astype(np.float64), cu, 0.2, 0.28)
    logp = oracle.pg_loss_fwd(*args(np.zeros(T)), logits=logits.astype(np.float64))["logp"]
    old = (logp + rng.choice([-0.1, 0.1, 0.5], T)).astype(np.float32)
    ref = oracle.pg_loss_fwd(*args(old.astype(np.float64)), logits=logits.astype(np.float64))
    t = lambda x: torch.as_tensor(x).cuda()
    desc = spo.make_desc(None, None, t(tg), t(old), t(mask), t(adv), t(cu), 0.2, 0.28, logits=t(logits))
    for _ in range(2):
        loss, lp, lse, stats = spo.spo_pg_loss_fwd(desc)
        torch.cuda.synchronize()
        np.testing.assert_allclose(f64(lp), ref["logp"], atol=1e-5, rtol=0)
        np.testing.assert_allclose(f64(lse), ref["lse"], atol=1e-5, rtol=0)
        m = mask.astype(bool)
        st = f64(stats)
        assert st[0] == ref["M"] and abs(st[1] - (1 - ref["active"][m].mean())) < 1e-6
        assert abs(st[2] - ref["ratio"][m].mean()) < 1e-4 and abs(loss.item() - ref["loss"]) <= 1e-5


def test_many_tokens_of_few_splits(spo, oracle):
    # 6 splits, and enough blocks of tokens that one wavefront merges all of them, eight blocks per workgroup
    say("fused bf16 T=140001 H=64 V=1500, forward")
    case = Case(wl.scaled(MID, name="long", H=64, V=1500), [40000, 1, 100000])
    case.set_old_from_oracle(oracle)
    fwd = spo.spo_pg_loss_fwd(case.to_gpu(spo, 0))
    torch.cuda.synchronize()
    check_forward(case, oracle, fwd)


@pytest.mark.parametrize("dtype,H", [("bf16", 64), ("bf16", 1024), ("bf16", 1088), ("fp32", 192), ("fp32", 576)])
@pytest.mark.parametrize("T", [16384, 16385, 16387])   # four target logits per wavefront from the second on, where rows are short
def test_target_logits_of_long_batches(spo, oracle, dtype, H, T):
    say(f"target logits {dtype} T={T} H={H}")
    case = Case(wl.scaled(MID, name="targets", H=H, V=40, dtype=dtype), [T - 5, 5])
    case.set_old_from_oracle(oracle)
    desc = case.to_gpu(spo, 0)
    *fwd, dx, dw = spo.spo_pg_loss_fwd_bwd(desc, 1.0, d_hidden_dtype=torch.float32)   # its references are made there too
    torch.cuda.synchronize()
    check_forward(case, oracle, fwd)
    rb = oracle.pg_loss_bwd(*case.oracle_inputs(), *case.eps)
    assert rel_l2(f64(dx), rb["d_hidden"]) < GRAD_TOL and rel_l2(f64(dw), rb["d_W"]) < GRAD_TOL


def test_target_id_out_of_range_gives_nan_not_garbage(spo, oracle):
    # sampled-token ids are not validated on the host; an id outside [0, V) must neither read out of
    # bounds nor leave a stale number behind: the token's log-prob is NaN, all other tokens are untouched
    say("fused and logits-in: one target id outside the vocabulary")
    case = Case(MID, MID_LENGTHS)
    case.set_old_from_oracle(oracle)
    ref = oracle.pg_loss_fwd(*case.oracle_inputs(), *case.eps)
    bad = np.array([5, 300, 712])
    good = np.setdiff1d(np.arange(case.T), bad)
    case.target = case.target.copy()
    case.target[bad] = [MID.V, -1, 2 ** 31 - 1]
    for logits in (None, (case.hidden.float() @ case.W.float().t()).to(torch.bfloat16).cuda()):
        loss, logp, lse, _ = spo.spo_pg_loss_fwd(case.to_gpu(spo, logits=logits))
        torch.cuda.synchronize()
        lp = f64(logp)
        assert np.isnan(lp[bad]).all() and np.isnan(loss.item())
        if logits is None:
            np.testing.assert_allclose(lp[good], ref["logp"][good], atol=2e-4, rtol=0)
            np.testing.assert_allclose(f64(lse), ref["lse"], atol=2e-4, rtol=0)
        else:
            assert np.isfinite(lp[good]).all() and np.isfinite(f64(lse)).all()
