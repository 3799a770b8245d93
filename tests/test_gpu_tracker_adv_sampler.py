"""GPU parity of the tracker update, the advantages and the prioritized sampler
against the fp64 oracle, through the C ABI.  Indices and counts bit-exact,
fp32 values within 1e-5 relative."""
import sys

import numpy as np
import pytest
import torch

from paper_2509_13232_amd import workloads as wl

pytestmark = pytest.mark.gpu
RTOL = 1e-5


def say(msg):
    print("[case]", msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def spo():
    from paper_2509_13232_amd import binding
    binding.lib()
    assert torch.cuda.is_available()
    return binding


def dev(x, dtype=None):
    t = torch.as_tensor(np.asarray(x))
    if dtype is not None:
        t = t.to(dtype)
    return t.cuda().contiguous()


def _update_case(cfg, n, seed, unique=True):
    a, b = wl.tracker_state(cfg, seed)
    if unique:
        idx = wl.distinct_indices(cfg, n, seed)
    else:
        idx = np.random.default_rng(seed).integers(0, min(cfg.N, max(2, n // 4)), n).astype(np.int32)
    r = wl.rewards(cfg, idx, seed)
    kl = wl.kl_divergences(cfg, n, seed)
    return a, b, idx, r, kl


@pytest.mark.parametrize("name,n", [("C1", 8), ("C2", 64), ("C5", 4096)])
def test_tracker_update_matches_oracle(spo, oracle, name, n):
    cfg = wl.CONFIGS[name]
    say(f"tracker_update {name} n={n}")
    a, b, idx, r, kl = _update_case(cfg, n, 11)
    ea, eb, ev, _ = oracle.tracker_update(a, b, idx, r, kl, cfg.d_half, cfg.rho_min, cfg.rho_max)
    ga, gb = dev(a), dev(b)
    nobs = torch.zeros(cfg.N, dtype=torch.int32, device="cuda")
    gv = spo.spo_tracker_update(ga, gb, dev(idx), dev(r), dev(kl), cfg.d_half, cfg.rho_min, cfg.rho_max,
                                ids_unique=True, n_obs=nobs, want_v_prev=True)
    torch.cuda.synchronize()
    np.testing.assert_allclose(ga.cpu().numpy(), ea, rtol=RTOL)
    np.testing.assert_allclose(gb.cpu().numpy(), eb, rtol=RTOL)
    np.testing.assert_allclose(gv.cpu().numpy(), ev, rtol=RTOL)
    # untouched entries keep their bits, visit counters are exact
    untouched = np.ones(cfg.N, bool)
    untouched[idx] = False
    assert np.array_equal(ga.cpu().numpy()[untouched], a[untouched])
    assert np.array_equal(nobs.cpu().numpy(), np.bincount(idx, minlength=cfg.N))


def test_tracker_counts_are_exact_without_discount(spo, oracle):
    # discount 1: Beta posterior counts, bit for bit, over several iterations
    cfg = wl.CONFIGS["C2"]
    say("tracker_update discount=1 counts")
    a = np.full(cfg.N, 0.5, np.float32)
    b = np.full(cfg.N, 0.5, np.float32)
    ga, gb = dev(a), dev(b)
    ea, eb = a.astype(np.float64), b.astype(np.float64)
    for it in range(6):
        idx = wl.distinct_indices(cfg, 64, 100 + it)
        r = wl.rewards(cfg, idx, 100 + it)
        kl = wl.kl_divergences(cfg, 64, 100 + it)
        ea, eb, _, _ = oracle.tracker_update(ea, eb, idx, r, kl, cfg.d_half, 1.0, 1.0)
        spo.spo_tracker_update(ga, gb, dev(idx), dev(r), dev(kl), cfg.d_half, 1.0, 1.0)
    torch.cuda.synchronize()
    assert np.array_equal(ga.cpu().numpy().astype(np.float64), ea)
    assert np.array_equal(gb.cpu().numpy().astype(np.float64), eb)


def test_tracker_update_with_repeated_ids_is_sequential(spo, oracle):
    cfg = wl.CONFIGS["C2"]
    say("tracker_update repeated ids")
    a, b, idx, r, kl = _update_case(cfg, 300, 5, unique=False)
    assert len(set(idx.tolist())) < 300
    ea, eb, ev, _ = oracle.tracker_update(a, b, idx, r, kl, cfg.d_half, cfg.rho_min, cfg.rho_max)
    ga, gb = dev(a), dev(b)
    nobs = torch.zeros(cfg.N, dtype=torch.int32, device="cuda")
    gv = spo.spo_tracker_update(ga, gb, dev(idx), dev(r), dev(kl), cfg.d_half, cfg.rho_min, cfg.rho_max,
                                ids_unique=False, n_obs=nobs, want_v_prev=True)
    torch.cuda.synchronize()
    np.testing.assert_allclose(ga.cpu().numpy(), ea, rtol=RTOL)
    np.testing.assert_allclose(gb.cpu().numpy(), eb, rtol=RTOL)
    np.testing.assert_allclose(gv.cpu().numpy(), ev, rtol=RTOL)
    assert np.array_equal(nobs.cpu().numpy(), np.bincount(idx, minlength=cfg.N))


@pytest.mark.parametrize("B,G,N", [(16384, 8, 1 << 20), (40000, 3, 20000), (512, 512, 64)])
def test_tracker_update_of_batches_that_repeat_every_prompt(spo, oracle, B, G, N):
    # batch extensions that sample every prompt G times (Appendix "Batch Extensions"): B observations,
    # each id G times in shuffled order; also a batch beyond one window of the kernel (40000) and one
    # id repeated 512 times (as many rounds as observations).  Values 1e-5, visit counters exact, and
    # the slot table the kernel borrows is handed back clean (a second call gives the same answer).
    say(f"tracker_update B={B}, every id {G} times, N={N}")
    rng = np.random.default_rng([B, G])
    B = B // G * G
    ids = rng.choice(N, B // G, replace=False).astype(np.int32)
    idx = rng.permutation(np.repeat(ids, G)).astype(np.int32)
    a = rng.uniform(0.5, 50, N).astype(np.float32)
    b = rng.uniform(0.5, 50, N).astype(np.float32)
    r = (rng.random(B) < 0.4).astype(np.float32)
    kl = rng.exponential(0.02, B).astype(np.float32)
    ea, eb, ev, _ = oracle.tracker_update(a, b, idx, r, kl, 0.25, 0.875, 0.96)
    ws = torch.empty(spo.lib().spo_tracker_update_workspace_bytes(N), dtype=torch.uint8, device="cuda")
    for _ in range(2):
        ga, gb = dev(a), dev(b)
        nobs = torch.zeros(N, dtype=torch.int32, device="cuda")
        info = torch.full((1,), 7, dtype=torch.int32, device="cuda")
        gv = spo.spo_tracker_update(ga, gb, dev(idx), dev(r), dev(kl), 0.25, 0.875, 0.96, ids_unique=False,
                                    n_obs=nobs, want_v_prev=True, info=info, workspace=ws)
        torch.cuda.synchronize()
        np.testing.assert_allclose(ga.cpu().numpy(), ea, rtol=RTOL)
        np.testing.assert_allclose(gb.cpu().numpy(), eb, rtol=RTOL)
        np.testing.assert_allclose(gv.cpu().numpy(), ev, rtol=RTOL)
        assert np.array_equal(nobs.cpu().numpy(), np.bincount(idx, minlength=N))
        assert info.item() == 0


@pytest.mark.parametrize("B,n_ids,bad", [
    (1, 1, 0), (128, 5, 3), (129, 129, 1),          # one workgroup, and one observation more
    (256, 1, 0), (257, 1, 0), (257, 90, 2),         # the longest list sorted by ranks, and one more
    (1024, 1, 0), (1025, 2, 7),                     # one step of the list, and one more
    (4096, 1, 0), (9000, 1, 11),                    # one id fills the list; the list is applied and restarted
    (33000, 7, 100)])                               # a few long runs over many workgroups and restarts
def test_tracker_update_runs_of_one_id(spo, oracle, B, n_ids, bad):
    # an id's observations form a serial chain wherever the list they are collected in ends; ids outside the
    # table (bad of them) are skipped, flagged and get a NaN baseline
    N = 300
    say(f"tracker_update B={B}, {n_ids} ids, {bad} out of range")
    rng = np.random.default_rng([B, n_ids])
    idx = rng.choice(rng.choice(N, n_ids, replace=False), B).astype(np.int32)
    out = rng.choice(B, bad, replace=False)
    idx[out] = rng.choice([-1, N, 2 ** 31 - 1, -2 ** 31], bad)
    ok = np.ones(B, bool)
    ok[out] = False
    a, b = (rng.uniform(0.5, 50, N).astype(np.float32) for _ in range(2))
    r = (rng.random(B) < 0.4).astype(np.float32)
    kl = rng.exponential(0.02, B).astype(np.float32)
    ea, eb, ev, _ = oracle.tracker_update(a, b, idx[ok], r[ok], kl[ok], 0.25, 0.875, 0.96)
    ga, gb = dev(a), dev(b)
    nobs = torch.zeros(N, dtype=torch.int32, device="cuda")
    info = torch.full((1,), 7, dtype=torch.int32, device="cuda")
    gv = spo.spo_tracker_update(ga, gb, dev(idx), dev(r), dev(kl), 0.25, 0.875, 0.96, ids_unique=False, n_obs=nobs,
                                want_v_prev=True, info=info)
    torch.cuda.synchronize()
    # the state is rounded to fp32 after every observation on both sides; a discount forgets old roundings
    np.testing.assert_allclose(ga.cpu().numpy(), ea, rtol=RTOL)
    np.testing.assert_allclose(gb.cpu().numpy(), eb, rtol=RTOL)
    np.testing.assert_allclose(gv.cpu().numpy()[ok], ev, rtol=RTOL)
    assert np.isnan(gv.cpu().numpy()[~ok]).all() and info.item() == (1 if bad else 0)
    assert np.array_equal(nobs.cpu().numpy(), np.bincount(idx[ok], minlength=N))


def test_ids_out_of_range_or_repeated_are_flagged_not_followed(spo, oracle):
    say("tracker_update / advantages: ids outside the table, repeats under ids_unique")
    N, B = 1000, 64
    rng = np.random.default_rng(3)
    a = rng.uniform(0.5, 50, N).astype(np.float32)
    b = rng.uniform(0.5, 50, N).astype(np.float32)
    idx = rng.choice(N, B, replace=False).astype(np.int32)
    r = (rng.random(B) < 0.5).astype(np.float32)
    kl = rng.uniform(0, 0.05, B).astype(np.float32)
    bad = idx.copy()
    bad[[3, 40]] = [N, -1]
    good = np.ones(B, bool)
    good[[3, 40]] = False
    ea, eb, ev, _ = oracle.tracker_update(a, b, idx[good], r[good], kl[good], 0.25, 0.875, 0.96)
    for unique in (True, False):
        ga, gb = dev(a), dev(b)
        info = torch.zeros(1, dtype=torch.int32, device="cuda")
        gv = spo.spo_tracker_update(ga, gb, dev(bad), dev(r), dev(kl), 0.25, 0.875, 0.96, ids_unique=unique,
                                    want_v_prev=True, info=info)
        torch.cuda.synchronize()
        assert info.item() == 1                                            # out of range, nothing else
        np.testing.assert_allclose(ga.cpu().numpy(), ea, rtol=RTOL)       # the other observations are applied
        np.testing.assert_allclose(gb.cpu().numpy(), eb, rtol=RTOL)
        v = gv.cpu().numpy()
        assert np.isnan(v[~good]).all()
        np.testing.assert_allclose(v[good], ev, rtol=RTOL)
    # advantages: the flag, NaN for the response, no read outside the table
    info = torch.zeros(1, dtype=torch.int32, device="cuda")
    raw, nrm, _ = spo.spo_advantages(dev(a), dev(b), dev(bad), dev(r), info=info)
    torch.cuda.synchronize()
    assert info.item() == 1 and np.isnan(raw.cpu().numpy()[~good]).all() and np.isfinite(raw.cpu().numpy()[good]).all()
    assert torch.isnan(nrm).all()                                          # the batch statistics are NaN: nothing is normalised
    raw, nrm, _ = spo.spo_advantages(dev(a), dev(b), dev(idx), dev(r), info=info)
    torch.cuda.synchronize()
    assert info.item() == 0 and np.isfinite(nrm.cpu().numpy()).all()
    # a repeated id under ids_unique = 1 is found when the table is there to look
    rep = idx.copy()
    rep[10] = rep[50]
    info = torch.zeros(1, dtype=torch.int32, device="cuda")
    spo.spo_tracker_update(dev(a), dev(b), dev(rep), dev(r), dev(kl), 0.25, 0.875, 0.96, info=info, check_repeats=True)
    torch.cuda.synchronize()
    assert info.item() == 2
    spo.spo_tracker_update(dev(a), dev(b), dev(idx), dev(r), dev(kl), 0.25, 0.875, 0.96, info=info, check_repeats=True)
    torch.cuda.synchronize()
    assert info.item() == 0


def test_tracker_init(spo, oracle):
    say("tracker_init")
    v0 = (np.random.default_rng(0).integers(0, 9, 1000) / 8.0).astype(np.float32)
    ea, eb = oracle.tracker_init(v0, 0.875)
    ga, gb = spo.spo_tracker_init(dev(v0), 0.875)
    torch.cuda.synchronize()
    assert np.array_equal(ga.cpu().numpy().astype(np.float64), ea)
    assert np.array_equal(gb.cpu().numpy().astype(np.float64), eb)


@pytest.mark.parametrize("name,n", [("C1", 8), ("C2", 64), ("C3", 128), ("C5", 4096)])
@pytest.mark.parametrize("ddof,eps_norm,baseline", [(0, 0.0, True), (1, 1e-6, True), (0, 0.0, False)])
def test_advantages_match_oracle(spo, oracle, name, n, ddof, eps_norm, baseline):
    cfg = wl.CONFIGS[name]
    say(f"advantages {name} n={n} ddof={ddof} eps={eps_norm} baseline={baseline}")
    a, b, idx, r, _ = _update_case(cfg, n, 21)
    eraw, enrm, (mu, sigma) = oracle.advantages(a, b, idx, r, ddof, float(np.float32(eps_norm)), baseline)
    raw, nrm, st = spo.spo_advantages(dev(a), dev(b), dev(idx), dev(r), ddof, eps_norm, baseline)
    torch.cuda.synchronize()
    np.testing.assert_allclose(raw.cpu().numpy(), eraw, rtol=RTOL, atol=1e-7)
    np.testing.assert_allclose(nrm.cpu().numpy(), enrm, rtol=RTOL, atol=1e-6)
    np.testing.assert_allclose(st.cpu().numpy(), [mu, sigma], rtol=RTOL, atol=1e-7)
    # run-to-run bitwise reproducible
    _, nrm2, _ = spo.spo_advantages(dev(a), dev(b), dev(idx), dev(r), ddof, eps_norm, baseline)
    assert torch.equal(nrm, nrm2)


@pytest.mark.parametrize("B", [16384, 100003, 1 << 20])
@pytest.mark.parametrize("ddof,eps_norm,baseline", [(0, 0.0, True), (1, 1e-6, False)])
def test_advantages_of_large_batches_over_many_workgroups(spo, oracle, B, ddof, eps_norm, baseline):
    # with a workspace, batches of 16384 responses or more are spread over the chip: partial sums of
    # 4096 responses, added in a fixed order (a ragged last part at B = 100003); ids repeat
    cfg = wl.CONFIGS["C5"]
    say(f"advantages, wide path, B={B} ddof={ddof} baseline={baseline}")
    a, b = wl.tracker_state(cfg, 5)
    rng = np.random.default_rng([wl.MASTER_SEED, B])
    idx = rng.integers(0, cfg.N, B).astype(np.int32)
    r = (rng.random(B) < 0.4).astype(np.float32)
    eraw, enrm, (mu, sigma) = oracle.advantages(a, b, idx, r, ddof, float(np.float32(eps_norm)), baseline)
    ws = torch.empty(spo.lib().spo_advantages_workspace_bytes(B), dtype=torch.uint8, device="cuda")
    ga, gb, gi, gr = dev(a), dev(b), dev(idx), dev(r)
    info = torch.full((1,), 7, dtype=torch.int32, device="cuda")
    raw, nrm, st = spo.spo_advantages(ga, gb, gi, gr, ddof, eps_norm, baseline, info=info, workspace=ws)
    torch.cuda.synchronize()
    assert info.item() == 0
    np.testing.assert_allclose(raw.cpu().numpy(), eraw, rtol=RTOL, atol=1e-7)
    np.testing.assert_allclose(nrm.cpu().numpy(), enrm, rtol=RTOL, atol=1e-6)
    np.testing.assert_allclose(st.cpu().numpy(), [mu, sigma], rtol=RTOL, atol=1e-7)
    _, nrm2, st2 = spo.spo_advantages(ga, gb, gi, gr, ddof, eps_norm, baseline, workspace=ws)
    assert torch.equal(nrm, nrm2) and torch.equal(st, st2)                  # bitwise reproducible
    _, nrm1, st1 = spo.spo_advantages(ga, gb, gi, gr, ddof, eps_norm, baseline)   # one workgroup: same to fp64 rounding
    torch.cuda.synchronize()
    np.testing.assert_allclose(nrm1.cpu().numpy(), nrm.cpu().numpy(), rtol=1e-6, atol=1e-7)
    if baseline:    # an id out of range is flagged, not followed, here too
        bad = idx.copy()
        bad[B // 2] = cfg.N
        info.zero_()
        raw, nrm, _ = spo.spo_advantages(ga, gb, dev(bad), gr, ddof, eps_norm, baseline, info=info, workspace=ws)
        torch.cuda.synchronize()
        assert info.item() == 1 and torch.isnan(raw[B // 2]) and torch.isnan(nrm).all()


@pytest.mark.parametrize("B", [1, 64, 65, 1024, 1025, 4096, 4097, 16383, 16385])   # responses per thread: 1, 4, 16, any
@pytest.mark.parametrize("beta", [True, False])
def test_advantages_kept_in_registers(spo, oracle, B, beta):
    say(f"advantages in one workgroup, B={B} beta={beta}")
    rng = np.random.default_rng([B, 3])
    N = 5000
    a, b = (rng.uniform(0.5, 50, N).astype(np.float32) for _ in range(2))
    v = a / (a + b) if not beta else None
    idx = rng.integers(0, N, B).astype(np.int32)
    r = (rng.random(B) < 0.4).astype(np.float32)
    base = a.astype(np.float64)[idx] / (a.astype(np.float64) + b.astype(np.float64))[idx] if beta else v.astype(np.float64)[idx]
    raw64 = r.astype(np.float64) - base
    info = torch.full((1,), 7, dtype=torch.int32, device="cuda")
    state = (dev(a), dev(b)) if beta else (dev(v), None)
    raw, nrm, st = spo.spo_advantages(*state, dev(idx), dev(r), info=info)
    diag = spo.spo_advantage_diagnostics(raw, dev(r), 0.1, 0.3)
    torch.cuda.synchronize()
    sd = raw64.std()
    assert info.item() == 0
    np.testing.assert_allclose(raw.cpu().numpy(), raw64, rtol=1e-6, atol=1e-7)
    np.testing.assert_allclose(st.cpu().numpy(), [raw64.mean(), sd], rtol=1e-6, atol=1e-9)
    np.testing.assert_allclose(nrm.cpu().numpy(), (raw64 - raw64.mean()) / sd if sd else 0 * raw64, rtol=1e-5, atol=1e-6)
    raw32 = raw.cpu().numpy().astype(np.float64)
    np.testing.assert_allclose(diag.cpu().numpy(), [(np.abs(raw32) <= np.float32(0.1)).mean(), (np.abs(raw32) <= np.float32(0.3)).mean(),
                                                    raw32.var(), r.var()], rtol=1e-5, atol=1e-9)
    bad = idx.copy()
    bad[B - 1] = -1
    raw, nrm, _ = spo.spo_advantages(*state, dev(bad), dev(r), info=info)
    torch.cuda.synchronize()
    assert info.item() == 1 and torch.isnan(raw[B - 1]) and torch.isnan(nrm).all() and not torch.isnan(raw[:B - 1]).any()


def test_advantages_degenerate_batch(spo):
    say("advantages all-equal")
    a = dev(np.ones(4, np.float32))
    raw, nrm, st = spo.spo_advantages(a, a, dev(np.arange(4, dtype=np.int32)), dev(np.ones(4, np.float32)))
    torch.cuda.synchronize()
    assert nrm.cpu().tolist() == [0.0] * 4 and st.cpu().tolist() == [0.5, 0.0]


@pytest.mark.parametrize("name,B,seed,replace", [
    ("C1", 8, 0, False), ("C1", 16, 3, False), ("C1", 8, 0, True),
    ("C2", 64, 1, False), ("C3", 128, 2, False),
    ("C5", 4096, 7, False), ("C5", 4096, 7, True), ("C5", 16384, 9, False)])
def test_sampler_indices_are_bit_exact(spo, oracle, name, B, seed, replace):
    cfg = wl.CONFIGS[name]
    say(f"sample_prompts {name} B={B} seed={seed} replace={replace}")
    a, b = wl.tracker_state(cfg, 31)
    for it in (0, 5):
        eidx, eatt = oracle.sample_prompts(a, b, B, cfg.eps_explore, seed, it, replace, return_attempts=True)
        gidx, info = spo.spo_sample_prompts(dev(a), dev(b), B, cfg.eps_explore, seed, it, replace,
                                            return_info=True)
        torch.cuda.synchronize()
        assert np.array_equal(gidx.cpu().numpy(), eidx)
        assert info.cpu().tolist() == [0, int(eatt.max())]
        if not replace:
            assert len(set(eidx.tolist())) == B


@pytest.mark.parametrize("N,B,replace", [
    (1, 1, False), (1, 300, True), (64, 64, False), (65, 65, False), (257, 250, False),   # one workgroup of 1, 1, 2, 2 wavefronts
    (4095, 3000, False), (4096, 3500, False), (4096, 4096, True),                          # its largest tables
    (4096, 4097, True), (4097, 3500, False), (8193, 2000, True),                           # tables in memory, two and three blocks
    (16384, 12000, False),                                                                 # long chains of displaced slots
    (4096 * 1024, 500, False), (4096 * 1024 + 1, 500, False)])                             # most blocks that add up sums themselves, one more
def test_sampler_table_sizes(spo, oracle, N, B, replace):
    say(f"sample_prompts N={N} B={B} replace={replace}")
    rng = np.random.default_rng([N, B])
    a, b = (rng.uniform(0.5, 50, N).astype(np.float32) for _ in range(2))
    eidx, eatt = oracle.sample_prompts(a, b, B, 0.05, 3, 1 << 33, replace, return_attempts=True)
    for _ in range(2):
        gidx, info = spo.spo_sample_prompts(dev(a), dev(b), B, 0.05, 3, 1 << 33, replace, return_info=True)
        torch.cuda.synchronize()
        assert np.array_equal(gidx.cpu().numpy(), eidx) and info.cpu().tolist() == [0, int(eatt.max())]


@pytest.mark.parametrize("N,B,nonzero,max_attempts", [
    (5000, 200, 150, 3), (5000, 4000, 3000, 5),          # claims over many workgroups
    (5000, 5000, 4999, 400),                             # long chains, then a few that run out
    (4096, 200, 150, 3), (4096, 4096, 3000, 4),          # a table in LDS
    (300, 300, 299, 20), (64, 64, 1, 7)])
def test_sampler_exhausted_attempts_over_many_workgroups(spo, oracle, N, B, nonzero, max_attempts):
    # all weight on some of the prompts: a slot that finds none of them free within its attempts gets -1 and
    # holds nothing; the others keep what the sequential draw gives them
    say(f"sample_prompts exhausted attempts N={N} B={B} nonzero={nonzero} max_attempts={max_attempts}")
    rng = np.random.default_rng([N, B, nonzero])
    a, b = np.zeros(N, np.float32), np.ones(N, np.float32)
    a[rng.choice(N, nonzero, replace=False)] = rng.uniform(0.1, 3.0, nonzero)
    eidx, eatt = oracle.sample_prompts(a, b, B, 0.0, 4, 2, False, max_attempts=max_attempts, return_attempts=True,
                                       allow_exhausted=True)
    assert (eidx == -1).any() and (eidx >= 0).sum() > nonzero // 3
    for _ in range(2):
        gidx, info = spo.spo_sample_prompts(dev(a), dev(b), B, 0.0, 4, 2, False, max_attempts=max_attempts, return_info=True)
        torch.cuda.synchronize()
        assert np.array_equal(gidx.cpu().numpy(), eidx)
        assert info.cpu().tolist() == [1, int(eatt.max())] and eatt.max() == max_attempts


def test_sampler_reports_exhausted_attempts(spo, oracle):
    # one prompt holds nearly all the weight: later slots cannot find a free id in 2 attempts
    say("sample_prompts exhausted attempts")
    a = np.full(64, 1e-12, np.float32)
    b = np.full(64, 1.0, np.float32)
    a[3] = 1.0
    with pytest.raises(RuntimeError):
        oracle.sample_prompts(a, b, 8, 0.0, 0, 0, False, max_attempts=2)
    first = oracle.sample_prompts(a, b, 1, 0.0, 0, 0, False)
    gidx, info = spo.spo_sample_prompts(dev(a), dev(b), 8, 0.0, 0, 0, False, max_attempts=2, return_info=True)
    torch.cuda.synchronize()
    out = gidx.cpu().numpy()
    assert info.cpu().numpy()[0] == 1 and (out == -1).any() and out[0] == first[0]
    alive = out[out >= 0]
    assert len(set(alive.tolist())) == len(alive)


@pytest.mark.parametrize("replace", [True, False])
def test_sampler_with_all_weights_zero(spo, oracle, replace):
    # no exploration bonus and every estimate at 0 or 1: every weight is zero
    say(f"sample_prompts total weight zero, replace={replace}")
    a = np.array([0.0, 3.0, 0.0, 1.0], np.float32)
    b = np.array([2.0, 0.0, 5.0, 0.0], np.float32)
    with pytest.raises(RuntimeError):
        oracle.sample_prompts(a, b, 3, 0.0, 1, 2, replace)
    gidx, info = spo.spo_sample_prompts(dev(a), dev(b), 3, 0.0, 1, 2, replace, return_info=True)
    torch.cuda.synchronize()
    assert (gidx.cpu().numpy() == -1).all() and info.cpu().numpy()[0] == 1


def test_sampler_after_update_sees_new_state(spo, oracle):
    # the order of the training loop: sample -> advantages (pre-update) -> update
    cfg = wl.CONFIGS["C2"]
    say("loop order C2")
    a, b = wl.tracker_state(cfg, 41)
    ga, gb = dev(a), dev(b)
    idx = spo.spo_sample_prompts(ga, gb, 64, cfg.eps_explore, 0, 0)
    eidx = oracle.sample_prompts(a, b, 64, cfg.eps_explore, 0, 0)
    r = wl.rewards(cfg, eidx, 41)
    kl = wl.kl_divergences(cfg, 64, 41)
    raw, nrm, _ = spo.spo_advantages(ga, gb, idx, dev(r))
    spo.spo_tracker_update(ga, gb, idx, dev(r), dev(kl), cfg.d_half, cfg.rho_min, cfg.rho_max)
    raw_after, _, _ = spo.spo_advantages(ga, gb, idx, dev(r))
    torch.cuda.synchronize()
    eraw, enrm, _ = oracle.advantages(a, b, eidx, r)
    assert np.array_equal(idx.cpu().numpy(), eidx)
    np.testing.assert_allclose(raw.cpu().numpy(), eraw, rtol=RTOL, atol=1e-7)
    np.testing.assert_allclose(nrm.cpu().numpy(), enrm, rtol=RTOL, atol=1e-6)
    assert (raw_after.abs() < raw.abs()).all()
    ea, eb, _, _ = oracle.tracker_update(a, b, eidx, r, kl, cfg.d_half, cfg.rho_min, cfg.rho_max)
    idx2 = spo.spo_sample_prompts(ga, gb, 64, cfg.eps_explore, 0, 1)
    torch.cuda.synchronize()
    # the oracle's fp64 state rounded to fp32 is what the next draw must see
    assert np.array_equal(idx2.cpu().numpy(),
                          oracle.sample_prompts(ga.cpu().numpy(), gb.cpu().numpy(), 64, cfg.eps_explore, 0, 1))
    np.testing.assert_allclose(ga.cpu().numpy(), ea, rtol=RTOL)


def test_advantage_diagnostics_match_oracle(spo, oracle):
    cfg = wl.CONFIGS["C5"]
    say("advantage_diagnostics C5 n=4096")
    a, b, idx, r, _ = _update_case(cfg, 4096, 51)
    raw, _, _ = spo.spo_advantages(dev(a), dev(b), dev(idx), dev(r))
    diag = spo.spo_advantage_diagnostics(raw, dev(r), 1e-4, 0.02)
    torch.cuda.synchronize()
    rawc = raw.cpu().numpy()
    want = oracle.advantage_diagnostics(rawc, r, float(np.float32(1e-4)), float(np.float32(0.02)))
    got = diag.cpu().numpy()
    assert got[0] == np.float32(want[0]) and got[1] == np.float32(want[1])     # counts are exact
    np.testing.assert_allclose(got[2:], want[2:], rtol=RTOL)


def test_tracker_update_with_general_rewards(spo, oracle):
    cfg = wl.CONFIGS["C2"]
    say("tracker_update non-binary rewards")
    a, b, idx, _, kl = _update_case(cfg, 64, 61)
    r = np.random.default_rng(61).uniform(0, 1, 64).astype(np.float32)
    ea, eb, ev, _ = oracle.tracker_update(a, b, idx, r, kl, cfg.d_half, cfg.rho_min, cfg.rho_max)
    ga, gb = dev(a), dev(b)
    gv = spo.spo_tracker_update(ga, gb, dev(idx), dev(r), dev(kl), cfg.d_half, cfg.rho_min, cfg.rho_max,
                                want_v_prev=True)
    torch.cuda.synchronize()
    np.testing.assert_allclose(ga.cpu().numpy(), ea, rtol=RTOL)
    np.testing.assert_allclose(gb.cpu().numpy(), eb, rtol=RTOL)
    np.testing.assert_allclose(gv.cpu().numpy(), ev, rtol=RTOL)


@pytest.mark.parametrize("unique", [True, False])
def test_tracker_update_ema_matches_oracle(spo, oracle, unique):
    # moving-average form of the tracker, rewards outside [0, 1]
    cfg = wl.CONFIGS["C5"]
    say(f"tracker_update_ema unique={unique}")
    rng = np.random.default_rng(71)
    N, B = 4096, 1500
    v = rng.uniform(-1, 3, N).astype(np.float32)
    n = rng.uniform(1, 25, N).astype(np.float32)
    idx = (rng.permutation(N)[:B] if unique else rng.integers(0, 64, B)).astype(np.int32)
    r = rng.normal(1.0, 2.0, B).astype(np.float32)
    kl = rng.exponential(0.02, B).astype(np.float32)
    ev, en, evp = oracle.tracker_update_ema(v, n, idx, r, kl, cfg.d_half, cfg.rho_min, cfg.rho_max)
    gv, gn = dev(v), dev(n)
    cnt = torch.zeros(N, dtype=torch.int32, device="cuda")
    gvp = spo.spo_tracker_update_ema(gv, gn, dev(idx), dev(r), dev(kl), cfg.d_half, cfg.rho_min, cfg.rho_max,
                                     ids_unique=unique, n_obs=cnt, want_v_prev=True)
    torch.cuda.synchronize()
    np.testing.assert_allclose(gv.cpu().numpy(), ev, rtol=RTOL, atol=1e-6)
    np.testing.assert_allclose(gn.cpu().numpy(), en, rtol=RTOL)
    np.testing.assert_allclose(gvp.cpu().numpy(), evp, rtol=RTOL, atol=1e-6)
    assert np.array_equal(cnt.cpu().numpy(), np.bincount(idx, minlength=N))


def test_advantages_from_the_estimate_itself(spo, oracle):
    say("advantages with beta=None")
    rng = np.random.default_rng(72)
    N, B = 512, 200
    v = rng.uniform(-1, 3, N).astype(np.float32)
    idx = rng.permutation(N)[:B].astype(np.int32)
    r = rng.normal(1.0, 2.0, B).astype(np.float32)
    eraw, enrm, est = oracle.advantages(v, None, idx, r)
    raw, nrm, st = spo.spo_advantages(dev(v), None, dev(idx), dev(r))
    torch.cuda.synchronize()
    np.testing.assert_allclose(raw.cpu().numpy(), eraw, rtol=RTOL, atol=1e-6)
    np.testing.assert_allclose(nrm.cpu().numpy(), enrm, rtol=RTOL, atol=1e-6)
    np.testing.assert_allclose(st.cpu().numpy(), est, rtol=RTOL)


@pytest.mark.parametrize("B", [7168, 7169, 8191, 8192, 8193, 15361, 100003])   # a thread's whole groups of eight, and what is left
def test_diagnostics_of_long_batches(spo, B):
    say(f"advantage diagnostics B={B}")
    rng = np.random.default_rng(B)
    a = (rng.standard_normal(B) * 0.05 + 3.0 * (rng.random(B) < 0.1)).astype(np.float32)
    r = rng.random(B).astype(np.float32)
    diag = spo.spo_advantage_diagnostics(dev(a), dev(r), 1e-3, 0.02)
    torch.cuda.synchronize()
    a64, r64 = a.astype(np.float64), r.astype(np.float64)
    want = [(np.abs(a) <= np.float32(1e-3)).mean(), (np.abs(a) <= np.float32(0.02)).mean(), a64.var(), r64.var()]
    np.testing.assert_allclose(diag.cpu().numpy(), want, rtol=2e-7, atol=0)   # fp64 sums, one rounding to fp32


@pytest.mark.parametrize("B", [8191, 8192, 8193, 15360, 15361])   # eight responses per thread, and up to sixteen
@pytest.mark.parametrize("beta", [True, False])
def test_advantages_in_two_batches_of_loads(spo, oracle, B, beta):
    test_advantages_kept_in_registers(spo, oracle, B, beta)


@pytest.mark.parametrize("B", [1025, 1281, 4096, 65536, 65537])   # one response per thread up to 256 workgroups, then four
def test_advantages_spread_from_small_batches_on(spo, oracle, B):
    cfg = wl.CONFIGS["C5"]
    say(f"advantages over many workgroups, B={B}")
    a, b = wl.tracker_state(cfg, 7)
    rng = np.random.default_rng([wl.MASTER_SEED, B, 2])
    idx = rng.integers(0, cfg.N, B).astype(np.int32)
    r = (rng.random(B) < 0.4).astype(np.float32)
    eraw, enrm, (mu, sigma) = oracle.advantages(a, b, idx, r, 1, 0.0, True)
    args = (dev(a), dev(b), dev(idx), dev(r), 1, 0.0, True)
    sizes = [spo.lib().spo_advantages_workspace_bytes(n) for n in range(1, B + 1, 97)] + [spo.lib().spo_advantages_workspace_bytes(B)]
    assert sizes == sorted(sizes)
    full = torch.full((sizes[-1] + 256,), 255, dtype=torch.uint8, device="cuda")
    for n in (sizes[-1], 16 * -(-B // 4096)):   # as asked for, and what workgroups of 4096 responses need
        full.fill_(255)
        raw, nrm, st = spo.spo_advantages(*args, workspace=full[:n])
        torch.cuda.synchronize()
        assert bool((full[n:] == 255).all())
        np.testing.assert_allclose(raw.cpu().numpy(), eraw, rtol=RTOL, atol=1e-7)
        np.testing.assert_allclose(nrm.cpu().numpy(), enrm, rtol=RTOL, atol=1e-6)
        np.testing.assert_allclose(st.cpu().numpy(), [mu, sigma], rtol=RTOL, atol=1e-7)


@pytest.mark.parametrize("N,most", [(0, 3072), (1000, 3072), (1 << 15, 3072), (40000, 2048), (300000, 1024)])   # 0: no baseline
@pytest.mark.parametrize("more", [0, 1])
def test_advantages_of_small_tables_stay_in_one_workgroup(spo, oracle, N, most, more):
    # which shows in the workspace: only launches over several workgroups write to it
    B = most + more
    say(f"advantages of {B} responses to {N} prompts")
    rng = np.random.default_rng([N, B])
    a, b = (rng.uniform(0.5, 50, max(N, 1)).astype(np.float32) for _ in range(2))
    idx = rng.integers(0, max(N, 1), B).astype(np.int32)
    r = (rng.random(B) < 0.4).astype(np.float32)
    eraw, enrm, (mu, sigma) = oracle.advantages(a, b, idx, r, 0, 0.0, N > 0)
    ws = torch.full((spo.lib().spo_advantages_workspace_bytes(B),), 255, dtype=torch.uint8, device="cuda")
    raw, nrm, st = spo.spo_advantages(dev(a), dev(b), dev(idx), dev(r), use_baseline=N > 0, workspace=ws)
    torch.cuda.synchronize()
    assert bool((ws == 255).all()) == (more == 0)
    np.testing.assert_allclose(raw.cpu().numpy(), eraw, rtol=RTOL, atol=1e-7)
    np.testing.assert_allclose(nrm.cpu().numpy(), enrm, rtol=RTOL, atol=1e-6)
    np.testing.assert_allclose(st.cpu().numpy(), [mu, sigma], rtol=RTOL, atol=1e-7)


@pytest.mark.parametrize("B", [1, 1024, 1025, 8192, 8193, 12288, 12289, 24576, 24577, 40960, 40961])   # 1, 8, 12, 24, 40 per thread, any number
def test_diagnostics_kept_in_registers(spo, B):
    say(f"diagnostics, B={B}")
    rng = np.random.default_rng([B, 4])
    adv = rng.standard_normal(B).astype(np.float32)
    r = (rng.random(B) < 0.4).astype(np.float32)
    d = spo.spo_advantage_diagnostics(dev(adv), dev(r), 0.1, 0.3).cpu().numpy()
    a64 = adv.astype(np.float64)
    want = [(np.abs(adv) <= np.float32(0.1)).mean(), (np.abs(adv) <= np.float32(0.3)).mean(), a64.var(), r.astype(np.float64).var()]
    np.testing.assert_allclose(d, want, rtol=1e-6, atol=1e-9)


@pytest.mark.parametrize("B,N,hot,offset", [
    (6, 40, 0.5, 1), (512, 300, 0.0, 0), (2048, 900, 0.0, 1), (2049, 40, 0.5, 2),    # lists that need no count: one length of
    (4096, 1, 0.0, 1), (4096, 20000, 0.0, 0),                                        # chunk and the next
    (4097, 20000, 0.9, 3), (8192, 300, 0.0, 0), (8193, 300, 0.9, 1),                 # counted, shorter chunks and the long ones
    (16383, 5000, 0.0, 0), (16385, 5000, 0.0, 1),   # one chunk of ids and a little more, from an odd place on
    (40000, 300, 0.0, 0),                           # few prompts: long lists, sorted by the other sort
    (33000, 20000, 0.9, 3)])                        # one prompt with most of them: lists applied and restarted
def test_tracker_update_reads_ids_in_chunks(spo, oracle, B, N, hot, offset):
    say(f"tracker update, repeated ids, B={B} N={N} hot={hot} offset={offset}")
    rng = np.random.default_rng([B, N])
    idx = rng.integers(0, N, B).astype(np.int32)
    idx[rng.random(B) < hot] = 17
    bad = rng.integers(0, B, 5)
    idx[bad[:3]], idx[bad[3:]] = N, -1
    r = (rng.random(B) < 0.4).astype(np.float32)
    kl = rng.exponential(0.02, B).astype(np.float32)
    a, b = (rng.uniform(0.5, 50, N).astype(np.float32) for _ in range(2))
    ea, eb = a.astype(np.float32).copy(), b.astype(np.float32).copy()
    for k in range(B):   # sequential, one rounding to fp32 per observation
        i = idx[k]
        if 0 <= i < N:
            rho = min(max(2.0 ** (-float(kl[k]) / 0.25), 0.875), 0.96)
            ea[i] = np.float32(rho * float(ea[i]) + float(r[k]))
            eb[i] = np.float32(rho * float(eb[i]) + (1.0 - float(r[k])))
    ga, gb = dev(a), dev(b)
    ids = torch.zeros(B + offset, dtype=torch.int32, device="cuda")
    ids[offset:] = dev(idx)
    info = torch.zeros(1, dtype=torch.int32, device="cuda")
    vp = spo.spo_tracker_update(ga, gb, ids[offset:], dev(r), dev(kl), 0.25, 0.875, 0.96, ids_unique=False, want_v_prev=True, info=info)
    torch.cuda.synchronize()
    assert info.item() == 1 and torch.isnan(vp[torch.as_tensor(np.unique(bad)).cuda()]).all()
    assert int(torch.isnan(vp).sum()) == len(np.unique(bad))
    np.testing.assert_allclose(ga.cpu().numpy(), ea, rtol=1e-5)
    np.testing.assert_allclose(gb.cpu().numpy(), eb, rtol=1e-5)


@pytest.mark.parametrize("N,B", [(4097, 300), (4160, 3500), (8193, 64), (100001, 3000), ((1 << 22) + 4097, 700)])
@pytest.mark.parametrize("replace", [False, True])
@pytest.mark.parametrize("zeros", [False, True])
def test_sampler_searches_of_blocks(spo, oracle, N, B, replace, zeros):
    # ends of blocks of 4096 prompts and of runs of 64 in them, more blocks than LDS holds sums of; with eps = 0 whole
    # blocks may have no weight at all
    say(f"sampler, N={N} B={B} replace={replace} zeros={zeros}")
    rng = np.random.default_rng([N, B])
    a = rng.uniform(0.5, 50, N).astype(np.float32)
    b = rng.uniform(0.5, 50, N).astype(np.float32)
    if zeros:   # blocks without weight at both ends and between, but enough prompts left
        b[: 4096 if N > 2 * 4096 else 64] = 0
        b[N // 2: N // 2 + min(N // 8, 9000)] = 0
        b[-1:] = 0
        B = min(B, N // 2)
    eps = 0.0 if zeros else 0.05
    idx, info = spo.spo_sample_prompts(dev(a), dev(b), B, eps, 11, 5, replace, return_info=True)
    torch.cuda.synchronize()
    want = oracle.sample_prompts(a, b, B, eps, 11, 5, replace)
    want = want[0] if isinstance(want, tuple) else want
    np.testing.assert_array_equal(idx.cpu().numpy(), want)
