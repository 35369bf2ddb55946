"""Nucleus (top-p) sampling on the GPU against the oracle's rule: the sampler
alone on given logits, then inside the decode step (single calls, graph replay,
ragged positions)."""
import numpy as np
import pytest
import torch

import srm_synth
from gpu_util import to_dev

pytestmark = pytest.mark.gpu

MASS_TOL = 1e-5        # a cut decided by less probability than this may fall either way in fp32


@pytest.fixture(scope="module")
def srm():
    import paper_2605_08696_amd as pkg
    pkg.lib()
    return pkg


@pytest.fixture(scope="module")
def orc_mod(oracle_mod):
    return oracle_mod


def _check_rows(orc_mod, got, logits, T, top_p, seed, pos_of, b_of=None):
    """Every GPU choice equals the oracle's choice from the same logits, unless the oracle's own
    decision was a near tie (nucleus boundary within MASS_TOL, or top-2 scores within 1e-5 of
    the logit scale).  Returns (tolerated, rows where truncation changed the plain draw)."""
    tolerated = changed = 0
    for r in range(logits.shape[0]):
        b = r if b_of is None else b_of[r]
        tok, mg, mm = orc_mod.pick_topp(logits[r], T, top_p, seed, pos_of(r), b, want_margins=True)
        if orc_mod.pick(logits[r], T, seed, pos_of(r), b) != tok:
            changed += 1
        if got[r] != tok:
            assert mm < MASS_TOL or mg < 1e-5 * np.abs(logits[r]).max(), f"row {r}: {got[r]} != {tok}"
            tolerated += 1
    return tolerated, changed


@pytest.mark.parametrize("V,scale,T,top_p", [(40, 2.0, 1.0, 0.5), (1000, 3.0, 0.7, 0.9), (4099, 0.05, 0.7, 0.9),
                                            (4099, 4.0, 1.5, 0.99), (32000, 2.0, 0.7, 0.9), (32000, 0.02, 0.7, 0.9),
                                            (777, 6.0, 0.7, 0.05)])
def test_sample_logits_matches_oracle(srm, orc_mod, V, scale, T, top_p):
    rows = 256 if V >= 32000 else 600
    rng = np.random.default_rng(V + int(100 * top_p))
    logits = (rng.standard_normal((rows, V)) * scale).astype(np.float32)
    logits[3, :] = logits[3, 0]                               # a row of equal logits: everything is kept
    if V > 100:
        logits[4, 10:20] = logits[4].max() + 1.0              # ties at the top
    print(f"sample_logits V={V} scale={scale} T={T} top_p={top_p} rows={rows}", flush=True)
    dl = to_dev(logits)
    out = torch.full((rows,), -5, dtype=torch.int32, device="cuda")
    seed, pos = 77, 9
    srm.sample_logits(dl, T, top_p, seed, pos, out)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    tolerated, changed = _check_rows(orc_mod, got, logits, T, top_p, seed, lambda r: pos)
    assert tolerated <= max(2, rows // 50)
    if top_p <= 0.9:
        assert changed > 0                                      # the truncation mattered for some rows
    # same call again: bit-reproducible
    out2 = torch.empty_like(out)
    srm.sample_logits(dl, T, top_p, seed, pos, out2)
    assert torch.equal(out, out2)
    # top_p = 1: the plain Gumbel-max draw
    srm.sample_logits(dl, T, 1.0, seed, pos, out2)
    torch.cuda.synchronize()
    plain = out2.cpu().numpy()
    for r in range(0, rows, 7):
        assert plain[r] == orc_mod.pick(logits[r], T, seed, pos, r)


def test_sample_logits_frequencies_follow_truncated_softmax(srm, orc_mod):
    import scipy.stats
    lg = np.array([1.2, -0.3, 0.4, 2.0, 0.0, -1.5, 0.9, 0.1], np.float32)
    T, top_p, R = 0.7, 0.9, 80000
    keep, _ = orc_mod.nucleus(lg, T, top_p)
    p = np.exp(lg.astype(np.float64) / T) * keep; p /= p.sum()
    out = torch.empty(R, dtype=torch.int32, device="cuda")
    srm.sample_logits(to_dev(np.tile(lg, (R, 1))), T, top_p, 5, 0, out)
    torch.cuda.synchronize()
    counts = np.bincount(out.cpu().numpy(), minlength=lg.size)
    assert counts[~keep].sum() == 0
    assert scipy.stats.chisquare(counts[keep], p[keep] * R).pvalue > 1e-4


def _topp_run(model, prompts_np, G, T, top_p, seed, mode):
    """Prefill all but the last prompt token, then G nucleus-sampled steps."""
    B, P = prompts_np.shape
    dp = to_dev(prompts_np)
    ws = model.new_workspace(B * P)
    st, tk = model.new_state(B), torch.empty(B, dtype=torch.int32, device="cuda")
    model.prefill(dp[:, :P - 1].contiguous(), 1, st, tk, workspace=ws)
    tk.copy_(dp[:, P - 1])
    lg = torch.empty((B, model.vocab), dtype=torch.float32, device="cuda")
    out = torch.empty((G, B), dtype=torch.int32, device="cuda")
    if mode == "generate":
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            model.generate(B, P - 1, G, tk, st, out, workspace=ws, temperature=T, seed=seed, top_p=top_p, logits=lg)
        side.synchronize()
    elif mode == "ragged":
        pos = torch.full((B,), P - 1, dtype=torch.int32, device="cuda")
        for g in range(G):
            model.decode_step_ragged(B, pos, tk, st, tk, advance=True, temperature=T, seed=seed, top_p=top_p,
                                     logits=lg, workspace=ws)
            out[g] = tk
        assert (pos == P - 1 + G).all()
    else:
        for g in range(G):
            model.decode_step(B, P - 1 + g, tk, st, tk, logits=lg, workspace=ws, temperature=T, seed=seed,
                              top_p=top_p)
            out[g] = tk
    torch.cuda.synchronize()
    return out.cpu().numpy().T


@pytest.mark.parametrize("mode", ["steps", "generate", "ragged"])
def test_topp_generation_matches_oracle_fp32(srm, orc_mod, mode):
    cfg = srm_synth.CONFIGS["C1"]
    w = srm_synth.make_weights(cfg)
    w["head"] = w["head"] * 25.0                                # peaked enough for the nucleus to be a strict subset
    prompts = srm_synth.make_prompts(cfg)
    G, T, top_p, seed = 24, 0.7, 0.9, 2024
    print(f"top-p generation mode={mode}", flush=True)
    ref = orc_mod.Oracle(cfg, w, "f64").greedy(prompts, G, want_logits=True, temperature=T, seed=seed, top_p=top_p)
    plain = orc_mod.Oracle(cfg, w, "f64").greedy(prompts, G, temperature=T, seed=seed)
    assert (ref["tokens"] != plain["tokens"]).any()             # the truncation changes this run
    model = srm.Model(cfg, w)
    got = _topp_run(model, prompts, G, T, top_p, seed, mode)
    absmax = np.abs(ref["logits"]).max(axis=2)
    bad = got != ref["tokens"]
    near = (ref["margin"] < 1e-4 * absmax) | (ref["mass_margin"] < MASS_TOL)
    # a tolerated near tie may change everything after it in that row: compare up to the first one
    for b in range(got.shape[0]):
        stop = np.argmax(near[b]) if near[b].any() else G
        assert not bad[b, :stop].any(), f"row {b} differs from the oracle before any near tie"
    assert near.sum() <= 2
    # top_p = 1 through the same entry point is plain sampling; temperature 0 is greedy
    np.testing.assert_array_equal(_topp_run(model, prompts, 6, T, 1.0, seed, mode), plain["tokens"][:, :6])
    greedy = orc_mod.Oracle(cfg, w, "f64").greedy(prompts, 6)
    np.testing.assert_array_equal(_topp_run(model, prompts, 6, 0.0, 0.9, seed, mode), greedy["tokens"])


def test_topp_step_bf16_rows_against_oracle_rule(srm, orc_mod):
    """bf16 MFMA head (several tiles): every row's token equals the oracle's nucleus choice from the
    GPU's own logits, and the uniform and ragged entry points agree bit for bit."""
    cfg = srm_synth.tiny_config(vocab=1500, d_model=128, n_layers=2, n_heads=4, n_ctx=16, weight_dtype="bf16", seed=31)
    w = srm_synth.make_weights(cfg, stress=True)
    w["head"] = srm_synth.round_to_bf16(w["head"] * 30.0)
    model = srm.Model(cfg, w)
    B, T, top_p, seed, pos = 700, 0.8, 0.7, 11, 3
    rng = np.random.default_rng(2)
    tok = to_dev(rng.integers(0, cfg.vocab, B).astype(np.int32))
    st0 = torch.randn(cfg.n_layers * B * cfg.d_model, device="cuda") * 0.1
    ws = model.new_workspace(B)
    lg = torch.empty((B, cfg.vocab), dtype=torch.float32, device="cuda")
    out = torch.empty(B, dtype=torch.int32, device="cuda")
    st = st0.clone()
    print(f"top-p bf16 step B={B}", flush=True)
    model.decode_step(B, pos, tok, st, out, logits=lg, workspace=ws, temperature=T, seed=seed, top_p=top_p)
    torch.cuda.synchronize()
    logits = lg.cpu().numpy()
    tolerated, changed = _check_rows(orc_mod, out.cpu().numpy(), logits, T, top_p, seed, lambda r: pos)
    assert tolerated <= 3 and changed > 0
    st2, out2 = st0.clone(), torch.empty_like(out)
    posr = torch.full((B,), pos, dtype=torch.int32, device="cuda")
    posr[5] = -1                                                # one idle slot
    model.decode_step_ragged(B, posr, tok, st2, out2, advance=True, temperature=T, seed=seed, top_p=top_p, logits=lg,
                             workspace=ws)
    torch.cuda.synchronize()
    live = torch.ones(B, dtype=torch.bool, device="cuda"); live[5] = False
    assert torch.equal(out2[live], out[live]) and int(out2[5]) == -1
    assert int(posr[5]) == -1 and (posr[live] == pos + 1).all()
    with pytest.raises(srm.SrmError):                           # the truncation needs the logits buffer
        model.decode_step(B, pos, tok, st, out, workspace=ws, temperature=T, seed=seed, top_p=top_p)


@pytest.mark.parametrize("V,groups", [(1501, 0), (32000, 0), (5001, 5), (5000, 8), (32000, 40)])
def test_topp_search_against_oracle_rule(srm, orc_mod, V, groups):
    """The nucleus search of the decode step: distinct logits (the cut lies in a step of few elements) and logits that
    take `groups` values only, each in more elements than a step may gather; vocabularies that are read by fours and
    that are not.  Every row's token equals the oracle's choice from the GPU's own logits."""
    cfg = srm_synth.tiny_config(vocab=V, d_model=64, n_layers=1, n_heads=4, n_ctx=16, seed=5)
    w = srm_synth.make_weights(cfg, stress=True)
    w["head"] = w["head"] * 20.0
    if groups:
        w["head"] = w["head"][np.arange(V) % groups].copy()
    model = srm.Model(cfg, w)
    B, T, top_p, seed, pos = 40, 0.8, 0.7, 12, 3
    print(f"top-p search V={V} groups={groups}", flush=True)
    tok = to_dev(np.arange(B, dtype=np.int32) * 7 % V)
    st = torch.randn(cfg.n_layers * B * cfg.d_model, device="cuda") * 0.1
    lg = torch.empty((B, V), dtype=torch.float32, device="cuda")
    out = torch.empty(B, dtype=torch.int32, device="cuda")
    model.decode_step(B, pos, tok, st, out, logits=lg, workspace=model.new_workspace(B), temperature=T, seed=seed,
                      top_p=top_p)
    torch.cuda.synchronize()
    tolerated, changed = _check_rows(orc_mod, out.cpu().numpy(), lg.cpu().numpy(), T, top_p, seed, lambda r: pos)
    assert tolerated <= 2 and changed > 0


@pytest.mark.parametrize("V", [333, 1501])
@pytest.mark.parametrize("kind", ["close", "far"])
def test_topp_search_at_the_ends_of_the_float_range(srm, orc_mod, V, kind):
    """Logits so close together that the search's steps per unit of logit are beyond the float range (all elements in
    the last step: few enough to be gathered, and too many), and so far apart that the difference between the largest
    and w0 is (all in the first step).  Both distributions put w0 outside the nucleus in a good part of the rows."""
    cfg = srm_synth.tiny_config(vocab=V, d_model=64, n_layers=1, n_heads=4, n_ctx=16, seed=6)
    w = srm_synth.make_weights(cfg, stress=True)
    rng = np.random.default_rng(V)
    if kind == "close":                              # equally likely within the precision of the noise
        x, T, top_p = rng.standard_normal(V).clip(-3.2, 3.2) * 2e-37, 0.8, 0.7
    else:                                            # one logit 3.6e38 above the others, at a temperature of that order
        x, T, top_p = rng.uniform(-3.2e38, -3.1e38, V), 0.8e38, 0.05
        x[V // 3] = 0.5e38
    w["lnf_g"], w["lnf_b"] = np.zeros_like(w["lnf_g"]), np.eye(1, cfg.d_model, dtype=np.float32)[0]
    w["head"] = np.zeros_like(w["head"])
    w["head"][:, 0] = x                              # the logits of every row
    B, seed, pos = 40, 12, 3
    print(f"top-p search V={V} {kind}", flush=True)
    model = srm.Model(cfg, w)
    st = torch.zeros(cfg.n_layers * B * cfg.d_model, device="cuda")
    lg = torch.empty((B, V), dtype=torch.float32, device="cuda")
    out = torch.empty(B, dtype=torch.int32, device="cuda")
    model.decode_step(B, pos, to_dev(np.zeros(B, np.int32)), st, out, logits=lg, workspace=model.new_workspace(B),
                      temperature=T, seed=seed, top_p=top_p)
    torch.cuda.synchronize()
    logits = lg.cpu().numpy()
    assert np.array_equal(logits[0], w["head"][:, 0])
    tolerated, changed = _check_rows(orc_mod, out.cpu().numpy(), logits, T, top_p, seed, lambda r: pos)
    assert tolerated == 0 and changed > 3


@pytest.mark.parametrize("seed", [96672, 140406, 213598, 422384, 756542, 1199177])
def test_topp_search_counts_a_long_flat_tail(srm, orc_mod, seed):
    """One dominant token, 256 of probability 1.4e-6 and 31 743 of 2.4e-10 each, 7.5e-6 together.  The seeds (found with
    the oracle's generator) draw one of the 256 whose mass from above exceeds the cut by 2e-6 .. 5e-6: outside the
    nucleus, but inside for a search that loses or rounds up the tail.  At fp32 the streaming pass that lists the row
    rounds by 2^-24 of a mass of 1, a thirtieth of that distance."""
    V, pos = 32000, 3
    x = np.full(V, np.log(0.51 * 2.0 ** -31))
    x[0] = 0.0
    mid = 1 + 120 * np.arange(256)
    x[mid] = np.log(1.4e-6) - 1e-4 * np.arange(256)
    top_p = float(np.float32(0.99981743))
    cfg = srm_synth.tiny_config(vocab=V, d_model=64, n_layers=1, n_heads=4, n_ctx=16, seed=6)
    w = srm_synth.make_weights(cfg, stress=True)
    w["lnf_g"], w["lnf_b"] = np.zeros_like(w["lnf_g"]), np.eye(1, cfg.d_model, dtype=np.float32)[0]
    w["head"] = np.zeros_like(w["head"])
    w["head"][:, 0] = x                              # the logits, whatever the token
    print(f"top-p search with a flat tail, seed={seed}", flush=True)
    model = srm.Model(cfg, w)
    lg = torch.empty((1, V), dtype=torch.float32, device="cuda")
    out = torch.empty(1, dtype=torch.int32, device="cuda")
    model.decode_step(1, pos, to_dev(np.zeros(1, np.int32)), torch.zeros(cfg.n_layers * cfg.d_model, device="cuda"), out,
                      logits=lg, workspace=model.new_workspace(1), temperature=1.0, seed=seed, top_p=top_p)
    torch.cuda.synchronize()
    logits = lg.cpu().numpy()[0]
    assert np.array_equal(logits, w["head"][:, 0])
    drawn = orc_mod.pick(logits, 1.0, seed, pos, 0)
    assert drawn in mid[130:133]
    assert int(out[0]) == orc_mod.pick_topp(logits, 1.0, top_p, seed, pos, 0) != drawn


@pytest.mark.parametrize("B,V", [(257, 31004), (300, 31004), (300, 31002), (300, 2001)])
def test_noise_in_the_head_of_large_tiles(srm, orc_mod, B, V):
    """Plain sampling inside the bf16 LM head: the persistent 256x256 tile (31 004 columns, the row tile's groups of
    sixteen rows whole, ragged and empty), the 256x256 tile of odd vocabularies and the 128x128 one.  Every row's token
    is the oracle's choice from the GPU's own logits, the same without a logits buffer, at one position and at positions
    of each row's own, idle rows among them."""
    cfg = srm_synth.tiny_config(vocab=V, d_model=128, n_layers=1, n_heads=4, n_ctx=16, weight_dtype="bf16", seed=33)
    w = srm_synth.make_weights(cfg, stress=True)
    w["head"] = srm_synth.round_to_bf16(w["head"] * 30.0)
    model = srm.Model(cfg, w)
    T, seed, pos = 0.8, 13, 3
    rng = np.random.default_rng(4)
    tok = to_dev(rng.integers(0, V, B).astype(np.int32))
    st0 = torch.randn(cfg.n_layers * B * cfg.d_model, device="cuda") * 0.1
    posr0 = rng.integers(0, cfg.n_ctx - 1, B).astype(np.int32)
    posr0[[0, B // 2, B - 1]] = -1
    ws = model.new_workspace(B)
    lg = torch.empty((B, V), dtype=torch.float32, device="cuda")
    for ragged in (False, True):
        print(f"sampled head B={B} V={V} ragged={ragged}", flush=True)
        res = []
        for logits in (lg, None):
            st, out = st0.clone(), torch.full((B,), -7, dtype=torch.int32, device="cuda")
            if ragged:
                model.decode_step_ragged(B, to_dev(posr0), tok, st, out, advance=False, temperature=T, seed=seed,
                                         logits=logits, workspace=ws)
            else:
                model.decode_step(B, pos, tok, st, out, logits=logits, workspace=ws, temperature=T, seed=seed)
            res.append(out.cpu().numpy())
        np.testing.assert_array_equal(res[0], res[1])
        live = np.flatnonzero(posr0 >= 0) if ragged else np.arange(B)
        if ragged:
            assert (res[0][posr0 < 0] == -1).all()
        tolerated, _ = _check_rows(orc_mod, res[0][live], lg.cpu().numpy()[live], T, 1.0, seed,
                                   lambda r: int(posr0[live[r]]) if ragged else pos, b_of=live)
        assert tolerated <= 2
