"""Architectural variants through the C ABI, against the oracle run with the same switch."""
import dataclasses

import numpy as np
import pytest
import torch

import srm_synth
from gpu_util import to_dev, rel_err_rows, check_tokens

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def srm():
    import paper_2605_08696_amd as pkg
    pkg.lib()
    return pkg


@pytest.fixture(scope="module")
def orc_mod(oracle_mod):
    return oracle_mod


# ---- non-projected mixer layers ("Method", last paragraph; Tables S2-S4) -----------------------
def test_non_projected_fp32_all_paths_match_oracle(srm, orc_mod):
    cfg = dataclasses.replace(srm_synth.CONFIGS["C1"], use_projections=False)
    w = srm_synth.make_weights(cfg)
    orc = orc_mod.Oracle(cfg, w, "f64")
    model = srm.Model(cfg, w)
    prompts = srm_synth.make_prompts(cfg)                      # [8][16]
    B, P = prompts.shape
    G = 24
    ref = orc.greedy(prompts, G, want_logits=True)
    print("non-projected fp32: prefill + generate", flush=True)
    ws = model.new_workspace(B * P)
    st, tk = model.new_state(B), torch.empty(B, dtype=torch.int32, device="cuda")
    lg = torch.empty((B, cfg.vocab), dtype=torch.float32, device="cuda")
    model.prefill(to_dev(prompts), 1, st, tk, logits=lg, workspace=ws)
    assert rel_err_rows(lg.cpu().numpy(), ref["logits"][:, 0]) <= 1e-4
    out = torch.empty((G - 1, B), dtype=torch.int32, device="cuda")
    first = tk.cpu().numpy().copy()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        model.generate(B, P, G - 1, tk, st, out, workspace=ws)
    side.synchronize()
    got = np.concatenate([first[:, None], out.cpu().numpy().T], axis=1)
    absmax = np.abs(ref["logits"]).max(axis=2)
    assert check_tokens(got, ref["tokens"], ref["margin"], absmax) == 0
    # step by step from scratch, with logits and hidden state of every position
    toks = srm_synth.make_prompts(cfg, batch=3, length=20)
    rf = orc.recurrent_forward(toks)
    st3 = model.new_state(3); st3.zero_()
    o3 = torch.empty(3, dtype=torch.int32, device="cuda")
    l3 = torch.empty((3, cfg.vocab), dtype=torch.float32, device="cuda")
    h3 = torch.empty((3, cfg.d_model), dtype=torch.float32, device="cuda")
    tc = to_dev(toks).t().contiguous()
    for t in range(20):
        model.decode_step(3, t, tc[t], st3, o3, logits=l3, hidden=h3, workspace=ws)
        assert rel_err_rows(l3.cpu().numpy(), rf["logits"][:, t]) <= 1e-4
        assert rel_err_rows(h3.cpu().numpy(), rf["hidden"][:, t]) <= 1e-4
    # parallel form
    hid = torch.empty((3, 20, cfg.d_model), dtype=torch.float32, device="cuda")
    lgp = torch.empty((3, 20, cfg.vocab), dtype=torch.float32, device="cuda")
    model.parallel_forward(to_dev(toks), hid, logits=lgp, workspace=model.new_workspace(60))
    torch.cuda.synchronize()
    assert rel_err_rows(hid.cpu().numpy().reshape(60, -1), rf["hidden"].reshape(60, -1)) <= 1e-4
    assert rel_err_rows(lgp.cpu().numpy().reshape(60, -1), rf["logits"].reshape(60, -1)) <= 1e-4
    # ragged entry points
    lens = [3, 20, 11]
    pk = np.concatenate([toks[i, :n] for i, n in enumerate(lens)]).astype(np.int32)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    str_, tkr = model.new_state(3), torch.empty(3, dtype=torch.int32, device="cuda")
    pos = torch.empty(3, dtype=torch.int32, device="cuda")
    keep = model.prefill_ragged(to_dev(pk), off, str_, tkr, pos=pos, logits=l3, workspace=ws)
    torch.cuda.synchronize()
    del keep
    for b, n in enumerate(lens):
        assert rel_err_rows(l3[b:b + 1].cpu().numpy(), rf["logits"][b:b + 1, n - 1]) <= 1e-4


@pytest.mark.parametrize("B,d", [(5, 128), (300, 128), (300, 512)])
def test_non_projected_bf16_decode_matches_oracle(srm, orc_mod, B, d):
    cfg = srm_synth.tiny_config(vocab=400, d_model=d, n_layers=3, n_heads=4, n_ctx=12, weight_dtype="bf16", seed=61,
                                use_projections=False)
    w = srm_synth.make_weights(cfg, stress=True)
    T = 8
    toks = srm_synth.make_prompts(cfg, batch=B, length=T)
    rows = sorted({0, 1, B // 2, B - 1})
    ref = orc_mod.Oracle(cfg, w, "f64").recurrent_forward(toks[rows])
    model = srm.Model(cfg, w)
    ws, st = model.new_workspace(B * T), model.new_state(B)
    st.zero_()
    out = torch.empty(B, dtype=torch.int32, device="cuda")
    lg = torch.empty((B, cfg.vocab), dtype=torch.float32, device="cuda")
    tc = to_dev(toks).t().contiguous()
    print(f"non-projected bf16 B={B}", flush=True)
    for t in range(T):
        model.decode_step(B, t, tc[t], st, out, logits=lg, workspace=ws)
        assert rel_err_rows(lg[rows].cpu().numpy(), ref["logits"][:, t]) <= 2e-2
    # prefill of the same tokens reaches the same state
    st2, tk2 = model.new_state(B), torch.empty(B, dtype=torch.int32, device="cuda")
    model.prefill(to_dev(toks), 1, st2, tk2, workspace=ws)
    torch.cuda.synchronize()
    assert (st - st2).abs().max() <= 2e-2 * st.abs().max()
    s_ref = ref["state"]                                       # [rows][L][d]
    s_got = st.view(cfg.n_layers, B, cfg.d_model)[:, rows].permute(1, 0, 2).cpu().numpy()
    assert np.abs(s_got - s_ref).max() <= 2e-2 * np.abs(s_ref).max()


# ---- half-precision cache ("SRM architecture optimization", last sentence) ----------------------
def test_half_state_fp32_weights_all_paths_match_oracle(srm, orc_mod):
    cfg = dataclasses.replace(srm_synth.CONFIGS["C1"], state_dtype="fp16")
    w = srm_synth.make_weights(cfg)
    orc = orc_mod.Oracle(cfg, w, "f64")
    model = srm.Model(cfg, w)
    assert model.state_bytes(10) == cfg.n_layers * 10 * cfg.d_model * 2
    prompts = srm_synth.make_prompts(cfg)
    B, P = prompts.shape
    G = 24
    ref = orc.greedy(prompts, G, want_logits=True)
    print("half state: prefill + generate", flush=True)
    ws = model.new_workspace(B * P)
    st, tk = model.new_state(B), torch.empty(B, dtype=torch.int32, device="cuda")
    assert st.dtype == torch.float16
    lg = torch.empty((B, cfg.vocab), dtype=torch.float32, device="cuda")
    model.prefill(to_dev(prompts), 1, st, tk, logits=lg, workspace=ws)
    assert rel_err_rows(lg.cpu().numpy(), ref["logits"][:, 0]) <= 1e-3
    # the same prompts one decode step at a time: every update is rounded alike; the two paths use different
    # GEMM kernels (fp32 sums in another order), so a cache value may differ in its last binary16 place
    st_b, tk_b = model.new_state(B), torch.empty(B, dtype=torch.int32, device="cuda")
    pc = to_dev(prompts).t().contiguous()
    for t in range(P):
        model.decode_step(B, t, pc[t], st_b, tk_b, workspace=ws)
    torch.cuda.synchronize()
    assert (st != st_b).float().mean() < 0.2                   # last-place differences persist and spread downstream
    assert (st.float() - st_b.float()).abs().max() <= 2e-3 * st_b.float().abs().max()
    assert torch.equal(tk, tk_b)
    out = torch.empty((G - 1, B), dtype=torch.int32, device="cuda")
    first = tk.cpu().numpy().copy()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        model.generate(B, P, G - 1, tk, st, out, workspace=ws)
    side.synchronize()
    got = np.concatenate([first[:, None], out.cpu().numpy().T], axis=1)
    absmax = np.abs(ref["logits"]).max(axis=2)
    # the GPU rounds an fp32 sum to binary16, the oracle an fp64 sum: a rare last-bit difference in a cache
    # value may move a logit by ~1e-4 relative, so near ties are judged with that margin
    assert check_tokens(got, ref["tokens"], ref["margin"], absmax, rtol=1e-3) <= 2
    # cache against the oracle's after the whole run: binary16 values, equal except rare last-place differences
    seq = np.concatenate([prompts, ref["tokens"][:, :G - 1]], axis=1)
    s_ref = orc.greedy(seq, 1)["state"]                         # [B][L][d]
    if (got == ref["tokens"]).all():
        s_got = st.float().view(cfg.n_layers, B, cfg.d_model).permute(1, 0, 2).cpu().numpy()
        diff = s_got != s_ref
        assert diff.mean() < 0.3
        assert np.abs(s_got - s_ref).max() <= 2e-3 * np.abs(s_ref).max()
    # ragged decode equals the uniform step bit for bit
    st_c, tk_c = st_b.clone(), tk_b.clone()
    pos = torch.full((B,), P, dtype=torch.int32, device="cuda")
    model.decode_step(B, P, tk_b, st_b, tk_b, workspace=ws)
    model.decode_step_ragged(B, pos, tk_c, st_c, tk_c, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(st_b, st_c) and torch.equal(tk_b, tk_c)


@pytest.mark.parametrize("use_projections,B,fuse", [(True, 300, True), (False, 300, True), (True, 3000, True),
                                                    (True, 3000, False)])
def test_half_state_bf16_weights_match_oracle(srm, orc_mod, use_projections, B, fuse, monkeypatch):
    """bf16 weights with a binary16 cache; the state update in the in-projection's epilogue, and (fuse False: the
    library's switch for it) as a kernel of its own."""
    if not fuse:
        monkeypatch.setenv("SRM_FUSE_MIXER", "0")
    cfg = srm_synth.tiny_config(vocab=400, d_model=512, n_layers=2, n_heads=4, n_ctx=12, weight_dtype="bf16", seed=62,
                                use_projections=use_projections, state_dtype="fp16")
    w = srm_synth.make_weights(cfg, stress=True)
    T = 8
    toks = srm_synth.make_prompts(cfg, batch=B, length=T)
    rows = sorted({0, 1, B // 2, B - 1})
    ref = orc_mod.Oracle(cfg, w, "f64").recurrent_forward(toks[rows])
    model = srm.Model(cfg, w)
    ws, st = model.new_workspace(B * T), model.new_state(B)
    out = torch.empty(B, dtype=torch.int32, device="cuda")
    lg = torch.empty((B, cfg.vocab), dtype=torch.float32, device="cuda")
    tc = to_dev(toks).t().contiguous()
    print(f"half state bf16 B={B} projections={use_projections}", flush=True)
    for t in range(T):
        model.decode_step(B, t, tc[t], st, out, logits=lg, workspace=ws)
        assert rel_err_rows(lg[rows].cpu().numpy(), ref["logits"][:, t]) <= 2e-2
    st2, tk2 = model.new_state(B), torch.empty(B, dtype=torch.int32, device="cuda")
    model.prefill(to_dev(toks), 1, st2, tk2, workspace=ws)
    torch.cuda.synchronize()
    assert (st.float() - st2.float()).abs().max() <= 2e-2 * st.float().abs().max()
    s_got = st.float().view(cfg.n_layers, B, cfg.d_model)[:, rows].permute(1, 0, 2).cpu().numpy()
    assert np.abs(s_got - ref["state"]).max() <= 2e-2 * np.abs(ref["state"]).max()


def _ln_on_load_case(srm, orc_mod, d, B, fuse_mixer, monkeypatch, dtype="bf16"):
    cfg = srm_synth.tiny_config(vocab=333, d_model=d, n_layers=3, n_heads=4, n_ctx=8, weight_dtype=dtype, seed=91)
    w = srm_synth.make_weights(cfg, stress=True)
    model = srm.Model(cfg, w)
    T = 4
    toks = srm_synth.make_prompts(cfg, batch=B, length=T)
    ref = orc_mod.Oracle(cfg, w, "f64").recurrent_forward(toks)
    if not fuse_mixer:
        monkeypatch.setenv("SRM_FUSE_MIXER", "0")
    tol = 2e-2 if dtype == "bf16" else 1e-4
    res = []
    for on_load in (True, False):
        if not on_load:
            monkeypatch.setenv("SRM_LN_ON_LOAD", "0")
        ws, st = model.new_workspace(B), model.new_state(B)
        out = torch.empty(B, dtype=torch.int32, device="cuda")
        lg = torch.empty((B, cfg.vocab), dtype=torch.float32, device="cuda")
        hd = torch.empty((B, cfg.d_model), dtype=torch.float32, device="cuda")
        tc = to_dev(toks).t().contiguous()
        steps = []
        print(f"LayerNorm on load {dtype} d={d} B={B} fused mixer={fuse_mixer} on_load={on_load}", flush=True)
        for t in range(T):
            model.decode_step(B, t, tc[t], st, out, logits=lg, hidden=hd, workspace=ws)
            steps.append((lg.clone(), out.clone(), hd.clone()))
        torch.cuda.synchronize()
        res.append((steps, st.clone()))
    for t in range(T):
        assert torch.equal(res[0][0][t][0], res[1][0][t][0]) and torch.equal(res[0][0][t][1], res[1][0][t][1])
        assert torch.equal(res[0][0][t][2], res[1][0][t][2])          # the residual stream after the last block
        assert rel_err_rows(res[0][0][t][0].cpu().numpy(), ref["logits"][:, t]) <= tol
        assert rel_err_rows(res[0][0][t][2].cpu().numpy(), ref["hidden"][:, t]) <= tol
    assert torch.equal(res[0][1], res[1][1])


@pytest.mark.parametrize("d,B", [(64, 2), (128, 8), (256, 1), (512, 5), (1024, 8), (1024, 1), (320, 3), (1024, 9)])
@pytest.mark.parametrize("fuse_mixer", [True, False])
def test_layernorm_made_by_the_consuming_gemm_equals_the_separate_kernel(srm, orc_mod, d, B, fuse_mixer, monkeypatch):
    """A handful of samples of a bf16 model: the step without LayerNorm launches (every LayerNorm made by the
    GEMM that consumes it) against the step with them (the library's switch): the same logits, tokens and states
    bit for bit over four steps, and the logits against the oracle."""
    _ln_on_load_case(srm, orc_mod, d, B, fuse_mixer, monkeypatch)


@pytest.mark.parametrize("d,B", [(64, 1), (256, 1), (256, 8), (256, 16), (96, 9), (1024, 16), (1024, 3)])
@pytest.mark.parametrize("fuse_mixer", [True, False])
def test_layernorm_made_by_the_fp32_gemm_equals_the_separate_kernel(srm, orc_mod, d, B, fuse_mixer, monkeypatch):
    """The same comparison for fp32 models, up to the sixteen rows and 1024 columns of the panel."""
    _ln_on_load_case(srm, orc_mod, d, B, fuse_mixer, monkeypatch, "fp32")


@pytest.mark.parametrize("d,B", [(1024, 16), (320, 11)])
def test_layernorm_made_by_the_gemm_up_to_its_last_row_count(srm, orc_mod, d, B, monkeypatch):
    """The same comparison up to the sixteen rows of the panel."""
    test_layernorm_made_by_the_consuming_gemm_equals_the_separate_kernel(srm, orc_mod, d, B, True, monkeypatch)


@pytest.mark.parametrize("d,B", [(1024, 17), (1024, 64), (1024, 65), (768, 50), (320, 33)])
def test_layernorm_made_by_the_in_projection_of_dozens_of_rows(srm, orc_mod, d, B, monkeypatch):
    """The same comparison where only the in-projection normalises, in several row tiles: from seventeen rows to the
    last that fit one round of the chip (64 of 1024 columns), and the first that do not."""
    _ln_on_load_case(srm, orc_mod, d, B, True, monkeypatch)


@pytest.mark.parametrize("d,B,layers", [(256, 9, 3), (256, 100, 3), (512, 33, 2), (512, 700, 2)])
@pytest.mark.parametrize("half_state", [False, True])
def test_token_mixing_in_one_kernel_matches_the_separate_kernels(srm, orc_mod, d, B, layers, half_state, monkeypatch):
    """A dozen to about a thousand rows of a bf16 model: the step whose token mixing is one kernel per layer
    (LayerNorm1 to out-projection, its slabs added by LayerNorm2) against
    the step of separate kernels (the library's switch) over four steps: logits, residual stream and states agree
    to bf16 rounding, both match the oracle, and the one-kernel step is the one the library takes by itself."""
    cfg = srm_synth.tiny_config(vocab=333, d_model=d, n_layers=layers, n_heads=4, n_ctx=8, weight_dtype="bf16", seed=92,
                                state_dtype="fp16" if half_state else "fp32")
    w = srm_synth.make_weights(cfg, stress=True)
    model = srm.Model(cfg, w)
    T = 4
    toks = srm_synth.make_prompts(cfg, batch=B, length=T)
    rows = sorted({0, B // 2, B - 1})
    ref = orc_mod.Oracle(cfg, w, "f64").recurrent_forward(toks[rows])
    res = []
    for mode in ("1", "0", None):
        if mode is None:
            monkeypatch.delenv("SRM_TOKEN_MIX", raising=False)
        else:
            monkeypatch.setenv("SRM_TOKEN_MIX", mode)
        ws, st = model.new_workspace(B), model.new_state(B)
        out = torch.empty(B, dtype=torch.int32, device="cuda")
        lg = torch.empty((B, cfg.vocab), dtype=torch.float32, device="cuda")
        hd = torch.empty((B, cfg.d_model), dtype=torch.float32, device="cuda")
        tc = to_dev(toks).t().contiguous()
        steps = []
        print(f"token mixing in one kernel d={d} B={B} half={half_state} SRM_TOKEN_MIX={mode}", flush=True)
        for t in range(T):
            model.decode_step(B, t, tc[t], st, out, logits=lg, hidden=hd, workspace=ws)
            steps.append((lg.clone(), out.clone(), hd.clone()))
        torch.cuda.synchronize()
        res.append((steps, st.clone()))
    tol = 4e-2 if half_state else 2e-2
    for t in range(T):
        for k in (0, 1):
            assert rel_err_rows(res[k][0][t][0][rows].cpu().numpy(), ref["logits"][:, t]) <= tol
            assert rel_err_rows(res[k][0][t][2][rows].cpu().numpy(), ref["hidden"][:, t]) <= tol
        assert rel_err_rows(res[0][0][t][0].cpu().numpy(), res[1][0][t][0].cpu().numpy()) <= tol
        # the library's own choice at these row counts is the one-kernel step: the same bits
        assert torch.equal(res[0][0][t][0], res[2][0][t][0]) and torch.equal(res[0][0][t][1], res[2][0][t][1])
    assert torch.equal(res[0][1], res[2][1])
    assert (res[0][1].float() - res[1][1].float()).abs().max() <= tol * res[1][1].float().abs().max()
    model.close()


# ---- head layouts: row-only, column-only, combined ("Method", after Eq. 2; Table S0) ------------
@pytest.mark.parametrize("layout,H", [("row", 4), ("column", 4), ("combined", 4), ("row", 1), ("combined", 1),
                                      ("column", 3)])
def test_head_layouts_fp32_all_paths_match_oracle(srm, orc_mod, layout, H):
    d = 96 if H == 3 else 64
    cfg = srm_synth.tiny_config(vocab=300, d_model=d, n_layers=3, n_heads=H, n_ctx=96, seed=71, head_layout=layout)
    cfg = dataclasses.replace(cfg, name=f"{layout}{H}")
    w = srm_synth.make_weights(cfg, stress=True)
    orc = orc_mod.Oracle(cfg, w, "f64")
    model = srm.Model(cfg, w)
    sd = cfg.state_width
    assert model.state_bytes(10) == cfg.n_layers * 10 * sd * 4
    B, P, G = 6, 12, 10
    prompts = srm_synth.make_prompts(cfg, batch=B, length=P)
    ref = orc.greedy(prompts, G, want_logits=True)
    print(f"head layout {layout} H={H}: prefill + generate", flush=True)
    ws = model.new_workspace(B * 80)
    st, tk = model.new_state(B), torch.empty(B, dtype=torch.int32, device="cuda")
    assert st.shape == (cfg.n_layers, B, sd)
    lg = torch.empty((B, cfg.vocab), dtype=torch.float32, device="cuda")
    model.prefill(to_dev(prompts), 1, st, tk, logits=lg, workspace=ws)
    assert rel_err_rows(lg.cpu().numpy(), ref["logits"][:, 0]) <= 1e-4
    out = torch.empty((G - 1, B), dtype=torch.int32, device="cuda")
    first = tk.cpu().numpy().copy()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        model.generate(B, P, G - 1, tk, st, out, workspace=ws)
    side.synchronize()
    got = np.concatenate([first[:, None], out.cpu().numpy().T], axis=1)
    assert check_tokens(got, ref["tokens"], ref["margin"], np.abs(ref["logits"]).max(axis=2)) == 0
    s_ref = ref["state"]                                       # [B][L][sd] after P + G - 1 tokens
    s_got = st.permute(1, 0, 2).cpu().numpy()
    assert np.abs(s_got - s_ref).max() <= 1e-4 * np.abs(s_ref).max()
    # teacher-forced steps (fused mixer epilogue at this size), parallel form, chunked prefill of one long prompt
    T = 80
    toks = srm_synth.make_prompts(cfg, batch=2, length=T)
    rf = orc.recurrent_forward(toks)
    st2 = model.new_state(2)
    o2 = torch.empty(2, dtype=torch.int32, device="cuda")
    l2 = torch.empty((2, cfg.vocab), dtype=torch.float32, device="cuda")
    h2 = torch.empty((2, d), dtype=torch.float32, device="cuda")
    tc = to_dev(toks).t().contiguous()
    for t in range(T):
        model.decode_step(2, t, tc[t], st2, o2, logits=l2, hidden=h2, workspace=ws)
        if t % 9 == 0 or t == T - 1:
            assert rel_err_rows(l2.cpu().numpy(), rf["logits"][:, t]) <= 1e-4
            assert rel_err_rows(h2.cpu().numpy(), rf["hidden"][:, t]) <= 1e-4
    hid = torch.empty((2, T, d), dtype=torch.float32, device="cuda")
    lgp = torch.empty((2, T, cfg.vocab), dtype=torch.float32, device="cuda")
    model.parallel_forward(to_dev(toks), hid, logits=lgp, workspace=ws)
    torch.cuda.synchronize()
    assert rel_err_rows(hid.cpu().numpy().reshape(2 * T, -1), rf["hidden"].reshape(2 * T, -1)) <= 1e-4
    assert rel_err_rows(lgp.cpu().numpy().reshape(2 * T, -1), rf["logits"].reshape(2 * T, -1)) <= 1e-4
    st3, tk3 = model.new_state(2), torch.empty(2, dtype=torch.int32, device="cuda")
    model.prefill(to_dev(toks), 1, st3, tk3, logits=l2, workspace=ws)          # 2 prompts x 80: the chunked scan
    torch.cuda.synchronize()
    assert rel_err_rows(l2.cpu().numpy(), rf["logits"][:, T - 1]) <= 1e-4
    assert (st3 - st2).abs().max() <= 1e-4 * st2.abs().max()
    # ragged prompts and ragged decode
    lens = [5, 80]
    pk = np.concatenate([toks[i, :n] for i, n in enumerate(lens)]).astype(np.int32)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    st4, tk4 = model.new_state(2), torch.empty(2, dtype=torch.int32, device="cuda")
    pos = torch.empty(2, dtype=torch.int32, device="cuda")
    keep = model.prefill_ragged(to_dev(pk), off, st4, tk4, pos=pos, logits=l2, workspace=ws)
    torch.cuda.synchronize()
    del keep
    for b, n in enumerate(lens):
        assert rel_err_rows(l2[b:b + 1].cpu().numpy(), rf["logits"][b:b + 1, n - 1]) <= 1e-4
    pos[1] = -1                                                # row 1 is at the end of the table: idle
    model.decode_step_ragged(2, pos, to_dev(toks[:, 5].copy()), st4, tk4, advance=True, logits=l2, workspace=ws)
    torch.cuda.synchronize()
    assert rel_err_rows(l2[0:1].cpu().numpy(), rf["logits"][0:1, 5]) <= 1e-4
    assert int(pos[0]) == 6 and int(pos[1]) == -1 and int(tk4[1]) == -1


@pytest.mark.parametrize("layout", ["row", "column", "combined"])
@pytest.mark.parametrize("B,fuse", [(40, True), (9000, True), (9000, False)])
def test_head_layouts_bf16_decode_and_prefill_match_oracle(srm, orc_mod, layout, B, fuse, monkeypatch):
    """bf16 weights; the state update in the in-projection's epilogue (small tile, large tile) and, through the
    library's switch, as the separate streaming kernel."""
    if not fuse:
        monkeypatch.setenv("SRM_FUSE_MIXER", "0")
    cfg = srm_synth.tiny_config(vocab=520, d_model=128, n_layers=2, n_heads=4, n_ctx=12, weight_dtype="bf16", seed=72,
                                head_layout=layout)
    w = srm_synth.make_weights(cfg, stress=True)
    T = 7
    toks = srm_synth.make_prompts(cfg, batch=B, length=T)
    rows = sorted({0, 1, B // 2, B - 1})
    ref = orc_mod.Oracle(cfg, w, "f64").recurrent_forward(toks[rows])
    model = srm.Model(cfg, w)
    ws, st = model.new_workspace(B * T if B < 1000 else B), model.new_state(B)
    out = torch.empty(B, dtype=torch.int32, device="cuda")
    lg = torch.empty((B, cfg.vocab), dtype=torch.float32, device="cuda")
    tc = to_dev(toks).t().contiguous()
    print(f"head layout {layout} bf16 B={B}", flush=True)
    for t in range(T):
        model.decode_step(B, t, tc[t], st, out, logits=lg, workspace=ws)
        assert rel_err_rows(lg[rows].cpu().numpy(), ref["logits"][:, t]) <= 2e-2
    s_ref = ref["state"]                                       # [rows][L][sd]
    s_got = st[:, rows].permute(1, 0, 2).cpu().numpy()
    assert np.abs(s_got - s_ref).max() <= 2e-2 * np.abs(s_ref).max()
    st2, tk2 = model.new_state(B), torch.empty(B, dtype=torch.int32, device="cuda")
    model.prefill(to_dev(toks), 1, st2, tk2, workspace=ws)     # in passes when the workspace is one step's
    torch.cuda.synchronize()
    assert (st - st2).abs().max() <= 2e-2 * st.abs().max()
    assert ((tk2 >= 0) & (tk2 < cfg.vocab)).all()


def test_combined_heads_with_half_precision_cache(srm, orc_mod):
    cfg = srm_synth.tiny_config(vocab=300, d_model=64, n_layers=2, n_heads=2, n_ctx=32, seed=73, head_layout="combined",
                                state_dtype="fp16")
    w = srm_synth.make_weights(cfg)
    toks = srm_synth.make_prompts(cfg, batch=4, length=24)
    ref = orc_mod.Oracle(cfg, w, "f64").recurrent_forward(toks)
    model = srm.Model(cfg, w)
    assert model.state_bytes(4) == cfg.n_layers * 4 * 128 * 2
    ws, st = model.new_workspace(4 * 24), model.new_state(4)
    out = torch.empty(4, dtype=torch.int32, device="cuda")
    lg = torch.empty((4, cfg.vocab), dtype=torch.float32, device="cuda")
    tc = to_dev(toks).t().contiguous()
    for t in range(24):
        model.decode_step(4, t, tc[t], st, out, logits=lg, workspace=ws)
        assert rel_err_rows(lg.cpu().numpy(), ref["logits"][:, t]) <= 2e-3
    s_got = st.float().permute(1, 0, 2).cpu().numpy()
    assert np.abs(s_got - ref["state"]).max() <= 2e-3 * np.abs(ref["state"]).max()


def test_head_layout_errors(srm):
    cfg = srm_synth.tiny_config(vocab=64, d_model=64, n_layers=1, n_heads=2, n_ctx=8, head_layout="combined",
                                use_projections=False)
    with pytest.raises(srm.SrmError):
        srm.Model(cfg, srm_synth.make_weights(cfg))            # combined heads need the projections
    cfg = srm_synth.tiny_config(vocab=64, d_model=96, n_layers=1, n_heads=3, n_ctx=8)
    with pytest.raises(srm.SrmError):
        srm.Model(cfg, srm_synth.make_weights(cfg))            # mixed heads: even count
    cfg = srm_synth.tiny_config(vocab=64, d_model=96, n_layers=1, n_heads=3, n_ctx=8, head_layout="row")
    srm.Model(cfg, srm_synth.make_weights(cfg)).close()


# ---- mixer with k filters along the hidden dimension (Eq. 11) ------------------------------------
@pytest.mark.parametrize("H,k", [(1, 4), (2, 3), (1, 8)])
def test_kernel_mixer_fp32_all_paths_match_oracle(srm, orc_mod, H, k):
    d = 64
    cfg = srm_synth.tiny_config(vocab=300, d_model=d, n_layers=3, n_heads=H, n_ctx=96, seed=75, head_layout="column",
                                mixer_kernel=k)
    w = srm_synth.make_weights(cfg, stress=True)
    orc = orc_mod.Oracle(cfg, w, "f64")
    model = srm.Model(cfg, w)
    assert model.state_bytes(10) == cfg.n_layers * 10 * k * d * 4
    B, P, G = 5, 12, 10
    prompts = srm_synth.make_prompts(cfg, batch=B, length=P)
    ref = orc.greedy(prompts, G, want_logits=True)
    print(f"kernel mixer H={H} k={k}: prefill + generate", flush=True)
    ws = model.new_workspace(B * 80)
    st, tk = model.new_state(B), torch.empty(B, dtype=torch.int32, device="cuda")
    lg = torch.empty((B, cfg.vocab), dtype=torch.float32, device="cuda")
    model.prefill(to_dev(prompts), 1, st, tk, logits=lg, workspace=ws)
    assert rel_err_rows(lg.cpu().numpy(), ref["logits"][:, 0]) <= 1e-4
    out = torch.empty((G - 1, B), dtype=torch.int32, device="cuda")
    first = tk.cpu().numpy().copy()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        model.generate(B, P, G - 1, tk, st, out, workspace=ws)
    side.synchronize()
    got = np.concatenate([first[:, None], out.cpu().numpy().T], axis=1)
    assert check_tokens(got, ref["tokens"], ref["margin"], np.abs(ref["logits"]).max(axis=2)) == 0
    s_got = st.permute(1, 0, 2).cpu().numpy()                  # [B][L][k*d], filter-major like the oracle's
    assert np.abs(s_got - ref["state"]).max() <= 1e-4 * np.abs(ref["state"]).max()
    T = 80
    toks = srm_synth.make_prompts(cfg, batch=2, length=T)
    rf = orc.recurrent_forward(toks)
    st2 = model.new_state(2)
    o2 = torch.empty(2, dtype=torch.int32, device="cuda")
    l2 = torch.empty((2, cfg.vocab), dtype=torch.float32, device="cuda")
    tc = to_dev(toks).t().contiguous()
    for t in range(T):
        model.decode_step(2, t, tc[t], st2, o2, logits=l2, workspace=ws)
        if t % 9 == 0 or t == T - 1:
            assert rel_err_rows(l2.cpu().numpy(), rf["logits"][:, t]) <= 1e-4
    hid = torch.empty((2, T, d), dtype=torch.float32, device="cuda")
    lgp = torch.empty((2, T, cfg.vocab), dtype=torch.float32, device="cuda")
    model.parallel_forward(to_dev(toks), hid, logits=lgp, workspace=ws)
    torch.cuda.synchronize()
    assert rel_err_rows(hid.cpu().numpy().reshape(2 * T, -1), rf["hidden"].reshape(2 * T, -1)) <= 1e-4
    assert rel_err_rows(lgp.cpu().numpy().reshape(2 * T, -1), rf["logits"].reshape(2 * T, -1)) <= 1e-4
    st3, tk3 = model.new_state(2), torch.empty(2, dtype=torch.int32, device="cuda")
    model.prefill(to_dev(toks), 1, st3, tk3, logits=l2, workspace=ws)          # the chunked scan
    torch.cuda.synchronize()
    assert rel_err_rows(l2.cpu().numpy(), rf["logits"][:, T - 1]) <= 1e-4
    assert (st3 - st2).abs().max() <= 1e-4 * st2.abs().max()


@pytest.mark.parametrize("B", [40, 5000])
def test_kernel_mixer_bf16_matches_oracle(srm, orc_mod, B):
    cfg = srm_synth.tiny_config(vocab=520, d_model=128, n_layers=2, n_heads=2, n_ctx=12, weight_dtype="bf16", seed=76,
                                head_layout="column", mixer_kernel=4)
    w = srm_synth.make_weights(cfg, stress=True)
    T = 7
    toks = srm_synth.make_prompts(cfg, batch=B, length=T)
    rows = sorted({0, 1, B // 2, B - 1})
    ref = orc_mod.Oracle(cfg, w, "f64").recurrent_forward(toks[rows])
    model = srm.Model(cfg, w)
    ws, st = model.new_workspace(B), model.new_state(B)
    out = torch.empty(B, dtype=torch.int32, device="cuda")
    lg = torch.empty((B, cfg.vocab), dtype=torch.float32, device="cuda")
    tc = to_dev(toks).t().contiguous()
    print(f"kernel mixer bf16 B={B}", flush=True)
    for t in range(T):
        model.decode_step(B, t, tc[t], st, out, logits=lg, workspace=ws)
        assert rel_err_rows(lg[rows].cpu().numpy(), ref["logits"][:, t]) <= 2e-2
    s_got = st[:, rows].permute(1, 0, 2).cpu().numpy()
    assert np.abs(s_got - ref["state"]).max() <= 2e-2 * np.abs(ref["state"]).max()


def test_kernel_mixer_errors(srm):
    cfg = srm_synth.tiny_config(vocab=64, d_model=64, n_layers=1, n_heads=2, n_ctx=8, mixer_kernel=2)
    w = srm_synth.make_weights(dataclasses.replace(cfg, head_layout="column"))
    with pytest.raises(srm.SrmError):
        srm.Model(cfg, w)                                      # needs column-repeat heads
    cfg = dataclasses.replace(cfg, head_layout="column", use_projections=False)
    with pytest.raises(srm.SrmError):
        srm.Model(cfg, w)                                      # needs the projections


@pytest.mark.parametrize("variant", [dict(head_layout="combined"), dict(head_layout="column", mixer_kernel=2),
                                     dict(head_layout="row")])
def test_variants_at_the_large_configuration_shape(srm, orc_mod, variant):
    """C4's shape and batch (the launch configuration bench.py times: 256x256 tiles, the state update in the
    in-projection's epilogue, mixer rows of 2d for the combined / two-filter models): teacher-forced steps
    from a zero state, the oracle on the first and the last row."""
    cfg = dataclasses.replace(srm_synth.CONFIGS["C4"], n_ctx_fixed=64, **variant)
    w = srm_synth.make_weights(cfg)
    B, T = cfg.batch, 4
    toks = srm_synth.make_prompts(cfg, batch=B, length=T)
    rows = [0, B - 1]
    ref = orc_mod.Oracle(cfg, w, "f64").recurrent_forward(toks[rows])
    model = srm.Model(cfg, w)
    assert model.state_bytes(B) == cfg.n_layers * B * cfg.state_width * 4
    ws, st = model.new_workspace(B), model.new_state(B)
    out = torch.empty(B, dtype=torch.int32, device="cuda")
    lg = torch.empty((B, cfg.vocab), dtype=torch.float32, device="cuda")
    tc = to_dev(toks).t().contiguous()
    print(f"large shape, {variant}", flush=True)
    for t in range(T):
        model.decode_step(B, t, tc[t], st, out, logits=lg, workspace=ws)
        assert rel_err_rows(lg[rows].cpu().numpy(), ref["logits"][:, t]) <= 2e-2
    s_got = st[:, rows].permute(1, 0, 2).cpu().numpy()
    assert np.abs(s_got - ref["state"]).max() <= 2e-2 * np.abs(ref["state"]).max()
    assert bool(torch.isfinite(st).all()) and bool(((out >= 0) & (out < cfg.vocab)).all())


@pytest.mark.parametrize("use_projections", [True, False])
def test_matrices_read_ahead_change_no_bits(srm, use_projections, monkeypatch):
    """A bf16 model whose matrices exceed the last-level cache (its head alone): LayerNorm launches carry extra
    work-groups that read the matrices of the next launches, from 24 rows on where the layers have projections.  The rows
    of a step are those of the same step over 16 rows (the GEMMs of both sum alike)."""
    cfg = srm_synth.tiny_config(vocab=530000, d_model=256, n_layers=2, n_heads=4, n_ctx=16, weight_dtype="bf16",
                                use_projections=use_projections, seed=17)
    rng = np.random.default_rng(5)
    model = srm.Model(cfg, srm_synth.make_weights(cfg))
    monkeypatch.setenv("SRM_TOKEN_MIX", "0")
    monkeypatch.setenv("SRM_LN_ON_LOAD", "0")
    n = 16
    for B in (23, 24, 130):
        print(f"read ahead: projections {use_projections}, {B} rows", flush=True)
        tok = to_dev(rng.integers(0, cfg.vocab, B).astype(np.int32))
        state = to_dev(rng.standard_normal((cfg.n_layers, B, cfg.d_model)).astype(np.float32))
        out, hidden = torch.empty(B, dtype=torch.int32, device="cuda"), torch.empty((B, cfg.d_model), device="cuda")
        st = state.clone()
        model.decode_step(B, 7, tok, st, out, hidden=hidden, workspace=model.new_workspace(B))
        out2, hidden2 = torch.empty(n, dtype=torch.int32, device="cuda"), torch.empty((n, cfg.d_model), device="cuda")
        for b0 in (0, B - n):
            st2 = state[:, b0:b0 + n].contiguous()
            model.decode_step(n, 7, tok[b0:b0 + n].contiguous(), st2, out2, hidden=hidden2, workspace=model.new_workspace(n))
            assert torch.equal(hidden[b0:b0 + n], hidden2) and torch.equal(st[:, b0:b0 + n], st2)
            assert torch.equal(out[b0:b0 + n], out2)


@pytest.mark.parametrize("use_projections", [True, False])
@pytest.mark.parametrize("switches", [{}, {"SRM_TOKEN_MIX": "0"}, {"SRM_TOKEN_MIX": "0", "SRM_LN_ON_LOAD": "0"}])
def test_a_step_with_and_without_read_ahead_gives_the_same_bits(srm, use_projections, switches, monkeypatch):
    """The same call with the extra work-groups and without them, in each arrangement of a layer: token mixing in one kernel
    and the in-projection that normalises its rows (LayerNorm2 then names four matrices), separate launches, and from 4096
    rows on the LayerNorm of several rows per wavefront (5003: neither kernel's rows fill its last work-group)."""
    cfg = srm_synth.tiny_config(vocab=530000, d_model=256, n_layers=2, n_heads=4, n_ctx=16, weight_dtype="bf16",
                                use_projections=use_projections, seed=19)
    rng = np.random.default_rng(6)
    model = srm.Model(cfg, srm_synth.make_weights(cfg))
    for name, value in switches.items():
        monkeypatch.setenv(name, value)
    for B in (1, 40, 130, 5003):
        print(f"read ahead on and off: projections {use_projections}, {switches}, {B} rows", flush=True)
        tok = to_dev(rng.integers(0, cfg.vocab, B).astype(np.int32))
        state = to_dev(rng.standard_normal((cfg.n_layers, B, cfg.d_model)).astype(np.float32))
        ws, got = model.new_workspace(B), []
        for switch in ("1", "0"):
            monkeypatch.setenv("SRM_READ_AHEAD", switch)
            out, hidden = torch.empty(B, dtype=torch.int32, device="cuda"), torch.empty((B, cfg.d_model), device="cuda")
            st = state.clone()
            model.decode_step(B, 7, tok, st, out, hidden=hidden, workspace=ws)
            got.append((out, hidden, st))
        assert all(torch.equal(a, b) for a, b in zip(*got))
        assert bool(torch.isfinite(got[0][1]).all())


@pytest.mark.parametrize("d,B", [(128, 51201), (192, 51201), (320, 79005)])
def test_state_update_behind_few_k_tiles_of_the_largest_tile(srm, orc_mod, d, B, monkeypatch):
    """The state update in the epilogue of 256x256 tiles behind two, three and five k tiles, one output tile per work-group
    and several, against the update as a kernel of its own (same bits) and the oracle on the first and the last row."""
    cfg = srm_synth.tiny_config(vocab=64, d_model=d, n_layers=1, n_heads=4, n_ctx=8, weight_dtype="bf16", seed=21)
    w = srm_synth.make_weights(cfg, stress=True)
    model, T = srm.Model(cfg, w), 2
    toks = srm_synth.make_prompts(cfg, batch=B, length=T)
    rows, tc = [0, B - 1], to_dev(toks).t().contiguous()
    ref = orc_mod.Oracle(cfg, w, "f64").recurrent_forward(toks[rows])
    ws, res = model.new_workspace(B), []
    for fuse in ("1", "0"):
        monkeypatch.setenv("SRM_FUSE_MIXER", fuse)
        print(f"state update in the largest tile d={d} B={B} SRM_FUSE_MIXER={fuse}", flush=True)
        st, out = model.new_state(B), torch.empty(B, dtype=torch.int32, device="cuda")
        hidden = torch.empty((B, d), dtype=torch.float32, device="cuda")
        lg = torch.empty((B, cfg.vocab), dtype=torch.float32, device="cuda")
        for t in range(T):
            model.decode_step(B, t, tc[t], st, out, logits=lg, hidden=hidden, workspace=ws)
            assert rel_err_rows(lg[rows].cpu().numpy(), ref["logits"][:, t]) <= 2e-2
        res.append((st, out, hidden))
    assert all(torch.equal(a, b) for a, b in zip(*res))
