"""Prefill whose last layer continues on each prompt's last row alone: on both sides of the rules for the shortest prompt and
for the rows (512 beyond the last ones, at this width), one pass or several, against the oracle."""
import dataclasses

import numpy as np
import pytest
import torch

import srm_synth
from gpu_util import to_dev, rel_err_rows, kernel_launches

pytestmark = pytest.mark.gpu

MODELS = {"tiny": {}, "narrow mlp": dict(mlp_expansion=1), "bare": dict(use_projections=False),
          "combined": dict(head_layout="combined"), "one layer": dict(n_layers=1)}


@pytest.fixture(scope="module")
def srm():
    import paper_2605_08696_amd as pkg
    pkg.lib()
    return pkg


@pytest.mark.parametrize("lens", [[1, 600], [2, 520, 2], [3, 3, 530, 4], [4, 256, 258], [171] * 3, [513], [512]], ids=str)
@pytest.mark.parametrize("name", list(MODELS))
def test_prefill_of_the_last_rows_matches_oracle(srm, oracle_mod, name, lens):
    cfg = srm_synth.tiny_config(vocab=301, d_model=256, n_layers=2, n_heads=4, n_ctx=600, weight_dtype="fp32", seed=31)
    cfg = dataclasses.replace(cfg, **MODELS[name])
    w = srm_synth.make_weights(cfg)
    model, orc = srm.Model(cfg, w), oracle_mod.Oracle(cfg, w, "f64")
    N, rows = len(lens), sum(lens)
    rng = np.random.default_rng(rows)
    prompts = rng.integers(0, cfg.vocab, (N, max(lens))).astype(np.int32)
    toks = to_dev(np.concatenate([prompts[i, :n] for i, n in enumerate(lens)]))
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    uniform = len(set(lens)) == 1
    print(f"prefill of last rows {name} lens={lens}", flush=True)
    got = []
    for how in ["packed", "passes"] + ["uniform"] * uniform:
        room = max(lens) + 1 if how == "passes" else rows
        n = model.workspace_bytes(room)
        if srm.prefill_ragged_plan(cfg, off, n)["chunk_len"] != srm.prefill_ragged_plan(cfg, off, 1 << 40)["chunk_len"]:
            continue                                   # passes too small for the chunked scan's sums: another mixer's rounding
        buf = torch.randint(0, 256, (n + 4096,), dtype=torch.uint8, device="cuda")
        guard = buf[n:].clone()
        st, tk = model.new_state(N), torch.empty(N, dtype=torch.int32, device="cuda")
        lg = torch.empty((N, cfg.vocab), dtype=torch.float32, device="cuda")
        if how == "uniform":
            keep = model.prefill(toks.view(N, -1), 1, st, tk, logits=lg, workspace=buf[:n])
        else:
            keep = model.prefill_ragged(toks, off, st, tk, logits=lg, workspace=buf[:n])
        torch.cuda.synchronize()
        del keep
        assert torch.equal(buf[n:], guard)
        got.append((lg, st, tk))
    sv = got[0][1].view(cfg.n_layers, N, -1)
    for b, n in enumerate(lens):
        ref = orc.greedy(prompts[b:b + 1, :n], 1, want_logits=True)
        # fp32 sums of at most 1024 products against double ones: the repository's bound for fp32 models
        assert rel_err_rows(got[0][0][b:b + 1].cpu().numpy(), ref["logits"][:, 0]) <= 1e-4
        assert np.abs(sv[:, b].cpu().numpy() - ref["state"][0]).max() <= 1e-4 * np.abs(ref["state"][0]).max()
    for other in got[1:]:
        for x, y in zip(got[0], other):
            assert torch.equal(x, y)


@pytest.mark.parametrize("lens", [[3, 530, 4], [513], [512], [258] * 3, [2, 560], [1, 580]], ids=str)
@pytest.mark.parametrize("name,d", [("tiny", 256), ("bare", 256), ("combined", 256), ("narrow mlp", 512)])
def test_prefill_of_the_last_rows_bf16(srm, oracle_mod, name, d, lens):
    """The same in bf16, whose rows are half as wide in memory as the residual stream's: packed and uniform prompts against the
    oracle within the repository's bound for bf16 models, and whether the last rows are gathered."""
    cfg = srm_synth.tiny_config(vocab=301, d_model=d, n_layers=2, n_heads=4, n_ctx=600, weight_dtype="bf16", seed=31)
    cfg = dataclasses.replace(cfg, **MODELS[name])
    N, rows = len(lens), sum(lens)
    w = srm_synth.make_weights(cfg)
    model, orc = srm.Model(cfg, w), oracle_mod.Oracle(cfg, w, "f64")
    prompts = np.random.default_rng(rows).integers(0, cfg.vocab, (N, max(lens))).astype(np.int32)
    toks = to_dev(np.concatenate([prompts[i, :n] for i, n in enumerate(lens)]))
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    n, ff = model.workspace_bytes(rows), cfg.mlp_expansion * d
    gathered = (rows - N) * d >= 1 << 17 and (ff + model.sd) * 2 + 4 * d + 512 <= min(lens) * ff * 2       # enough to save, and room
    for how in ["packed"] + ["uniform"] * (len(set(lens)) == 1):
        buf = torch.randint(0, 256, (n + 4096,), dtype=torch.uint8, device="cuda")
        guard = buf[n:].clone()
        st, tk = model.new_state(N), torch.empty(N, dtype=torch.int32, device="cuda")
        lg = torch.empty((N, cfg.vocab), dtype=torch.float32, device="cuda")
        print(f"bf16 prefill of last rows {name} d={d} lens={lens} {how}", flush=True)
        keep = []

        def prefill():
            if how == "uniform":
                model.prefill(toks.view(N, -1), 1, st, tk, logits=lg, workspace=buf[:n])
            else:
                keep.append(model.prefill_ragged(toks, off, st, tk, logits=lg, workspace=buf[:n]))

        assert kernel_launches("last_rows_kernel", prefill) == gathered
        assert torch.equal(buf[n:], guard)
        sv = st.view(cfg.n_layers, N, -1)
        for b, m in enumerate(lens):
            ref = orc.greedy(prompts[b:b + 1, :m], 1, want_logits=True)
            assert rel_err_rows(lg[b:b + 1].cpu().numpy(), ref["logits"][:, 0]) <= 2e-2
            assert np.abs(sv[:, b].cpu().numpy() - ref["state"][0]).max() <= 2e-2 * np.abs(ref["state"][0]).max()
        assert torch.equal(tk.long(), lg.argmax(dim=1))
    model.close()


@pytest.mark.parametrize("N,P", [(1, 64), (1, 65), (1, 257), (2, 320), (1, 321), (1, 512), (1, 513), (1, 580), (20, 64), (40, 321)])
def test_block_scan_bf16_of_few_and_many_blocks(srm, oracle_mod, N, P):
    """The block form of the mixer on both sides of one block per CU (20 x 64 positions: 80 blocks here, 40 x 321: 960) and at the
    ends of its requests of 256 and 512 rows: prefill and sequence form of a bf16 model against the oracle (the repository's
    bound for bf16 models)."""
    cfg = srm_synth.tiny_config(vocab=300, d_model=128, n_layers=2, n_heads=4, n_ctx=600, weight_dtype="bf16", seed=13)
    w = srm_synth.make_weights(cfg)
    model, orc = srm.Model(cfg, w), oracle_mod.Oracle(cfg, w, "f64")
    prompts = np.random.default_rng(P).integers(0, cfg.vocab, (N, P)).astype(np.int32)
    ws = model.new_workspace(N * P)
    st, tk = model.new_state(N), torch.empty(N, dtype=torch.int32, device="cuda")
    hid = torch.empty((N, P, cfg.d_model), dtype=torch.float32, device="cuda")
    print(f"block scan bf16 N={N} P={P}", flush=True)
    model.prefill(to_dev(prompts), 1, st, tk, workspace=ws)
    model.parallel_forward(to_dev(prompts), hid, workspace=ws)
    torch.cuda.synchronize()
    sv = st.view(cfg.n_layers, N, cfg.d_model).cpu().numpy()
    for b in sorted({0, N // 2, N - 1}):
        ref = orc.greedy(prompts[b:b + 1], 1, want_logits=True)
        assert np.abs(sv[:, b] - ref["state"][0]).max() <= 2e-2 * np.abs(ref["state"][0]).max()
        want = orc.parallel_forward(prompts[b:b + 1])["hidden"]
        assert np.abs(hid[b:b + 1].cpu().numpy() - want).max() <= 2e-2 * np.abs(want).max()
