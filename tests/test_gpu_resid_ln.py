"""LayerNorm made by the projections that add to the residual stream (many rows of a bf16 model, the 256x256 persistent tile) against
the LayerNorm launches (the library's switch) and the oracle."""
import numpy as np
import pytest
import torch

import srm_synth
from gpu_util import to_dev, rel_err_rows, kernel_launches

pytestmark = pytest.mark.gpu
SWITCH = "SRM_LN_ON_LOAD"


@pytest.fixture(scope="module")
def srm():
    import paper_2605_08696_amd as pkg
    pkg.lib()
    return pkg


@pytest.fixture(scope="module")
def orc_mod(oracle_mod):
    return oracle_mod




# column tiles of a row: four, three, two; a last row tile of one row, of a part, whole; several rounds of the chip
@pytest.mark.parametrize("d,B,variant", [(1024, 12801, {}), (1024, 32768, dict(state_dtype="fp16")), (768, 17300, {}), (512, 25700, {}),
                                         (1024, 16384, dict(head_layout="combined"))])
def test_decode_with_the_layernorm_in_the_residual_epilogue(srm, orc_mod, d, B, variant, monkeypatch):
    cfg = srm_synth.tiny_config(vocab=260, d_model=d, n_layers=2, n_heads=4, n_ctx=8, weight_dtype="bf16", seed=91, **variant)
    w = srm_synth.make_weights(cfg, stress=True)
    for y in w["layers"]:                            # rows far from a mean of zero, and wide ones
        y["b_out"] = y["b_out"] + np.linspace(-2.0, 6.0, d).astype(np.float32)
    model = srm.Model(cfg, w)
    toks = srm_synth.make_prompts(cfg, batch=B, length=2)
    some = [0, 255, 256, B // 2, B - 2, B - 1]
    ref = orc_mod.Oracle(cfg, w, "f64").recurrent_forward(toks[some])
    tc, ws = to_dev(toks).t().contiguous(), model.new_workspace(B)

    def steps():
        st, out = model.new_state(B), torch.empty(B, dtype=torch.int32, device="cuda")
        res = []
        for t in range(2):
            lg, hd = torch.empty((B, cfg.vocab), device="cuda"), torch.empty((B, d), device="cuda")
            model.decode_step(B, t, tc[t], st, out, logits=lg, hidden=hd, workspace=ws)
            res += [lg, hd]
        torch.cuda.synchronize()
        return res + [st]

    print(f"LayerNorm in the residual epilogue d={d} B={B} {variant}", flush=True)
    ws.random_(0, 256)
    one = steps()
    assert kernel_launches("gemm_bf16_persist_kernel", steps) > 0
    again = steps()
    assert all(torch.equal(a, b) for a, b in zip(one, again))
    # nobody waits: what each work-group has not made is made by the last of its rows', the same bits
    monkeypatch.setenv("SRM_ONE_KERNEL_POLLS", "0")
    hurried = steps()
    monkeypatch.delenv("SRM_ONE_KERNEL_POLLS")
    assert all(torch.equal(a, b) for a, b in zip(one, hurried))
    monkeypatch.setenv(SWITCH, "0")
    many = steps()
    monkeypatch.delenv(SWITCH)
    assert not all(torch.equal(a, b) for a, b in zip(one, many))      # (another order of the sums: the epilogue is what ran)
    tol = 4e-2 if cfg.state_dtype == "fp16" else 2e-2
    for t in range(2):
        for k, name in ((0, "logits"), (1, "hidden")):
            assert rel_err_rows(one[2 * t + k][some].cpu().numpy(), ref[name][:, t]) <= tol
            assert rel_err_rows(one[2 * t + k].cpu().numpy(), many[2 * t + k].cpu().numpy()) <= tol
    # no further from 64 bits than the launches: the error of the normalised rows is the rounding to bf16
    err = [np.sqrt(np.mean((r[3][some].double().cpu().numpy() - ref["hidden"][:, 1]) ** 2)) for r in (one, many)]
    assert err[0] <= 1.25 * err[1]
    model.close()


def test_streams_with_a_cu_mask_and_captured_ones(srm, monkeypatch):
    """On a stream that keeps off some CUs the tiles of a row may not run side by side, so the LayerNorm launches stay; a captured
    step makes the LayerNorm in the epilogue as an eager one does, in every replay."""
    import ctypes
    cfg = srm_synth.tiny_config(vocab=260, d_model=1024, n_layers=2, n_heads=4, n_ctx=8, weight_dtype="bf16", seed=94)
    model, B = srm.Model(cfg, srm_synth.make_weights(cfg, stress=True)), 13000
    tok, ws = to_dev((np.arange(B) % cfg.vocab).astype(np.int32)), model.new_workspace(B)
    state, out, lg = model.new_state(B), torch.empty(B, dtype=torch.int32, device="cuda"), torch.empty((B, cfg.vocab), device="cuda")

    def step(stream=None):
        state.zero_()
        torch.cuda.synchronize()
        model.decode_step(B, 1, tok, state, out, logits=lg, workspace=ws, stream=stream)
        torch.cuda.synchronize()
        return out.clone(), state.clone(), lg.clone()

    one = step()
    monkeypatch.setenv(SWITCH, "0")
    many = step()
    monkeypatch.delenv(SWITCH)
    assert not torch.equal(one[2], many[2])
    hip = ctypes.CDLL("libamdhip64.so")
    handle, mask = ctypes.c_void_p(), (ctypes.c_uint32 * 8)(*[0xffffffff] * 4)
    assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(handle), 8, mask) == 0
    print("many rows on a stream of 128 CUs", flush=True)
    got = step(torch.cuda.ExternalStream(handle.value))
    assert hip.hipStreamDestroy(handle) == 0
    assert all(torch.equal(a, b) for a, b in zip(got, many))

    print("many rows, captured", flush=True)
    graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=stream):
        model.decode_step(B, 1, tok, state, out, logits=lg, workspace=ws, stream=stream)
    for _ in range(3):
        for x in (state, out, lg):
            x.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip((out, state, lg), one))
        assert all(torch.equal(a, b) for a, b in zip(step(), one))
    model.close()


@pytest.mark.parametrize("d,B,fused", [(1024, 16384, True), (1024, 27000, False), (1024, 27300, True), (1024, 32768, True), (768, 17300, True),
                                       (768, 38000, False), (512, 53000, False), (512, 53300, True)])
def test_tiles_of_a_row_in_one_round_of_the_chip(srm, d, B, fused, monkeypatch):
    """More tiles than fit the device at once: where those of a row are not all of one round the LayerNorm launches stay."""
    cfg = srm_synth.tiny_config(vocab=260, d_model=d, n_layers=1, n_heads=4, n_ctx=4, weight_dtype="bf16", seed=96)
    model = srm.Model(cfg, srm_synth.make_weights(cfg, stress=True))
    tok, ws = to_dev((np.arange(B) % cfg.vocab).astype(np.int32)), model.new_workspace(B)

    def step():
        st, out, hid = model.new_state(B), torch.empty(B, dtype=torch.int32, device="cuda"), torch.empty((B, d), device="cuda")
        model.decode_step(B, 0, tok, st, out, hidden=hid, workspace=ws)
        torch.cuda.synchronize()
        return hid

    print(f"rounds of the chip d={d} B={B}", flush=True)
    one = step()
    monkeypatch.setenv(SWITCH, "0")
    many = step()
    assert torch.equal(one, many) != fused
    assert rel_err_rows(one.cpu().numpy(), many.cpu().numpy()) <= 2e-2
    model.close()


def test_several_streams_at_once(srm):
    """Steps of as many rows as fill the device on three streams at once: work-groups that find a tile of their rows not even begun
    leave theirs to the last, with the bits of a step alone."""
    cfg = srm_synth.tiny_config(vocab=260, d_model=1024, n_layers=4, n_heads=4, n_ctx=8, weight_dtype="bf16", seed=95)
    model, B, n, T = srm.Model(cfg, srm_synth.make_weights(cfg, stress=True)), 16384, 3, 4
    tok = to_dev((np.arange(B) % cfg.vocab).astype(np.int32))
    ws, streams = [model.new_workspace(B) for _ in range(n)], [torch.cuda.Stream() for _ in range(n)]

    def fresh():
        return model.new_state(B), torch.empty(B, dtype=torch.int32, device="cuda"), torch.empty((B, 1024), device="cuda")

    def steps(i, st, out, hid):
        for t in range(T):
            model.decode_step(B, t, tok, st, out, hidden=hid, workspace=ws[i], stream=streams[i])

    alone, sets = fresh(), [fresh() for _ in range(n)]
    torch.cuda.synchronize()
    steps(0, *alone)
    torch.cuda.synchronize()
    print("many rows on three streams at once", flush=True)
    for s in streams:
        with torch.cuda.stream(s):
            torch.cuda._sleep(20_000_000)
    for i in range(n):
        steps(i, *sets[i])
    torch.cuda.synchronize()
    for got in sets:
        assert all(torch.equal(a, b) for a, b in zip(got, alone))
    model.close()


def test_prefill_and_sequence_form_with_the_layernorm_in_the_residual_epilogue(srm, monkeypatch):
    """Prompts in one pass and in several, and the sequence form, against the LayerNorm launches."""
    cfg = srm_synth.tiny_config(vocab=260, d_model=1024, n_layers=3, n_heads=4, n_ctx=70, weight_dtype="bf16", seed=92)
    model = srm.Model(cfg, srm_synth.make_weights(cfg, stress=True))
    N, P = 420, 64
    toks = to_dev(srm_synth.make_prompts(cfg, batch=N, length=P))

    def run(rows):
        st, tk = model.new_state(N), torch.empty(N, dtype=torch.int32, device="cuda")
        lg, hid = torch.empty((N, cfg.vocab), device="cuda"), torch.empty((N, P, 1024), device="cuda")
        model.prefill(toks, 1, st, tk, logits=lg, workspace=model.new_workspace(rows))
        model.parallel_forward(toks, hid, workspace=model.new_workspace(rows))
        torch.cuda.synchronize()
        return st, lg, hid.view(N * P, 1024)

    print("prefill and sequence form", flush=True)
    one, two = run(N * P), run(N * P // 2)
    monkeypatch.setenv(SWITCH, "0")
    many = run(N * P)
    assert not torch.equal(one[2], many[2])
    for got in (one, two):
        assert (got[0] - many[0]).abs().max() <= 2e-2 * many[0].abs().max()
        assert rel_err_rows(got[1].cpu().numpy(), many[1].cpu().numpy()) <= 2e-2
        assert float((got[2] - many[2]).norm() / many[2].norm()) <= 2e-2
    model.close()


@pytest.mark.parametrize("ragged", [False, True])
def test_prefill_whose_last_rows_are_as_many(srm, ragged, monkeypatch):
    """The last layer goes on with the prompts' last rows, so many that its projections make the LayerNorm too, in other row tiles than
    the layers in front of it."""
    cfg = srm_synth.tiny_config(vocab=260, d_model=1024, n_layers=2, n_heads=4, n_ctx=8, weight_dtype="bf16", seed=93)
    model = srm.Model(cfg, srm_synth.make_weights(cfg, stress=True))
    N, P = 16300, 2
    toks = to_dev(srm_synth.make_prompts(cfg, batch=N, length=P))

    def run():
        st, tk = model.new_state(N), torch.empty(N, dtype=torch.int32, device="cuda")
        lg, ws = torch.empty((N, cfg.vocab), device="cuda"), model.new_workspace(N * P)
        ws.random_(0, 256)
        if ragged:
            model.prefill_ragged(toks.reshape(-1), np.arange(0, N * P + 1, P, dtype=np.int32), st, tk, logits=lg, workspace=ws)
        else:
            model.prefill(toks, 1, st, tk, logits=lg, workspace=ws)
        torch.cuda.synchronize()
        return st, lg

    print(f"last rows, ragged={ragged}", flush=True)
    one, again = run(), run()
    assert kernel_launches("last_rows_kernel", run) > 0
    assert all(torch.equal(a, b) for a, b in zip(one, again))
    monkeypatch.setenv(SWITCH, "0")
    many = run()
    assert not torch.equal(one[1], many[1])
    assert (one[0] - many[0]).abs().max() <= 2e-2 * many[0].abs().max()
    assert rel_err_rows(one[1].cpu().numpy(), many[1].cpu().numpy()) <= 2e-2
    model.close()
