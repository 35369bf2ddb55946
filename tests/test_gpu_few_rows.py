"""Decode steps of a handful of samples as one kernel (a bf16 model of 512 or 1024 channels, an fp32 one of 256) against the
oracle and against the step kernels (the library's switch)."""
import dataclasses

import numpy as np
import pytest
import torch

import srm_synth
from gpu_util import to_dev, rel_err_rows, check_tokens, kernel_events, kernel_launches, kernel_grids

pytestmark = pytest.mark.gpu
SWITCH = "SRM_ONE_KERNEL_STEP"


@pytest.fixture(scope="module")
def srm():
    import paper_2605_08696_amd as pkg
    pkg.lib()
    return pkg


@pytest.fixture(scope="module")
def orc_mod(oracle_mod):
    return oracle_mod


def _launches(fn):
    """How often the kernels of few.hpp run in fn()."""
    return kernel_launches("few_rows_kernel", fn)


def _steps(model, cfg, B, T, toks, garbage=None, **how):
    """T steps on given tokens in a workspace full of `garbage`, with a guard behind it."""
    n = model.workspace_bytes(B)
    buf = torch.empty(n + 4096, dtype=torch.uint8, device="cuda")
    buf.random_(0, 256) if garbage is None else buf.fill_(garbage)
    guard = buf[n:].clone()
    st, out = model.new_state(B), torch.empty(B, dtype=torch.int32, device="cuda")
    lg = torch.empty((B, cfg.vocab), dtype=torch.float32, device="cuda")
    hd = torch.empty((B, cfg.d_model), dtype=torch.float32, device="cuda")
    tc = to_dev(toks).t().contiguous()
    res = []
    for t in range(T):
        model.decode_step(B, t, tc[t], st, out, logits=lg, hidden=hd, workspace=buf[:n], **how)
        res.append((lg.clone(), hd.clone(), out.clone()))
    torch.cuda.synchronize()
    assert torch.equal(buf[n:], guard)
    return res, st


CASES = [("bf16", 1024, 1, {}), ("bf16", 1024, 3, dict(state_dtype="fp16")), ("bf16", 1024, 4, dict(head_layout="row", n_heads=1)),
         ("bf16", 512, 1, dict(state_dtype="fp16")), ("bf16", 512, 2, dict(head_layout="column")), ("bf16", 512, 4, {}),
         ("bf16", 1024, 2, dict(use_projections=False)), ("bf16", 512, 3, dict(use_projections=False, state_dtype="fp16")),
         ("fp32", 256, 1, {}), ("fp32", 256, 5, dict(state_dtype="fp16")), ("fp32", 256, 8, {})]


@pytest.mark.parametrize("dtype,d,B,variant", CASES)
@pytest.mark.parametrize("vocab", [333, 1400])
def test_one_kernel_step_matches_oracle_and_step_kernels(srm, orc_mod, dtype, d, B, variant, vocab, monkeypatch):
    """Rows below, at and above the ones that the kernel is unrolled for; vocabularies that are no multiple of four and leave
    work-groups without columns, or with several groups of them; garbage of two kinds in the workspace."""
    kw = dict(vocab=vocab, d_model=d, n_layers=6, n_heads=4, n_ctx=12, weight_dtype=dtype, seed=53)
    kw.update(variant)
    cfg = srm_synth.tiny_config(**kw)
    w = srm_synth.make_weights(cfg, stress=True)
    model = srm.Model(cfg, w)
    T = 4
    toks = srm_synth.make_prompts(cfg, batch=B, length=T)
    ref = orc_mod.Oracle(cfg, w, "f64").recurrent_forward(toks)
    print(f"one-kernel step {dtype} d={d} B={B} V={vocab} {variant}", flush=True)
    runs = {}
    assert _launches(lambda: runs.update(one=_steps(model, cfg, B, T, toks))) == T
    one, st = runs["one"]
    again, st2 = _steps(model, cfg, B, T, toks, garbage=0)
    monkeypatch.setenv(SWITCH, "0")
    assert _launches(lambda: runs.update(many=_steps(model, cfg, B, T, toks))) == 0
    many, st3 = runs["many"]
    half = cfg.state_dtype == "fp16"
    tol = (4e-2 if half else 2e-2) if dtype == "bf16" else (1e-3 if half else 1e-4)
    for t in range(T):
        assert all(torch.equal(a, b) for a, b in zip(one[t], again[t]))         # a fixed order of sums: the same bits
        assert rel_err_rows(one[t][0].cpu().numpy(), ref["logits"][:, t]) <= tol
        assert rel_err_rows(one[t][1].cpu().numpy(), ref["hidden"][:, t]) <= tol
        assert rel_err_rows(one[t][0].cpu().numpy(), many[t][0].cpu().numpy()) <= tol
        assert torch.equal(one[t][2].long(), one[t][0].argmax(dim=1))
    assert torch.equal(st, st2)
    assert (st.float() - st3.float()).abs().max() <= tol * st3.float().abs().max()
    s_got = st.float().view(cfg.n_layers, B, cfg.d_model).permute(1, 0, 2).cpu().numpy()
    s_ref = orc_mod.Oracle(cfg, w, "f64").greedy(toks, 1)["state"]
    assert np.abs(s_got - s_ref).max() <= tol * np.abs(s_ref).max()
    model.close()


@pytest.mark.parametrize("B,half", [(1, False), (3, False), (8, False), (8, True)])
def test_generation_in_one_kernel_matches_oracle(srm, orc_mod, B, half):
    """Many steps of one launch, greedy and sampled, tokens exact, twice in the same workspace."""
    cfg = dataclasses.replace(srm_synth.CONFIGS["C1"], state_dtype="fp16" if half else "fp32")
    w = srm_synth.make_weights(cfg)
    w["head"] = w["head"] * 25.0
    prompts = srm_synth.make_prompts(cfg)[:B]
    P, G = prompts.shape[1], 30
    model = srm.Model(cfg, w)
    orc = orc_mod.Oracle(cfg, w, "f64")
    ws = model.new_workspace(B * P)
    for temperature in (0.0, 0.7):
        kw = {"temperature": temperature, "seed": 7} if temperature else {}
        ref = orc.greedy(prompts, G, want_logits=True, **kw)
        dp = to_dev(prompts)
        for _ in range(2):
            st, tk = model.new_state(B), torch.empty(B, dtype=torch.int32, device="cuda")
            model.prefill(dp[:, :P - 1].contiguous(), 1, st, tk, workspace=ws)
            tk.copy_(dp[:, P - 1])
            out = torch.full((G, B), -7, dtype=torch.int32, device="cuda")
            print(f"generation in one kernel B={B} half={half} T={temperature}", flush=True)
            assert _launches(lambda: model.generate(B, P - 1, G, tk, st, out, workspace=ws, **kw)) == 1
            got = out.cpu().numpy().T
            ties = check_tokens(got, ref["tokens"], ref["margin"], np.abs(ref["logits"]).max(axis=2), rtol=1e-3 if half else 1e-4)
            assert (tk.cpu().numpy() == got[:, -1]).all()
            if not half:
                assert ties == 0
                s_got = st.view(cfg.n_layers, B, cfg.d_model).permute(1, 0, 2).cpu().numpy()
                assert np.abs(s_got - ref["state"]).max() <= 1e-4 * np.abs(ref["state"]).max()


@pytest.mark.parametrize("temperature", [0.0, 0.8])
@pytest.mark.parametrize("d,B,layers,half", [(512, 1, 5, False), (512, 3, 7, True), (1024, 2, 7, False), (1024, 4, 6, False), (1024, 4, 5, True)])
def test_bf16_generation_in_one_kernel_matches_oracle(srm, orc_mod, d, B, layers, half, temperature):
    """Tokens and state carried from step to step of one launch, the LayerNorm buffers across odd numbers of layers, sampling
    between steps: every token is the oracle's choice from its logits on the same tokens, or within the bf16 bound of it, and
    so is the state behind the last."""
    cfg = srm_synth.tiny_config(vocab=333, d_model=d, n_layers=layers, n_heads=4, n_ctx=40, weight_dtype="bf16", seed=71,
                                state_dtype="fp16" if half else "fp32")
    w = srm_synth.make_weights(cfg, stress=True)
    model, G = srm.Model(cfg, w), 12
    start = (np.arange(B) * 29 + 5).astype(np.int32)
    st, ws, tk = model.new_state(B), model.new_workspace(B), to_dev(start)
    out = torch.full((G, B), -7, dtype=torch.int32, device="cuda")
    kw = {"temperature": temperature, "seed": 9} if temperature else {}
    print(f"bf16 generation in one kernel d={d} B={B} layers={layers} half={half} T={temperature}", flush=True)
    assert _launches(lambda: model.generate(B, 0, G, tk, st, out, workspace=ws, **kw)) == 1
    got = out.cpu().numpy().T
    assert (tk.cpu().numpy() == got[:, -1]).all() and (got >= 0).all() and (got < cfg.vocab).all()
    fed = np.concatenate([start[:, None], got[:, :-1]], axis=1)
    orc = orc_mod.Oracle(cfg, w, "f64")
    logits = orc.recurrent_forward(fed)["logits"]
    tol = 4e-2 if half else 2e-2                       # the repository's bounds of bf16 logits, of the largest of a row
    for b in range(B):
        for g in range(G):
            row = logits[b, g].astype(np.float64)
            score = row + temperature * np.array([orc_mod.gumbel(9, g, b, v) if temperature else 0.0 for v in range(cfg.vocab)])
            assert score.max() - score[got[b, g]] <= 2 * tol * np.abs(row).max(), (b, g)
    ref = orc.greedy(fed, 1)["state"]
    s_got = st.float().view(layers, B, d).permute(1, 0, 2).cpu().numpy()
    assert np.abs(s_got - ref).max() <= tol * np.abs(ref).max()
    model.close()


def test_sampled_and_nucleus_steps_choose_from_their_own_logits(srm, orc_mod):
    cfg = srm_synth.tiny_config(vocab=1001, d_model=512, n_layers=6, n_heads=4, n_ctx=16, weight_dtype="bf16", seed=31)
    w = srm_synth.make_weights(cfg, stress=True)
    w["head"] = srm_synth.round_to_bf16(w["head"] * 30.0)
    model = srm.Model(cfg, w)
    B, T, seed, pos = 4, 0.8, 5, 3
    tok = to_dev(np.arange(B, dtype=np.int32) * 7)
    st, out = model.new_state(B), torch.empty(B, dtype=torch.int32, device="cuda")
    lg = torch.empty((B, cfg.vocab), dtype=torch.float32, device="cuda")
    ws = model.new_workspace(B)
    for top_p in (None, 0.5):
        for s in range(seed, seed + 6):
            model.decode_step(B, pos, tok, st, out, logits=lg, workspace=ws, temperature=T, seed=s, top_p=top_p)
            got, L = out.cpu().numpy(), lg.cpu().numpy().astype(np.float64)
            for b in range(B):
                want = (orc_mod.pick(L[b], T, s, pos, b) if top_p is None else orc_mod.pick_topp(L[b], T, top_p, s, pos, b))
                assert got[b] == want


@pytest.mark.parametrize("dtype,d,B,variant", CASES)
def test_one_work_group_alone_gives_the_same_bits(srm, dtype, d, B, variant, monkeypatch):
    """A launch whose work-groups have not all started is done by one of them.  Forced from the host, first by an arrival that
    is withdrawn from the start, then by a wait of one look, which ends either way."""
    kw = dict(vocab=1001, d_model=d, n_layers=6, n_heads=4, n_ctx=12, weight_dtype=dtype, seed=59)
    kw.update(variant)
    cfg = srm_synth.tiny_config(**kw)
    model = srm.Model(cfg, srm_synth.make_weights(cfg, stress=True))
    toks = srm_synth.make_prompts(cfg, batch=B, length=3)
    for how in (dict(), dict(temperature=0.8, seed=3)):
        want, st = _steps(model, cfg, B, 3, toks, **how)
        for mode in ("2", "3"):
            monkeypatch.setenv(SWITCH, mode)
            print(f"one work-group alone {dtype} d={d} B={B} {variant} mode {mode}", flush=True)
            got, st2 = _steps(model, cfg, B, 3, toks, **how)
            monkeypatch.delenv(SWITCH)
            for a, b in zip(want, got):
                assert all(torch.equal(x, y) for x, y in zip(a, b))
            assert torch.equal(st, st2)
    model.close()


@pytest.mark.parametrize("dtype,d,B", [("fp32", 256, 5), ("bf16", 512, 3), ("bf16", 1024, 2)])
def test_generation_by_one_work_group_alone(srm, dtype, d, B, monkeypatch):
    """All steps of a generate call, their tokens and state carried on, five and seven layers."""
    for layers in (5, 7):
        cfg = srm_synth.tiny_config(vocab=333, d_model=d, n_layers=layers, n_heads=4, n_ctx=40, weight_dtype=dtype, seed=61)
        model = srm.Model(cfg, srm_synth.make_weights(cfg, stress=True))
        G, got = 9, []
        for mode in (None, "2", "3"):
            if mode:
                monkeypatch.setenv(SWITCH, mode)
            st, ws = model.new_state(B), model.new_workspace(B)
            tk, out = to_dev(np.arange(B, dtype=np.int32)), torch.full((G, B), -7, dtype=torch.int32, device="cuda")
            print(f"generation by one work-group alone d={d} layers={layers} mode {mode}", flush=True)
            assert _launches(lambda: model.generate(B, 2, G, tk, st, out, workspace=ws, temperature=0.7, seed=11)) == 1
            got.append((st, tk, out))
        monkeypatch.delenv(SWITCH)
        assert torch.equal(got[0][1], got[0][2][-1]) and (got[0][2] >= 0).all()
        for other in got[1:]:
            assert all(torch.equal(a, b) for a, b in zip(got[0], other))
        model.close()


def test_a_wait_that_gives_up_leaves_marked_tokens(srm, monkeypatch):
    """The bound of the waits behind the arrival, set so short from the host that some give up at once: every wavefront ends,
    the tokens are -1 (behind a nucleus pass too, which takes a negative token for an idle row), and the next call is right."""
    for dtype, d, B, bare in (("bf16", 512, 3, False), ("bf16", 1024, 4, True), ("fp32", 256, 8, False)):
        cfg = srm_synth.tiny_config(vocab=1001, d_model=d, n_layers=6, n_heads=4, n_ctx=16, weight_dtype=dtype, seed=67,
                                    use_projections=not bare)
        model = srm.Model(cfg, srm_synth.make_weights(cfg, stress=True))
        ws, lg = model.new_workspace(B), torch.zeros((B, cfg.vocab), dtype=torch.float32, device="cuda")
        tok = to_dev(np.arange(B, dtype=np.int32) * 7)

        def step(**how):
            st, out = model.new_state(B), torch.full((B,), 5, dtype=torch.int32, device="cuda")
            model.decode_step(B, 1, tok, st, out, logits=lg, workspace=ws, **how)
            torch.cuda.synchronize()
            return out, st, lg.clone()

        def generate():
            st, tk, out = model.new_state(B), tok.clone(), torch.full((4, B), -7, dtype=torch.int32, device="cuda")
            model.generate(B, 1, 4, tk, st, out, workspace=ws)
            torch.cuda.synchronize()
            return tk, out

        ways = (dict(), dict(temperature=0.7, seed=3), dict(temperature=0.7, top_p=0.6, seed=3))
        want = [step(**how) for how in ways]
        monkeypatch.setenv("SRM_ONE_KERNEL_POLLS", "0")
        for how in ways:
            print(f"a wait that gives up {dtype} d={d} B={B} {how}", flush=True)
            assert (step(**how)[0] == -1).all()
        if not bare:
            tk, out = generate()
            assert (tk == -1).all() and (out == -1).any()
        monkeypatch.delenv("SRM_ONE_KERNEL_POLLS")
        for how, w in zip(ways, want):
            assert all(torch.equal(a, b) for a, b in zip(step(**how), w))
        model.close()


def test_which_calls_run_as_one_kernel(srm, monkeypatch):
    """By rows, layers and the switch, and never into a graph that is being captured."""
    cfg = srm_synth.tiny_config(vocab=300, d_model=512, n_layers=6, n_heads=4, n_ctx=16, weight_dtype="bf16", seed=3)
    model = srm.Model(cfg, srm_synth.make_weights(cfg))
    tok, out = torch.zeros(5, dtype=torch.int32, device="cuda"), torch.empty(5, dtype=torch.int32, device="cuda")

    def step(B, ws=None, m=model):
        st = m.new_state(B)
        ws = m.new_workspace(B) if ws is None else ws
        return lambda: m.decode_step(B, 0, tok[:B], st, out[:B], workspace=ws)

    step(1)(), step(5)()
    assert _launches(step(4)) == 1 and _launches(step(3)) == 1 and _launches(step(5)) == 0
    side, st, ws = torch.cuda.Stream(), model.new_state(2), model.new_workspace(2)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        model.decode_step(2, 0, tok[:2], st, out[:2], workspace=ws)
    assert _launches(graph.replay) == 0
    monkeypatch.setenv(SWITCH, "0")
    assert _launches(step(4)) == 0
    monkeypatch.delenv(SWITCH)
    shallow = dataclasses.replace(cfg, n_layers=3)
    other = srm.Model(shallow, srm_synth.make_weights(shallow))
    assert _launches(step(1, m=other)) == 0


def test_stream_that_keeps_off_some_cus_takes_the_step_kernels(srm, orc_mod, monkeypatch):
    """The work-groups wait for each other, and a stream with a CU mask need not have room for all of them: 32 of its CUs hold
    no more than half of 64 work-groups.  The step kernels' results there, bit for bit."""
    import ctypes
    cfg = srm_synth.tiny_config(vocab=300, d_model=512, n_layers=6, n_heads=4, n_ctx=16, weight_dtype="bf16", seed=3)
    model = srm.Model(cfg, srm_synth.make_weights(cfg))
    B = 3
    tok = to_dev(np.arange(B, dtype=np.int32) * 5)
    ws = model.new_workspace(B)

    def step(stream=None):
        st, out = model.new_state(B), torch.empty(B, dtype=torch.int32, device="cuda")
        lg = torch.empty((B, cfg.vocab), dtype=torch.float32, device="cuda")
        torch.cuda.synchronize()
        model.decode_step(B, 0, tok, st, out, logits=lg, workspace=ws, stream=stream)
        torch.cuda.synchronize()
        return lg, out, st

    step()
    assert _launches(step) == 1
    hip = ctypes.CDLL("libamdhip64.so")
    handle, mask = ctypes.c_void_p(), (ctypes.c_uint32 * 8)(0xffffffff)
    assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(handle), 8, mask) == 0
    masked = torch.cuda.ExternalStream(handle.value)
    print("step on a stream of 32 CUs", flush=True)
    assert _launches(lambda: step(masked)) == 0
    got = step(masked)
    monkeypatch.setenv(SWITCH, "0")
    assert all(torch.equal(a, b) for a, b in zip(got, step()))
    assert hip.hipStreamDestroy(handle) == 0


def test_calls_on_several_streams_and_threads(srm):
    """Kernels whose work-groups wait for each other, launched from four threads on four streams into workspaces of their own,
    with two models and other work in between: each stream's results are those of the same calls alone."""
    import threading
    models = []
    for dtype, d in (("bf16", 1024), ("fp32", 256)):
        cfg = srm_synth.tiny_config(vocab=700, d_model=d, n_layers=6, n_heads=4, n_ctx=64, weight_dtype=dtype, seed=23)
        models.append((cfg, srm.Model(cfg, srm_synth.make_weights(cfg))))

    def job(k):
        cfg, model = models[k % 2]
        B = 1 + k
        tok = to_dev((np.arange(B) * 11 + k).astype(np.int32))
        st, ws = model.new_state(B), model.new_workspace(B)
        lg = torch.empty((B, cfg.vocab), dtype=torch.float32, device="cuda")
        busy = torch.zeros(1 << 20, device="cuda")
        for t in range(40):
            model.decode_step(B, t, tok, st, tok, logits=lg, workspace=ws)
            busy += 1.0
        return lg, st, tok

    alone = [job(k) for k in range(4)]
    torch.cuda.synchronize()
    got, streams = [None] * 4, [torch.cuda.Stream() for _ in range(4)]

    def run(k):
        with torch.cuda.stream(streams[k]):
            got[k] = job(k)

    print("one-kernel steps from four threads", flush=True)
    threads = [threading.Thread(target=run, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for a, b in zip(alone, got):
        assert all(torch.equal(x, y) for x, y in zip(a, b))


def test_streams_run_side_by_side_and_more_than_fit_in_turn(srm):
    """Generate calls of two models on seven streams, more than have a CU for each work-group at once: two of the first ones
    run at the same time, and all results are those of the same calls alone."""
    models = []
    for dtype, d in (("fp32", 256), ("bf16", 1024)):
        cfg = srm_synth.tiny_config(vocab=700, d_model=d, n_layers=6, n_heads=4, n_ctx=64, weight_dtype=dtype, seed=29)
        models.append((cfg, srm.Model(cfg, srm_synth.make_weights(cfg))))
    jobs, G = 7, 48

    def prepare(k):
        cfg, model = models[k % 2]
        B = 1 + k % 4
        return model, B, model.new_state(B), model.new_workspace(B), to_dev((np.arange(B) * 13 + k).astype(np.int32)), \
            torch.full((G, B), -7, dtype=torch.int32, device="cuda")

    def run(job, stream=None):
        model, B, st, ws, tk, out = job
        model.generate(B, 1, G, tk, st, out, workspace=ws, stream=stream)
        return tk, st, out

    alone = [run(prepare(k)) for k in range(jobs)]
    again = [prepare(k) for k in range(jobs)]
    streams = [torch.cuda.Stream() for _ in range(jobs)]
    torch.cuda.synchronize()
    print("one-kernel generation on seven streams", flush=True)
    got = []
    events = kernel_events("few_rows_kernel", lambda: got.extend(run(again[k], streams[k]) for k in range(jobs)))
    for a, b in zip(alone, got):
        assert all(torch.equal(x, y) for x, y in zip(a, b))
    spans = sorted((e.time_range.start, e.time_range.end) for e in events)
    assert len(spans) == jobs
    assert any(spans[i + 1][0] < spans[i][1] for i in range(jobs - 1)), spans


def test_packed_copies_only_where_a_call_can_use_them(srm, monkeypatch):
    """A model's second copy of its matrices: not where none of its calls can run as one kernel, and not with the switch off."""
    def memory_of(**kw):
        cfg = srm_synth.tiny_config(**{**dict(vocab=40000, d_model=512, n_layers=6, n_heads=4, n_ctx=16, weight_dtype="bf16", seed=3), **kw})
        w = srm_synth.make_weights(cfg)
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        model = srm.Model(cfg, w)
        used = before - torch.cuda.mem_get_info()[0]
        st, tok, lg = model.new_state(2), torch.zeros(2, dtype=torch.int32, device="cuda"), torch.empty((2, cfg.vocab), device="cuda")
        ws, out = model.new_workspace(2), torch.empty(2, dtype=torch.int32, device="cuda")
        n = _launches(lambda: model.decode_step(2, 0, tok, st, out, logits=lg, workspace=ws))
        assert torch.equal(out.long(), lg.argmax(dim=1))
        model.close()
        return used, n

    matrices = 2 * (40000 + 6 * 10 * 512) * 512                        # bytes of head and blocks; the embedding is kept once
    memory_of()
    with_copies, one = memory_of()
    monkeypatch.setenv(SWITCH, "0")
    without, none = memory_of()
    monkeypatch.delenv(SWITCH)
    assert one == 1 and none == 0 and with_copies - without >= 0.9 * matrices
    bare = memory_of(use_projections=False, n_layers=5)
    monkeypatch.setenv(SWITCH, "0")
    assert bare[1] == 0 and memory_of(use_projections=False, n_layers=5)[0] == bare[0]


def test_model_whose_packed_copies_find_no_room_takes_the_step_kernels(srm, monkeypatch):
    """Device memory filled up to the model's own allocation and about three quarters of the copies (400 MB): the model is made
    all the same, and its steps are those of the switch."""
    import ctypes
    small = srm_synth.tiny_config(vocab=300, d_model=1024, n_layers=6, n_heads=4, n_ctx=16, weight_dtype="bf16", seed=3)
    srm.Model(small, srm_synth.make_weights(small)).close()            # (kernels loaded)
    cfg = dataclasses.replace(small, vocab=120000)
    w = srm_synth.make_weights(small)
    rng = np.random.default_rng(5)
    for name in ("embed", "head"):
        w[name] = (0.02 * rng.standard_normal((cfg.vocab, cfg.d_model), dtype=np.float32))
    tok, B = to_dev(np.arange(3, dtype=np.int32)), 3
    lg = torch.empty((B, cfg.vocab), dtype=torch.float32, device="cuda")
    hip = ctypes.CDLL("libamdhip64.so")
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    matrices = 2 * (cfg.vocab + 6 * 10 * 1024) * 1024                  # bytes of the copies
    own = matrices + 2 * cfg.vocab * 1024 + (8 << 20)
    held = []

    def hold(n):
        at = ctypes.c_void_p()
        if hip.hipMalloc(ctypes.byref(at), ctypes.c_size_t(n)) != 0:
            hip.hipGetLastError()
            return False
        held.append(at)
        return True

    try:
        assert hold(torch.cuda.mem_get_info()[0] - own - matrices)     # (more can be had than is said to be free)
        for _ in range(400):                                           # until the model fits and three quarters of the copies do not
            if not hold(own + matrices * 3 // 4):
                break
            assert hip.hipFree(held.pop()) == 0 and hold(32 << 20)
        print(f"device memory filled, {len(held)} pieces", flush=True)
        model = srm.Model(cfg, w)
    finally:
        for at in held:
            assert hip.hipFree(at) == 0

    def step():
        st, out, ws = model.new_state(B), torch.empty(B, dtype=torch.int32, device="cuda"), model.new_workspace(B)
        model.decode_step(B, 0, tok, st, out, logits=lg, workspace=ws)
        torch.cuda.synchronize()
        return lg.clone(), out, st

    assert _launches(step) == 0
    got = step()
    monkeypatch.setenv(SWITCH, "0")
    assert all(torch.equal(a, b) for a, b in zip(got, step()))
    assert torch.equal(got[1].long(), got[0].argmax(dim=1))
    model.close()


@pytest.mark.parametrize("dtype,d", [("bf16", 512), ("bf16", 1024), ("fp32", 256)])
def test_workspace_of_the_row_arrays_alone(srm, dtype, d, monkeypatch):
    """The words lie where the arrays of the rows would, and only those of a few rows need more room.  A workspace of the arrays
    alone holds as many rows as ever, and no more: a step of a few by the step kernels where the words find no room, a larger
    batch in one pass, prompts and sequences of that many positions."""
    cfg = srm_synth.tiny_config(vocab=700, d_model=d, n_layers=6, n_heads=4, n_ctx=64, weight_dtype=dtype, seed=23)
    model = srm.Model(cfg, srm_synth.make_weights(cfg))
    most, cols, gw = (4, 8, 2 * d) if dtype == "bf16" else (8, 4, 4 * d)
    deep = dataclasses.replace(cfg, n_layers=65)                       # (never one kernel: its workspace is the arrays)

    def arrays(rows):
        return srm.workspace_bytes_config(deep, rows)

    def words(B):
        unrolled = next(n for n in (1, 2, 4, 8) if n >= B)
        return 512 + unrolled * (2 * d + gw + 2 * (d // cols)) * 8 + 256

    for rows in (most, 9, 32, 300):
        assert model.workspace_bytes(rows) == max(arrays(rows), words(min(rows, most)))
    assert model.workspace_bytes(32) == arrays(32) and model.workspace_bytes(300) == arrays(300)

    def step(B, nbytes, **how):
        ws = torch.randint(0, 256, (nbytes + 4096,), dtype=torch.uint8, device="cuda")
        guard, st, out = ws[nbytes:].clone(), model.new_state(B), torch.empty(B, dtype=torch.int32, device="cuda")
        tok, lg = to_dev((np.arange(B) % cfg.vocab).astype(np.int32)), torch.empty((B, cfg.vocab), device="cuda")
        model.decode_step(B, 2, tok, st, out, logits=lg, workspace=ws[:nbytes], **how)
        torch.cuda.synchronize()
        assert torch.equal(ws[nbytes:], guard)
        return out, st, lg

    print(f"workspace of the arrays alone {dtype} d={d}", flush=True)
    for B in (1, 2, most, most + 1, 300):
        for how in (dict(), dict(temperature=0.7, top_p=0.9, seed=5)):
            small, whole = step(B, arrays(B), **how), step(B, model.workspace_bytes(B), **how)
            assert _launches(lambda: step(B, model.workspace_bytes(B), **how)) == (B <= most)
            one = B <= most and words(B) <= arrays(B)
            assert _launches(lambda: step(B, arrays(B), **how)) == one
            if B <= most and not one:
                monkeypatch.setenv(SWITCH, "0")
                whole = step(B, model.workspace_bytes(B), **how)
                monkeypatch.delenv(SWITCH)
            assert all(torch.equal(a, b) for a, b in zip(small, whole))
        with pytest.raises(srm.SrmError):
            step(min(B, 256), arrays(min(B, 256)) - 256)
    P = 40
    toks, st, tk = to_dev(srm_synth.make_prompts(cfg, batch=1, length=P)), model.new_state(1), torch.empty(1, dtype=torch.int32, device="cuda")
    off, hid = np.array([0, P], dtype=np.int32), torch.empty((1, P, d), dtype=torch.float32, device="cuda")
    ws = torch.empty(arrays(P), dtype=torch.uint8, device="cuda")
    model.prefill(toks, 1, st, tk, workspace=ws)
    keep = model.prefill_ragged(toks.view(-1), off, st, tk, workspace=ws)
    model.parallel_forward(toks, hid, workspace=ws)
    assert srm.prefill_ragged_plan(cfg, off, arrays(P))["passes"] == 1
    torch.cuda.synchronize()
    del keep
    with pytest.raises(srm.SrmError):
        srm.prefill_ragged_plan(cfg, off, arrays(P) - 256)
    with pytest.raises(srm.SrmError):                                  # a workspace of fewer rows
        model.prefill_ragged(toks.view(-1), off, st, tk, workspace=model.new_workspace(P - 8))
    model.close()


def test_workspace_size_without_a_model(srm):
    """The size computed from a configuration alone covers the words of the one-kernel steps too."""
    for dtype, d in (("bf16", 1024), ("bf16", 512), ("fp32", 256), ("bf16", 256)):
        cfg = srm_synth.tiny_config(vocab=700, d_model=d, n_layers=6, n_heads=4, n_ctx=64, weight_dtype=dtype, seed=23)
        model = srm.Model(cfg, srm_synth.make_weights(cfg))
        for rows in (1, 2, 3, 4, 5, 8, 9, 300):
            assert srm.workspace_bytes_config(cfg, rows) == model.workspace_bytes(rows), (dtype, d, rows)


@pytest.mark.parametrize("d,B,bare", [(512, 3, False), (1024, 2, False), (1024, 4, True)])
def test_calls_that_keep_the_step_kernels_agree_with_steps_as_one_kernel(srm, d, B, bare, monkeypatch):
    """A ragged step with all samples at one position, a captured step, and generation with a nucleus or without projections
    against eager steps that run as one kernel: equal up to the order of sums and the bf16 roundings behind it, the same
    tokens unless two scores lie that close, and the same bits with the switch off."""
    cfg = srm_synth.tiny_config(vocab=700, d_model=d, n_layers=6, n_heads=4, n_ctx=16, weight_dtype="bf16", seed=37,
                                use_projections=not bare)
    model = srm.Model(cfg, srm_synth.make_weights(cfg, stress=True))
    ws, P, G, tol = model.new_workspace(B), 3, 5, 4e-2           # each of the two within 2e-2 of exact sums
    tok0 = to_dev((np.arange(B) * 31 + 2).astype(np.int32))

    def logits():
        return torch.empty((B, cfg.vocab), dtype=torch.float32, device="cuda")

    def step(tok, pos, st, lg, **how):
        out = torch.empty(B, dtype=torch.int32, device="cuda")
        model.decode_step(B, pos, tok, st, out, logits=lg, workspace=ws, **how)
        return out

    def eager():
        st, lg = model.new_state(B), logits()
        return lg, step(tok0, P, st, lg), st

    def ragged():
        st, lg, out = model.new_state(B), logits(), torch.empty(B, dtype=torch.int32, device="cuda")
        pos = torch.full((B,), P, dtype=torch.int32, device="cuda")
        model.decode_step_ragged(B, pos, tok0, st, out, advance=False, logits=lg, workspace=ws)
        return lg, out, st

    def captured():
        st, lg, out = model.new_state(B), logits(), torch.empty(B, dtype=torch.int32, device="cuda")
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
            model.decode_step(B, P, tok0, st, out, logits=lg, workspace=ws)
        for _ in range(3):
            st.zero_()
            graph.replay()
            torch.cuda.synchronize()
        return lg, out, st

    def close(a, b):
        return (a.float() - b.float()).abs().max() <= tol * b.float().abs().max()

    print(f"calls with the step kernels d={d} B={B} bare={bare}", flush=True)
    eager(), ragged()
    seen = {"captured": captured()}
    assert _launches(lambda: seen.update(one=eager())) == 1
    assert _launches(lambda: seen.update(ragged=ragged())) == 0
    lg, out, st = seen["one"]
    for how in ("ragged", "captured"):
        lg2, out2, st2 = seen[how]
        assert rel_err_rows(lg2.cpu().numpy(), lg.cpu().numpy()) <= tol and close(st2, st)
        assert torch.equal(out2.long(), lg2.argmax(dim=1))
    monkeypatch.setenv(SWITCH, "0")
    plain = eager()
    for how in ("ragged", "captured"):
        assert all(torch.equal(a, b) for a, b in zip(plain, seen[how]))
    monkeypatch.delenv(SWITCH)

    ways = [dict(temperature=0.7, top_p=0.9, seed=4)] + ([dict()] if bare else [])
    for how in ways:
        def generate():
            st, tk, out = model.new_state(B), tok0.clone(), torch.full((G, B), -7, dtype=torch.int32, device="cuda")
            model.generate(B, P, G, tk, st, out, workspace=ws, **how, **({"logits": logits()} if "top_p" in how else {}))
            torch.cuda.synchronize()
            return out, st

        def steps(fed=None):                                     # on their own tokens, or on those of `fed`
            st, tk, rows, outs = model.new_state(B), tok0, [], []
            for g in range(G):
                lg = logits()
                out = step(tk, P + g, st, lg, **how)
                rows.append(lg)
                outs.append(out)
                tk = out if fed is None else fed[g]
            torch.cuda.synchronize()
            return torch.stack(outs), st, rows

        generate()
        assert _launches(lambda: seen.update(gen=generate())) == 0
        out, st = seen["gen"]
        monkeypatch.setenv(SWITCH, "0")
        same = steps()
        assert torch.equal(same[0], out) and torch.equal(same[1], st)
        monkeypatch.delenv(SWITCH)
        assert _launches(lambda: seen.update(steps=steps(out))) == G
        outs, st2, rows = seen["steps"]
        assert close(st2, st)
        for g in range(G):
            assert rel_err_rows(rows[g].cpu().numpy(), same[2][g].cpu().numpy()) <= tol
            if not how:                                          # both tokens are greedy choices from logits this close
                for b in range(B):
                    lost = rows[g][b].max() - rows[g][b, out[g, b]]
                    assert lost <= 2 * tol * rows[g][b].abs().max(), (g, b)
    model.close()


def test_streams_that_are_no_objects_of_their_own(srm):
    """Steps on the runtime's special stream handles (0: default, 1: legacy, 2: per thread) and on a stream that is destroyed
    behind them: results as on any other stream, and no error left behind for the next call."""
    import ctypes
    import types
    cfg = srm_synth.tiny_config(vocab=300, d_model=512, n_layers=6, n_heads=4, n_ctx=16, weight_dtype="bf16", seed=3)
    model = srm.Model(cfg, srm_synth.make_weights(cfg))
    hip, B = ctypes.CDLL("libamdhip64.so"), 3
    tok, ws = to_dev(np.arange(B, dtype=np.int32) * 5), model.new_workspace(B)

    def step(handle):
        st, out = model.new_state(B), torch.empty(B, dtype=torch.int32, device="cuda")
        lg = torch.empty((B, cfg.vocab), dtype=torch.float32, device="cuda")
        torch.cuda.synchronize()
        model.decode_step(B, 0, tok, st, out, logits=lg, workspace=ws, stream=types.SimpleNamespace(cuda_stream=handle))
        assert hip.hipGetLastError() == 0
        torch.cuda.synchronize()
        return lg, out, st

    want = step(torch.cuda.Stream().cuda_stream)
    for handle in (0, 1, 2):
        print(f"step on stream handle {handle}", flush=True)
        assert _launches(lambda: step(handle)) == 1
        assert all(torch.equal(a, b) for a, b in zip(step(handle), want))
    for _ in range(6):                                   # (more than the library keeps events for at a time)
        own = ctypes.c_void_p()
        assert hip.hipStreamCreate(ctypes.byref(own)) == 0
        assert all(torch.equal(a, b) for a, b in zip(step(own.value), want))
        assert hip.hipStreamDestroy(own) == 0
    assert all(torch.equal(a, b) for a, b in zip(step(0), want))


@pytest.mark.parametrize("B,half", [(9, False), (16, True), (23, False), (32, False)])
def test_generation_in_groups_matches_oracle(srm, orc_mod, B, half, monkeypatch):
    """fp32 generation of up to 32 samples, the rows in groups of one, two or four to an XCD: tokens and state of the oracle,
    sampled tokens keyed on the sample's number in the call, and the same bits by one work-group alone and beside another stream."""
    cfg = dataclasses.replace(srm_synth.CONFIGS["C1"], state_dtype="fp16" if half else "fp32", n_layers=3)
    w = srm_synth.make_weights(cfg)
    w["head"] = w["head"] * 25.0
    prompts = srm_synth.make_prompts(cfg, batch=B, length=5)
    P, G = prompts.shape[1], 12
    model, orc = srm.Model(cfg, w), orc_mod.Oracle(cfg, w, "f64")
    ws, dp = model.new_workspace(B * P), to_dev(prompts)

    def generate(temperature, stream=None):
        st, tk = model.new_state(B), torch.empty(B, dtype=torch.int32, device="cuda")
        model.prefill(dp[:, :P - 1].contiguous(), 1, st, tk, workspace=ws)
        tk.copy_(dp[:, P - 1])
        out = torch.full((G, B), -7, dtype=torch.int32, device="cuda")
        torch.cuda.synchronize()
        assert _launches(lambda: model.generate(B, P - 1, G, tk, st, out, workspace=ws, temperature=temperature, seed=7, stream=stream)) == 1
        return out, tk, st

    for temperature in (0.0, 0.7):
        kw = {"temperature": temperature, "seed": 7} if temperature else {}
        ref = orc.greedy(prompts, G, want_logits=True, **kw)
        print(f"generation in groups B={B} half={half} T={temperature}", flush=True)
        out, tk, st = generate(temperature)
        got = out.cpu().numpy().T
        check_tokens(got, ref["tokens"], ref["margin"], np.abs(ref["logits"]).max(axis=2), rtol=1e-3 if half else 1e-4)
        assert (tk.cpu().numpy() == got[:, -1]).all()
        if not half:
            s_got = st.view(cfg.n_layers, B, cfg.d_model).permute(1, 0, 2).cpu().numpy()
            assert np.abs(s_got - ref["state"]).max() <= 1e-4 * np.abs(ref["state"]).max()
        for mode in ("2", "3"):
            monkeypatch.setenv(SWITCH, mode)
            assert all(torch.equal(a, b) for a, b in zip(generate(temperature), (out, tk, st)))
            monkeypatch.delenv(SWITCH)
        assert all(torch.equal(a, b) for a, b in zip(generate(temperature, torch.cuda.Stream()), (out, tk, st)))
    monkeypatch.setenv("SRM_ONE_KERNEL_POLLS", "0")
    out, tk, st = generate(0.0)
    assert (tk == -1).any() and (out == -1).any()
    monkeypatch.delenv("SRM_ONE_KERNEL_POLLS")
    model.close()


def _alone(model, B=1, G=6):
    """Launches on one stream, behind which those of other streams in earlier tests no longer count."""
    st, tk, ws = model.new_state(B), torch.zeros(B, dtype=torch.int32, device="cuda"), model.new_workspace(B)
    out = torch.empty((G, B), dtype=torch.int32, device="cuda")
    for _ in range(9):
        torch.cuda.synchronize()
        model.generate(B, 3, G, tk, st, out, workspace=ws)
    torch.cuda.synchronize()


@pytest.mark.parametrize("B", [1, 2, 4, 8, 9, 16, 17, 32])
def test_groups_whatever_the_workspace(srm, B):
    """fp32 generation of up to 32 samples runs in groups of the whole device with a workspace of its rows as with a larger one:
    the same bits.  33 samples do not."""
    cfg = dataclasses.replace(srm_synth.CONFIGS["C1"], n_layers=4)
    model, G = srm.Model(cfg, srm_synth.make_weights(cfg)), 6

    def generate(B, rows, guard=4096):
        n = model.workspace_bytes(rows)
        ws = torch.randint(0, 256, (n + guard,), dtype=torch.uint8, device="cuda")
        behind = ws[n:].clone()
        st, tk = model.new_state(B), to_dev((np.arange(B) * 31 % cfg.vocab).astype(np.int32))
        out = torch.full((G, B), -7, dtype=torch.int32, device="cuda")
        model.generate(B, 3, G, tk, st, out, workspace=ws[:n], temperature=0.7, seed=5)
        torch.cuda.synchronize()
        assert torch.equal(ws[n:], behind)
        return out, tk, st

    print(f"groups of {B} samples", flush=True)
    _alone(model)
    runs = {}
    for rows in (B, 4 * B + 60):
        assert kernel_grids("few_rows_kernel", lambda: runs.update({rows: generate(B, rows)})) == [256]
    assert all(torch.equal(a, b) for a, b in zip(runs[B], runs[4 * B + 60]))
    if B == 32:
        assert _launches(lambda: generate(33, 33)) == 0
    model.close()


def _side_by_side(model, cfg, B, G=10, n=4):
    """Generations that wait on n streams at once against the same calls alone, one after the other: the grids of their launches."""
    streams, ws = [torch.cuda.Stream() for _ in range(n)], [model.new_workspace(B) for _ in range(n)]
    sets = [[model.new_state(B), None, torch.full((G, B), -7, dtype=torch.int32, device="cuda")] for _ in range(2 * n)]
    for k, one in enumerate(sets):
        one[1] = to_dev(((np.arange(B) * 31 + 7 * (k % n)) % cfg.vocab).astype(np.int32))

    def generate(k, i):
        st, tk, out = sets[k]
        model.generate(B, 3, G, tk, st, out, workspace=ws[i], temperature=0.7, seed=5 + i, stream=streams[i])

    def all_at_once():
        for s in streams:
            with torch.cuda.stream(s):
                torch.cuda._sleep(40_000_000)                          # (none has begun when the last is launched)
        for i in range(n):
            generate(n + i, i)

    def one_by_one():
        for i in range(n):
            generate(i, i)
            torch.cuda.synchronize()

    _alone(model)
    alone = kernel_grids("few_rows_kernel", one_by_one)
    grids = kernel_grids("few_rows_kernel", all_at_once)
    for i in range(n):
        assert all(torch.equal(a, b) for a, b in zip(sets[i], sets[n + i]))
    return alone, sorted(grids)


@pytest.mark.parametrize("B", [1, 3, 8])
def test_fp32_steps_in_groups_and_side_by_side_have_the_same_bits(srm, B):
    """Up to eight rows run in groups where one stream has the device for itself, streams in turn among them, and as one small grid
    among others of its kind where several run or wait."""
    cfg = dataclasses.replace(srm_synth.CONFIGS["C1"], n_layers=4)
    model = srm.Model(cfg, srm_synth.make_weights(cfg))
    print(f"fp32 generation, groups and side by side B={B}", flush=True)
    assert _side_by_side(model, cfg, B) == ([256] * 4, [64, 64, 64, 256])
    model.close()


@pytest.mark.parametrize("B", [9, 16, 32])
def test_groups_of_several_streams_in_line(srm, B):
    """From nine rows on all run in groups, which exchange through words of the model, one after the other."""
    cfg = dataclasses.replace(srm_synth.CONFIGS["C1"], n_layers=4)
    model = srm.Model(cfg, srm_synth.make_weights(cfg))
    print(f"groups of {B} samples on four streams", flush=True)
    assert _side_by_side(model, cfg, B) == ([256] * 4, [256] * 4)
    model.close()


@pytest.mark.parametrize("B", [1, 8, 9, 32])
def test_groups_that_do_not_share_a_cache(srm, B, monkeypatch):
    """Groups of work-groups on different XCDs: what they exchange is written through the caches, the bits are the same."""
    cfg = dataclasses.replace(srm_synth.CONFIGS["C1"], n_layers=4)
    model, G = srm.Model(cfg, srm_synth.make_weights(cfg)), 20
    ws = model.new_workspace(B)

    def generate():
        st, tk = model.new_state(B), to_dev((np.arange(B) * 31 % cfg.vocab).astype(np.int32))
        out = torch.full((G, B), -7, dtype=torch.int32, device="cuda")
        model.generate(B, 3, G, tk, st, out, workspace=ws, temperature=0.7, seed=5)
        torch.cuda.synchronize()
        return out, tk, st

    _alone(model)
    want = generate()
    monkeypatch.setenv(SWITCH, "4")
    print(f"groups of {B} samples across the XCDs", flush=True)
    runs = {}
    assert kernel_grids("few_rows_kernel", lambda: runs.update(got=generate())) == [256]
    assert all(torch.equal(a, b) for a, b in zip(runs["got"], want))
    model.close()


@pytest.mark.parametrize("B", [1, 8, 9, 32])
@pytest.mark.parametrize("started", [0, 31, 32, 67, 100, 254])
def test_work_groups_that_have_started_do_without_the_others(srm, B, started, monkeypatch):
    """Some work-groups do not start in time (their arrivals are withdrawn from the start): the others form as many whole groups as
    they can, which take the groups of rows in turn, and of less than one group a work-group is left alone; the same bits.  Where
    waits give up, the rows that a group has not come to are gone as well."""
    cfg = dataclasses.replace(srm_synth.CONFIGS["C1"], n_layers=2)
    model, G = srm.Model(cfg, srm_synth.make_weights(cfg)), 5
    ws = model.new_workspace(B)

    def generate():
        st, tk = model.new_state(B), to_dev((np.arange(B) * 31 % cfg.vocab).astype(np.int32))
        out = torch.full((G, B), -7, dtype=torch.int32, device="cuda")
        model.generate(B, 3, G, tk, st, out, workspace=ws, temperature=0.7, seed=5)
        torch.cuda.synchronize()
        return out, tk, st

    _alone(model)
    want = generate()
    monkeypatch.setenv(SWITCH, f"2:{started}")
    print(f"{started} work-groups have started B={B}", flush=True)
    runs = {}
    assert kernel_grids("few_rows_kernel", lambda: runs.update(got=generate())) == [256]
    assert all(torch.equal(a, b) for a, b in zip(runs["got"], want))
    if started >= 32:
        monkeypatch.setenv("SRM_ONE_KERNEL_POLLS", "0")
        out, tk, _ = generate()
        gone = out == -1
        assert gone.any() and torch.equal(out[~gone], want[0][~gone]) and torch.equal(tk, torch.where(gone[-1], -1, want[1]))
    model.close()


@pytest.mark.parametrize("B", [8, 9, 32])
def test_groups_whose_waits_give_up(srm, B, monkeypatch):
    """Groups wait on their own: a sample's tokens are right up to the step in which its group gives up and -1 from there on, the
    last one too; the next call is right."""
    cfg = dataclasses.replace(srm_synth.CONFIGS["C1"], n_layers=4)
    model, G = srm.Model(cfg, srm_synth.make_weights(cfg)), 8
    ws = model.new_workspace(B)

    def generate():
        st, tk = model.new_state(B), to_dev((np.arange(B) * 31 % cfg.vocab).astype(np.int32))
        out = torch.full((G, B), -7, dtype=torch.int32, device="cuda")
        model.generate(B, 3, G, tk, st, out, workspace=ws)
        torch.cuda.synchronize()
        return out, tk, st

    _alone(model)
    want = generate()
    print(f"groups of {B} samples whose waits give up", flush=True)
    monkeypatch.setenv("SRM_ONE_KERNEL_POLLS", "0")
    assert kernel_grids("few_rows_kernel", generate) == [256]
    out, tk, _ = generate()
    monkeypatch.delenv("SRM_ONE_KERNEL_POLLS")
    gone = out == -1
    assert gone.any() and (gone[1:] | ~gone[:-1]).all()                # once gone, gone
    assert torch.equal(out[~gone], want[0][~gone])
    assert torch.equal(tk, torch.where(gone[-1], -1, want[1]))
    assert all(torch.equal(a, b) for a, b in zip(generate(), want))
    model.close()
