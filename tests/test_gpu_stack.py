"""Decode steps of some dozens of samples and more whose layers run as one kernel (a bf16 model of 512 channels), against the
oracle and against the step kernels (the library's switch)."""
import numpy as np
import pytest
import torch

import srm_synth
from gpu_util import to_dev, rel_err_rows, kernel_launches, kernel_grids

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
    return kernel_launches("stack_kernel", fn)


def _config(**kw):
    args = dict(vocab=333, d_model=512, n_layers=6, n_heads=4, n_ctx=12, weight_dtype="bf16", seed=53)
    args.update(kw)
    return srm_synth.tiny_config(**args)


def _steps(model, cfg, toks, positions=None, garbage=None, **how):
    """Steps on given tokens [B][T] in a workspace full of `garbage`, with a guard behind it; positions: of each sample."""
    B, T = toks.shape
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
        if positions is None:
            model.decode_step(B, t, tc[t], st, out, logits=lg, hidden=hd, workspace=buf[:n], **how)
        else:
            pos = to_dev((positions + t).astype(np.int32))
            model.decode_step_ragged(B, pos, tc[t], st, out, advance=False, logits=lg, workspace=buf[:n], **how)
        res.append((lg.clone(), hd.clone(), out.clone()))
    torch.cuda.synchronize()
    assert torch.equal(buf[n:], guard)
    return res, st


# rows at the borders of the plan: whole and part groups of 16, a group's tile of one to four blocks of 16, two members on 32
# columns with tiles of three and four blocks, several tiles to a member
# (2049: four tiles become six; 2304: the most rows, whose positions fill their place in LDS); the smallest step, a second group of one row
ROWS = [5, 9, 16, 17, 33, 128, 129, 300, 512, 513, 1024, 1025, 2048, 2049, 2100, 2304]


@pytest.mark.parametrize("B", ROWS)
@pytest.mark.parametrize("variant", [{}, dict(state_dtype="fp16", head_layout="column")])
def test_layers_in_one_kernel_match_oracle_and_step_kernels(srm, orc_mod, B, variant, monkeypatch):
    cfg = _config(**variant)
    w = srm_synth.make_weights(cfg, stress=True)
    model, T = srm.Model(cfg, w), 2
    toks = srm_synth.make_prompts(cfg, batch=B, length=T)
    some = sorted({0, 15, 16, B // 8, B // 2, B - 17, B - 1} & set(range(B)))
    ref = orc_mod.Oracle(cfg, w, "f64").recurrent_forward(toks[some])
    print(f"layers in one kernel B={B} {variant}", flush=True)
    runs = {}
    assert _launches(lambda: runs.update(one=_steps(model, cfg, toks))) == T
    one, st = runs["one"]
    again, st2 = _steps(model, cfg, toks, garbage=0)
    monkeypatch.setenv(SWITCH, "0")
    assert _launches(lambda: runs.update(many=_steps(model, cfg, toks))) == 0
    many, st3 = runs["many"]
    tol = 4e-2 if cfg.state_dtype == "fp16" else 2e-2                  # the repository's bounds of bf16 logits
    for t in range(T):
        assert all(torch.equal(a, b) for a, b in zip(one[t], again[t]))         # a fixed order of sums: the same bits
        assert rel_err_rows(one[t][0][some].cpu().numpy(), ref["logits"][:, t]) <= tol
        assert rel_err_rows(one[t][1][some].cpu().numpy(), ref["hidden"][:, t]) <= tol
        assert rel_err_rows(one[t][0].cpu().numpy(), many[t][0].cpu().numpy()) <= tol
        assert torch.equal(one[t][2].long(), one[t][0].argmax(dim=1))
    assert torch.equal(st, st2)
    assert (st.float() - st3.float()).abs().max() <= tol * st3.float().abs().max()
    model.close()


@pytest.mark.parametrize("B,launches", [(4, 0), (5, 1), (2304, 1), (2305, 0)])
def test_where_the_kernel_ends(srm, B, launches):
    cfg = _config(vocab=200)
    model = srm.Model(cfg, srm_synth.make_weights(cfg))
    tok, st, ws = torch.zeros(B, dtype=torch.int32, device="cuda"), model.new_state(B), model.new_workspace(B)
    print(f"where the kernel ends B={B}", flush=True)
    assert _launches(lambda: model.decode_step(B, 1, tok, st, tok.clone(), workspace=ws)) == launches
    model.close()


@pytest.mark.parametrize("B", [5, 9, 130, 513, 1100, 2304])
def test_one_work_group_alone_gives_the_same_bits(srm, B, monkeypatch):
    """A launch of whose work-groups none has started in time is done by one of them: forced from the host, by arrivals that are
    withdrawn from the start, then by a wait of one look, which ends either way."""
    cfg = _config(vocab=200)
    model = srm.Model(cfg, srm_synth.make_weights(cfg, stress=True))
    toks = srm_synth.make_prompts(cfg, batch=B, length=2)
    want, st = _steps(model, cfg, toks)
    for mode in ("2", "3"):
        monkeypatch.setenv(SWITCH, mode)
        print(f"one work-group alone B={B} mode {mode}", flush=True)
        got, st2 = _steps(model, cfg, toks)
        monkeypatch.delenv(SWITCH)
        for a, b in zip(want, got):
            assert all(torch.equal(x, y) for x, y in zip(a, b))
        assert torch.equal(st, st2)
    model.close()


@pytest.mark.parametrize("B", [5, 300, 513, 2304])
@pytest.mark.parametrize("started", [7, 8, 17, 35, 100, 129, 255])
def test_work_groups_that_have_started_do_without_the_others(srm, B, started, monkeypatch):
    """Some work-groups do not start in time (their arrivals are withdrawn from the start): the others form groups of one to
    sixteen, some of which lie across XCDs, and of less than eight one is left alone; the same bits."""
    cfg = _config(vocab=200)
    model = srm.Model(cfg, srm_synth.make_weights(cfg, stress=True))
    toks = srm_synth.make_prompts(cfg, batch=B, length=2)
    want, st = _steps(model, cfg, toks)
    monkeypatch.setenv(SWITCH, f"2:{started}")
    print(f"{started} work-groups have started B={B}", flush=True)
    got, st2 = _steps(model, cfg, toks)
    for a, b in zip(want, got):
        assert all(torch.equal(x, y) for x, y in zip(a, b))
    assert torch.equal(st, st2)
    model.close()


@pytest.mark.parametrize("B", [5, 33, 300, 513, 1100, 2304])
def test_groups_that_do_not_share_a_cache(srm, B, monkeypatch):
    """Groups of work-groups on different XCDs, as they come about where the XCDs do not get as many work-groups each: what they
    exchange is written through the caches, the bits are the same, and the tokens -1 where their waits give up."""
    cfg = _config(vocab=200)
    model = srm.Model(cfg, srm_synth.make_weights(cfg, stress=True))
    toks = srm_synth.make_prompts(cfg, batch=B, length=3)
    want, st = _steps(model, cfg, toks)
    monkeypatch.setenv(SWITCH, "4")
    print(f"groups across the XCDs B={B}", flush=True)
    runs = {}
    for garbage in (None, 0):
        assert _launches(lambda: runs.update(got=_steps(model, cfg, toks, garbage=garbage))) == 3
        got, st2 = runs["got"]
        for a, b in zip(want, got):
            assert all(torch.equal(x, y) for x, y in zip(a, b))
        assert torch.equal(st, st2)
    monkeypatch.setenv("SRM_ONE_KERNEL_POLLS", "0")
    got, _ = _steps(model, cfg, toks)
    assert all((one[2] == -1).all() for one in got)
    model.close()


def test_ragged_step_in_one_kernel(srm, monkeypatch):
    """One position per sample, some outside the context: those keep their state and get -1; at one position for all the same
    bits as the plain step; otherwise the step kernels' results within the bf16 bound."""
    cfg = _config()
    model, B, T = srm.Model(cfg, srm_synth.make_weights(cfg, stress=True)), 200, 2
    toks = srm_synth.make_prompts(cfg, batch=B, length=T)
    plain, st = _steps(model, cfg, toks)
    same, st2 = _steps(model, cfg, toks, positions=np.zeros(B))
    for a, b in zip(plain, same):
        assert torch.equal(a[0], b[0]) and torch.equal(a[2], b[2])
    assert torch.equal(st, st2)
    positions = np.arange(B) % (cfg.n_ctx + 3) - 2
    print("ragged step in one kernel", flush=True)
    runs = {}
    assert _launches(lambda: runs.update(one=_steps(model, cfg, toks, positions=positions))) == T
    monkeypatch.setenv(SWITCH, "0")
    many, st4 = _steps(model, cfg, toks, positions=positions)
    one, st3 = runs["one"]
    for t in range(T):
        idle = torch.from_numpy(((positions + t < 0) | (positions + t >= cfg.n_ctx))).cuda()
        assert (one[t][2][idle] == -1).all() and (one[t][2][~idle] >= 0).all()
        assert rel_err_rows(one[t][0][~idle].cpu().numpy(), many[t][0][~idle].cpu().numpy()) <= 2e-2
    assert (st3 - st4).abs().max() <= 2e-2 * st4.abs().max()
    model.close()


def test_generation_and_slices(srm):
    """srm_generate gives the tokens and states of single steps, and a workspace of fewer rows takes the step in slices."""
    cfg = _config(vocab=400, n_ctx=40)
    model, B, G = srm.Model(cfg, srm_synth.make_weights(cfg, stress=True)), 600, 5
    start = to_dev((np.arange(B) * 7 % cfg.vocab).astype(np.int32))
    ws, small = model.new_workspace(B), model.new_workspace(256)
    results = []
    for stream in (None, torch.cuda.Stream()):
        st, tk, out = model.new_state(B), start.clone(), torch.full((G, B), -7, dtype=torch.int32, device="cuda")
        torch.cuda.synchronize()
        print(f"generation of {B} samples", flush=True)
        assert _launches(lambda: model.generate(B, 3, G, tk, st, out, workspace=ws, temperature=0.7, seed=9, stream=stream)) == G
        results.append((out, st))
    st, tk = model.new_state(B), start.clone()
    steps = []
    for g in range(G):
        model.decode_step(B, 3 + g, tk, st, tk, workspace=ws, temperature=0.7, seed=9)
        steps.append(tk.clone())
    results.append((torch.stack(steps), st))
    for out, st in results[1:]:
        assert torch.equal(out, results[0][0]) and torch.equal(st, results[0][1])
    st, out = model.new_state(B), torch.empty(B, dtype=torch.int32, device="cuda")
    lg, lg2 = (torch.empty((B, cfg.vocab), dtype=torch.float32, device="cuda") for _ in range(2))
    model.decode_step(B, 3, start, model.new_state(B), out, logits=lg, workspace=ws)
    assert _launches(lambda: model.decode_step(B, 3, start, st, out, logits=lg2, workspace=small)) == 3
    assert rel_err_rows(lg2.cpu().numpy(), lg.cpu().numpy()) <= 2e-2
    model.close()


@pytest.mark.parametrize("B,rows", [(600, 256), (258, 256), (2310, 2304), (2307, 256)])
def test_generation_in_slices(srm, B, rows):
    """srm_generate through a workspace of fewer rows: every step by the kernels of its slices, the last of which may be too small or
    the only one small enough for the kernel of all layers, as single steps through that workspace take them, on every stream."""
    cfg = _config(vocab=400, n_ctx=40)
    model, G = srm.Model(cfg, srm_synth.make_weights(cfg, stress=True)), 4
    start = to_dev((np.arange(B) * 7 % cfg.vocab).astype(np.int32))
    n = model.workspace_bytes(rows) + 256                              # (the step counters)
    stacks = sum(5 <= min(rows, B - b) <= 2304 for b in range(0, B, rows))
    st, tk, steps = model.new_state(B), start.clone(), []
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    for g in range(G):
        model.decode_step(B, 3 + g, tk, st, tk, workspace=ws, temperature=0.7, seed=9)
        steps.append(tk.clone())
    for stream in (None, torch.cuda.Stream()):
        st2, tk, out = model.new_state(B), start.clone(), torch.full((G, B), -7, dtype=torch.int32, device="cuda")
        torch.cuda.synchronize()
        print(f"generation of {B} samples through {rows} rows", flush=True)
        assert _launches(lambda: model.generate(B, 3, G, tk, st2, out, workspace=ws, temperature=0.7, seed=9, stream=stream)) == G * stacks
        assert torch.equal(out, torch.stack(steps)) and torch.equal(st2, st) and torch.equal(tk, steps[-1])
    model.close()


def test_a_wait_that_gives_up_leaves_marked_tokens(srm, monkeypatch):
    """The bound of the waits behind the arrival, set so short from the host that some give up at once: every wavefront ends,
    the tokens are -1 (behind a nucleus pass too), and the next call is right."""
    cfg = _config(vocab=1001, n_ctx=16)
    model, B = srm.Model(cfg, srm_synth.make_weights(cfg, stress=True)), 150
    ws, lg = model.new_workspace(B), torch.zeros((B, cfg.vocab), dtype=torch.float32, device="cuda")
    tok = to_dev(np.arange(B, dtype=np.int32))

    def step(**how):
        st, out = model.new_state(B), torch.full((B,), 5, dtype=torch.int32, device="cuda")
        model.decode_step(B, 1, tok, st, out, logits=lg, workspace=ws, **how)
        torch.cuda.synchronize()
        return out, st, lg.clone()

    ways = (dict(), dict(temperature=0.7, top_p=0.6, seed=3))
    want = [step(**how) for how in ways]
    monkeypatch.setenv("SRM_ONE_KERNEL_POLLS", "0")
    for how in ways:
        print(f"a wait that gives up {how}", flush=True)
        assert (step(**how)[0] == -1).all()
    monkeypatch.delenv("SRM_ONE_KERNEL_POLLS")
    for how, w in zip(ways, want):
        assert all(torch.equal(a, b) for a, b in zip(step(**how), w))
    model.close()


@pytest.mark.parametrize("how", [dict(), dict(temperature=0.7, seed=3), dict(temperature=0.7, top_p=0.6, seed=3)])
@pytest.mark.parametrize("rows", [300, 256])
def test_ragged_generation_with_an_end_token(srm, rows, how):
    """srm_generate_ragged gives the tokens, positions and states of single ragged steps: samples that are idle, that reach the end of
    the context and that emit the end token, whole and in slices."""
    cfg = _config(vocab=40, n_ctx=12)
    model, B, G, eos = srm.Model(cfg, srm_synth.make_weights(cfg, stress=True)), 300, 6, 7
    ws = torch.empty(model.workspace_bytes(rows) + 256, dtype=torch.uint8, device="cuda")
    lg = torch.empty((B, cfg.vocab), device="cuda")
    start = to_dev((np.arange(B) * 7 % cfg.vocab).astype(np.int32))
    pos0 = (torch.arange(B, device="cuda") % 14 - 1).to(torch.int32)
    st, tk, pos, want = model.new_state(B), start.clone(), pos0.clone(), []
    for g in range(G):
        model.decode_step_ragged(B, pos, tk, st, tk, advance=True, logits=lg, workspace=ws, **how)
        pos = torch.where(tk == eos, -1, pos).to(torch.int32)          # (single steps know no end token)
        want.append(tk.clone())
    want = torch.stack(want)
    assert (want == -1).any() and (want == eos).any()
    st2, tk2, pos2, out = model.new_state(B), start.clone(), pos0.clone(), torch.full((G, B), -7, dtype=torch.int32, device="cuda")
    print(f"ragged generation through {rows} rows {how}", flush=True)
    assert _launches(lambda: model.generate_ragged(B, G, pos2, tk2, st2, out, eos_id=eos, logits=lg, workspace=ws, **how)) == G * (-(-B // rows))
    assert torch.equal(out, want) and torch.equal(pos2, pos) and torch.equal(tk2, want[-1]) and torch.equal(st2, st)
    model.close()


@pytest.mark.parametrize("how", [dict(), dict(temperature=0.7, seed=3), dict(temperature=0.7, top_p=0.6, seed=3)])
@pytest.mark.parametrize("rows", [400, 256])
def test_a_generation_whose_wait_gives_up(srm, rows, how, monkeypatch):
    """A wait that gives up in one step of a generation only, forced from the host: the tokens from that step on are -1, also where
    the waits of later steps hold, in every slice behind it; the steps in front are right, and so is the next call."""
    cfg = _config(vocab=300, n_ctx=30)
    model, B, G, at = srm.Model(cfg, srm_synth.make_weights(cfg, stress=True)), 400, 5, 2
    ws = torch.empty(model.workspace_bytes(rows) + 256, dtype=torch.uint8, device="cuda")
    lg = torch.empty((B, cfg.vocab), device="cuda") if "top_p" in how else None
    start = to_dev((np.arange(B) * 7 % cfg.vocab).astype(np.int32))
    idle = torch.arange(B, device="cuda") % 7 == 3
    pos0 = torch.where(idle, -1, torch.arange(B, device="cuda") % 11).to(torch.int32)

    def plain():
        st, tk, out = model.new_state(B), start.clone(), torch.full((G, B), -7, dtype=torch.int32, device="cuda")
        model.generate(B, 3, G, tk, st, out, workspace=ws, logits=lg, **how)
        torch.cuda.synchronize()
        return out, tk, st

    def ragged():
        st, tk, out, pos = model.new_state(B), start.clone(), torch.full((G, B), -7, dtype=torch.int32, device="cuda"), pos0.clone()
        model.generate_ragged(B, G, pos, tk, st, out, workspace=ws, logits=lg, **how)
        torch.cuda.synchronize()
        return out, tk, st, pos

    for run in (plain, ragged):
        want = run()
        active = torch.ones_like(idle) if run is plain else ~idle
        assert (want[0][:, active] >= 0).all()
        print(f"generation, a wait gives up in step {at}: {rows} rows {how} {run.__name__}", flush=True)
        for bound in (f"0:{at}", "0"):
            monkeypatch.setenv("SRM_ONE_KERNEL_POLLS", bound)
            got = run()
            monkeypatch.delenv("SRM_ONE_KERNEL_POLLS")
            first = at if ":" in bound else 0
            assert torch.equal(got[0][:first], want[0][:first])
            assert (got[0][first + 1:] == -1).all() and (got[1] == -1).all()
            mid = got[0][first]                      # (a slice in front of the one that gives up has its tokens)
            assert ((mid == -1) | (mid == want[0][first])).all() and (mid[256 if rows == 256 else 0:] == -1).all()
            if run is ragged:
                there = pos0 + first + ((mid != -1) & active).int()
                assert torch.equal(got[3], torch.where(active, there, pos0))
        assert all(torch.equal(a, b) for a, b in zip(run(), want))
    model.close()


@pytest.mark.parametrize("B", [37, 300, 513, 1100])
def test_streams_in_turn_give_the_same_bits(srm, B):
    """Steps launched on two streams in turn, each behind a synchronisation, have the device for themselves."""
    cfg = _config(vocab=200)
    model = srm.Model(cfg, srm_synth.make_weights(cfg, stress=True))
    tok = to_dev((np.arange(B) * 3 % cfg.vocab).astype(np.int32))
    ws = [model.new_workspace(B) for _ in range(2)]
    streams = [torch.cuda.Stream() for _ in range(2)]

    def step(i):
        st, out = model.new_state(B), torch.empty(B, dtype=torch.int32, device="cuda")
        lg = torch.empty((B, cfg.vocab), dtype=torch.float32, device="cuda")
        torch.cuda.synchronize()
        model.decode_step(B, 2, tok, st, out, logits=lg, workspace=ws[i], stream=streams[i])
        return st, out, lg

    print(f"streams in turn B={B}", flush=True)
    for _ in range(9):
        want = step(0)
    got = [step(i % 2) for i in range(6)]
    assert _launches(lambda: got.append(step(1))) == 1
    assert kernel_grids("stack_kernel", lambda: got.extend(step(i % 2) for i in range(4))) == [256] * 4
    torch.cuda.synchronize()
    for one in got:
        assert all(torch.equal(a, b) for a, b in zip(one, want))
    model.close()


@pytest.mark.parametrize("n", [2, 4])
@pytest.mark.parametrize("B", [9, 300, 513, 1024, 1025])
def test_streams_side_by_side_share_the_device(srm, B, n, monkeypatch):
    """Steps on several streams whose kernels are all still waiting: the first takes the device, a second stream half of the
    work-groups, further ones a quarter, so that four fit side by side (from 1025 rows on all of it); the same bits, also by one
    work-group alone, and -1 for all samples of a launch one of whose waits gives up."""
    cfg = _config(vocab=200)
    model = srm.Model(cfg, srm_synth.make_weights(cfg, stress=True))
    tok = to_dev((np.arange(B) * 3 % cfg.vocab).astype(np.int32))
    ws, streams = [model.new_workspace(B) for _ in range(n)], [torch.cuda.Stream() for _ in range(n)]
    want = {}

    def steps():
        got = [(model.new_state(B), torch.empty(B, dtype=torch.int32, device="cuda"),
                torch.empty((B, cfg.vocab), dtype=torch.float32, device="cuda")) for _ in range(n)]
        torch.cuda.synchronize()
        for s in streams:
            with torch.cuda.stream(s):
                torch.cuda._sleep(40_000_000)                          # some 20 ms: none has begun when the last is launched
        for (st, out, lg), w, s in zip(got, ws, streams):
            model.decode_step(B, 2, tok, st, out, logits=lg, workspace=w, stream=s)
        torch.cuda.synchronize()
        want["got"] = got

    st, out, lg = model.new_state(B), torch.empty(B, dtype=torch.int32, device="cuda"), torch.empty((B, cfg.vocab), device="cuda")
    for _ in range(9):                                                 # (streams that have met are reckoned with for eight launches)
        st.zero_()
        torch.cuda.synchronize()
        model.decode_step(B, 2, tok, st, out, logits=lg, workspace=ws[0], stream=streams[0])
        torch.cuda.synchronize()
    print(f"{n} streams side by side B={B}", flush=True)
    assert sorted(kernel_grids("stack_kernel", steps)) == sorted([256, 128, 64, 64][:n] if B <= 1024 else [256] * n)
    for mode in (None, "2", "3", "4"):
        if mode:
            monkeypatch.setenv(SWITCH, mode)
            print(f"one work-group of each alone, or groups across the XCDs: mode {mode}", flush=True)
            steps()
            monkeypatch.delenv(SWITCH)
        for one in want["got"]:
            assert all(torch.equal(a, b) for a, b in zip(one, (st, out, lg)))
    monkeypatch.setenv("SRM_ONE_KERNEL_POLLS", "0")
    steps()
    monkeypatch.delenv("SRM_ONE_KERNEL_POLLS")
    # (a group of the few work-groups that have started in time may find all of them there at its first look, at every wait)
    assert any((one[1] == -1).all() for one in want["got"])
    assert all((one[1] == -1).all() or all(torch.equal(a, b) for a, b in zip(one, (st, out, lg))) for one in want["got"])
    steps()
    for one in want["got"]:
        assert all(torch.equal(a, b) for a, b in zip(one, (st, out, lg)))
    model.close()


def test_streams_side_by_side_beside_a_capture(srm):
    """Steps on two streams while the same thread captures a graph on a third: the graph is whole, the steps are right."""
    cfg, B = _config(vocab=200), 64
    model = srm.Model(cfg, srm_synth.make_weights(cfg, stress=True))
    tok = to_dev((np.arange(B) * 3 % cfg.vocab).astype(np.int32))
    ws, streams = [model.new_workspace(B) for _ in range(2)], [torch.cuda.Stream() for _ in range(2)]
    sets = [[model.new_state(B), torch.empty(B, dtype=torch.int32, device="cuda")] for _ in range(5)]
    x, cap, graph = torch.zeros(64, device="cuda"), torch.cuda.Stream(), torch.cuda.CUDAGraph()

    def step(i, k):
        model.decode_step(B, 2, tok, sets[k][0], sets[k][1], workspace=ws[i], stream=streams[i])

    step(0, 0)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=cap):
        x.add_(1.0)
        for k in range(1, 5):
            step(k % 2, k)
        x.add_(1.0)
    torch.cuda.synchronize()
    for _ in range(3):
        graph.replay()
    torch.cuda.synchronize()
    assert (x == 6.0).all()
    for st, out in sets[1:]:
        assert torch.equal(st, sets[0][0]) and torch.equal(out, sets[0][1])
    model.close()
