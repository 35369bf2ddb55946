"""Shared helpers of the GPU parity tests (no method arithmetic here)."""
import json
import os
import tempfile
import time

import numpy as np
import torch


def to_dev(a, dtype=None):
    t = torch.from_numpy(np.ascontiguousarray(a)).cuda()
    return t if dtype is None else t.to(dtype)


def rel_err_rows(got, ref):
    """max over rows of max|got-ref| / max|ref| along the last axis."""
    ref = np.asarray(ref, dtype=np.float64)
    scale = np.abs(ref).max(axis=-1, keepdims=True)
    return float((np.abs(np.asarray(got, dtype=np.float64) - ref) / scale).max())


def check_tokens(got, ref_tokens, ref_margin, ref_logits_absmax, rtol=1e-4):
    """Greedy tokens must equal the oracle's, except where the oracle's own top-2
    margin is below rtol * max|logit| (a tolerated near tie).  Returns the number
    of tolerated ties."""
    got = np.asarray(got); ref_tokens = np.asarray(ref_tokens)
    bad = got != ref_tokens
    tie = ref_margin < rtol * ref_logits_absmax
    assert not (bad & ~tie).any(), f"{int((bad & ~tie).sum())} tokens differ from the oracle"
    return int((bad & tie).sum())


def _profile(fn):
    """The profiler over fn().  It drops kernels whose times,
    converted from the GPU's clock to the host's, lie outside its window, and behind a long wait on the host they may be
    off by more than a few steps take: so the window has a margin on both sides, whose own kernels show that none of fn's
    is lost."""
    from torch.profiler import profile, ProfilerActivity

    def mark():
        torch.zeros(64, device="cuda").erfinv_()
        torch.cuda.synchronize()

    mark()
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        time.sleep(0.05)
        mark()
        fn()
        mark()
        time.sleep(0.05)
    assert sum("erfinv" in e.name for e in prof.events()) == 2, "the profiler has lost kernels"
    return prof


def kernel_events(name, fn):
    """The profiler's events of kernels whose names hold `name`, of fn()."""
    return [e for e in _profile(fn).events() if name in e.name]


def kernel_grids(name, fn):
    """The work-groups of each launch of such kernels in fn(), in the order in which they started."""
    prof = _profile(fn)
    with tempfile.TemporaryDirectory() as tmp:
        path = os.path.join(tmp, "trace.json")
        prof.export_chrome_trace(path)
        with open(path) as f:
            events = json.load(f)["traceEvents"]
    found = sorted((e["ts"], e["args"]["grid"][0]) for e in events if e.get("cat") == "kernel" and name in e["name"])
    return [grid for _, grid in found]


def kernel_launches(name, fn):
    """How often kernels whose names hold `name` run in fn()."""
    return len(kernel_events(name, fn))


class Generator:
    """Greedy generation loop over the C ABI (prefill + decode steps), with
    optional teacher forcing of the first rows."""

    def __init__(self, model, batch, prefill_rows):
        self.m = model
        self.B = batch
        self.state = model.new_state(batch)
        self.ws = model.new_workspace(max(batch, prefill_rows))
        self.tok = torch.empty(batch, dtype=torch.int32, device="cuda")

    def prefill(self, prompts_dev, fanout=1, logits=None):
        self.m.prefill(prompts_dev, fanout, self.state, self.tok, logits=logits, workspace=self.ws)

    def step(self, pos, logits=None, hidden=None):
        self.m.decode_step(self.B, pos, self.tok, self.state, self.tok, logits=logits, hidden=hidden,
                           workspace=self.ws)
