"""The binding's marshalling: the stream a call runs on, and what it refuses."""
import collections

import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

NAMES = ("accepted", "tokens", "kld", "mu_last", "var_short", "var_long", "wvir", "sf", "sl_hat", "sl_cap", "sl_next",
         "seq_err")


def _case():
    cfg = dict(W.CONFIGS["greedy"], B=12, V=4096)
    step = W.make_step(cfg, seed=3, device="cuda")
    st = W.make_signal_state(cfg, seed=3, device="cuda")
    args = (step.target, step.draft, step.sl, step.cu_sl, step.draft_tokens, step.temperature, step.u_acc, step.u_res,
            step.k_max)
    return step, st, args


def _ring(st):
    return st.hist.clone(), st.head.clone(), st.count.clone()


def test_calls_follow_the_current_stream(gpu_lib):
    """Captured on a side stream (a call on any other stream would not be in the
    graph) and given a stream outright: the bits of a call on the default one."""
    step, st, args = _case()
    want = gpu_lib.step(*args, *_ring(st), st.sl_max)
    torch.cuda.synchronize()
    ring = _ring(st)
    ws = gpu_lib.new_workspace(step.B, step.N, step.V, step.k_max)
    out = {k: torch.zeros_like(want[k]) for k in NAMES}
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())  # the copies and the fills above
    with torch.cuda.stream(side):
        gpu_lib.step(*args, *ring, st.sl_max, out=out, workspace=ws)
    side.synchronize()
    for k in NAMES:
        assert torch.equal(out[k].view(torch.int32), want[k].view(torch.int32)), k
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        gpu_lib.step(*args, *ring, st.sl_max, out=out, workspace=ws)
    for _ in range(3):
        for dst, src in zip(ring, (st.hist, st.head, st.count)):
            dst.copy_(src)
        for k in NAMES:
            out[k].zero_()
        graph.replay()
        torch.cuda.synchronize()
        for k in NAMES:
            assert torch.equal(out[k].view(torch.int32), want[k].view(torch.int32)), k
    ring = _ring(st)
    side.wait_stream(torch.cuda.current_stream())
    given = gpu_lib.step(*args, *ring, st.sl_max, stream=side)  # outputs and workspace made by the call
    taken = [torch.full_like(ws, 255) for _ in range(4)]  # the current stream's next tensors of that size
    side.synchronize()
    for k in NAMES:
        assert torch.equal(given[k].view(torch.int32), want[k].view(torch.int32)), k
    del taken


def test_refusals(gpu_lib):
    step, st, args = _case()
    bad = [
        (2, step.sl.cpu(), "sl must be a GPU tensor"),
        (2, step.sl.long(), "sl must be torch.int32, got torch.int64"),
        (3, step.cu_sl[:-1].contiguous(), "cu_sl has"),
        (5, torch.stack([step.temperature] * 2, 1)[:, 0], "temperature must be contiguous"),
        (0, step.target[:-1], "target has"),
        (0, step.target.half(), "logits must be"),
        (6, None, "invalid argument"),
    ]
    for i, value, text in bad:
        a = list(args)
        a[i] = value
        with pytest.raises(gpu_lib.DsdeError, match=text):
            gpu_lib.step(*a, *_ring(st), st.sl_max)
    out = gpu_lib.step(*args, *_ring(st), st.sl_max)
    del out["sl_hat"]
    with pytest.raises(KeyError, match="sl_hat"):
        gpu_lib.step(*args, *_ring(st), st.sl_max, out=out)
    small = torch.empty(64, dtype=torch.uint8, device="cuda")
    with pytest.raises(gpu_lib.DsdeError, match="workspace too small"):
        gpu_lib.step(*args, *_ring(st), st.sl_max, workspace=small)
    with pytest.raises(gpu_lib.DsdeError, match="workspace must be a GPU tensor"):
        gpu_lib.step(*args, *_ring(st), st.sl_max, workspace=False)
    torch.cuda.synchronize()


def test_outputs_in_any_mapping(gpu_lib):
    """Outputs are looked up by key: a mapping that is no dict, or a dict with a
    lookup of its own, serves as well as a dict."""
    step, st, args = _case()
    want = gpu_lib.step(*args, *_ring(st), st.sl_max)

    class Upper(dict):
        def __getitem__(self, key):
            return super().__getitem__(key.upper())

    for out in (collections.UserDict({k: torch.zeros_like(want[k]) for k in NAMES}),
                Upper({k.upper(): torch.zeros_like(want[k]) for k in NAMES})):
        got = gpu_lib.step(*args, *_ring(st), st.sl_max, out=out)
        torch.cuda.synchronize()
        assert got is out
        for k in NAMES:
            assert torch.equal(out[k].view(torch.int32), want[k].view(torch.int32)), k
    with pytest.raises(KeyError):
        gpu_lib.step(*args, *_ring(st), st.sl_max, out=collections.UserDict())
