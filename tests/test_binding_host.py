"""Host-side checks of the Python binding (no GPU needed): what it refuses before
it looks at a device pointer."""
import os
import subprocess
import sys

import pytest
import torch


@pytest.fixture(scope="module")
def dsde():
    import paper_2509_01083_amd as dsde
    dsde._bind()
    return dsde


def step_args(B=3, N=4, V=64, dtype=torch.bfloat16):
    """Arguments of dsde.step on the CPU: every check before the device one passes."""
    i32 = dict(dtype=torch.int32)
    return dict(target=torch.zeros(N + B, V, dtype=dtype), draft=torch.zeros(N, V, dtype=dtype),
                sl=torch.tensor([2, 1, 1], **i32), cu_sl=torch.tensor([0, 2, 3, 4], **i32),
                draft_tokens=torch.zeros(N, **i32), temperature=torch.ones(B), u_acc=torch.zeros(N),
                u_res=torch.zeros(B), k_max=2, hist=torch.zeros(B, 8), head=torch.zeros(B, **i32),
                count=torch.zeros(B, **i32), sl_max=torch.ones(B))


VERIFY = ("target", "draft", "sl", "cu_sl", "draft_tokens", "temperature", "u_acc", "u_res", "k_max")


def call(dsde, name, args):
    if name == "verify":
        args = {k: args[k] for k in VERIFY}
    return getattr(dsde, name)(**args)


@pytest.mark.parametrize("name", ["verify", "step", "step_static"])
def test_draft_must_match_the_target(dsde, name):
    """The kernels index draft rows with the target's element size and width: a
    draft of another type or width would be read past its end."""
    args = step_args()
    with pytest.raises(dsde.DsdeError, match="target must be a GPU tensor"):
        call(dsde, name, args)
    draft = args["draft"]
    for bad in (draft.float(), draft.half(), draft[:, :-1].contiguous(), torch.zeros(4, 65, dtype=draft.dtype)):
        with pytest.raises(dsde.DsdeError, match="draft logits must match the target's dtype and vocabulary"):
            call(dsde, name, dict(args, draft=bad))
    with pytest.raises(dsde.DsdeError, match="draft has too few dimensions"):
        call(dsde, name, dict(args, draft=draft[:, 0].contiguous()))


def test_step_takes_an_empty_draft_of_any_type(dsde):
    """Nothing drafted: the draft is not read, and step never asked for its type."""
    args = step_args(N=0)
    for draft in (torch.zeros(0, 64), torch.zeros(0, 0, dtype=torch.bfloat16), None):
        with pytest.raises(dsde.DsdeError, match="target must be a GPU tensor"):
            call(dsde, "step", dict(args, draft=draft))


class Recorder(torch.overrides.TorchFunctionMode):
    """The stream in force at every allocation of a call."""

    def __init__(self, stack):
        super().__init__()
        self.stack, self.seen = stack, []

    def __torch_function__(self, func, types, args=(), kwargs=None):
        if func in (torch.empty, torch.Tensor.contiguous):
            self.seen.append(self.stack[-1])
        return func(*args, **(kwargs or {}))


class FakeStream:
    cuda_stream = 77


class RawStream:  # an object with the raw handle alone
    cuda_stream = 78


class FakeNative:
    def __getattr__(self, name):
        return lambda *args: None


def calls_with_own_buffers(dsde):
    """Every call that makes buffers of its own, as (name, function of the stream, allocations)."""
    a = step_args()
    rows = tuple(a[k] for k in VERIFY)
    batch, k = rows[2:8], a["k_max"]
    ring = (a["hist"], a["head"], a["count"])
    u8 = dict(dtype=torch.uint8)
    parts, jobs = torch.zeros(2, 4, 64, **u8), torch.zeros(3, 44, **u8)
    err, ws = torch.zeros(3, dtype=torch.int32), torch.zeros(4096, **u8)
    out = dict(accepted=err, tokens=err, kld=a["u_acc"], seq_err=err, jobs=jobs)
    return [
        ("verify", lambda s: dsde.verify(*rows, stream=s), 5),
        ("verify, entropy", lambda s: dsde.verify(*rows, out=dict(out), draft_entropy=True, workspace=ws, stream=s), 1),
        ("verify, workspace", lambda s: dsde.verify(*rows, out=out, stream=s), 1),
        ("step", lambda s: dsde.step(*rows, *ring, a["sl_max"], draft_entropy=True, stream=s), 14),
        ("step_static", lambda s: dsde.step_static(*rows, *ring, a["sl_max"], stream=s), 12),
        ("kld_signal", lambda s: dsde.kld_signal(rows[2], rows[3], a["u_acc"], *ring, stream=s), 6),
        ("next_sl", lambda s: dsde.next_sl(a["u_res"], a["u_res"], a["sl_max"], stream=s), 4),
        ("shard_stats", lambda s: dsde.shard_stats(*rows[:2], 0, 64, *batch[:4], k, ws, stream=s), 2),
        ("shard_accept", lambda s: dsde.shard_accept(torch.zeros(2, 6, 64, **u8), 64, *batch, k, err, stream=s), 5),
        ("shard_accept_step", lambda s: dsde.shard_accept_step(parts, 64, *batch, k, err, *ring, a["sl_max"],
                                                               stream=s), 12),
        ("shard_draw_mass", lambda s: dsde.shard_draw_mass(*rows[:2], 0, parts[0], jobs, k, ws, stream=s), 1),
        ("shard_draw_pick", lambda s: dsde.shard_draw_pick(0, jobs, *rows[:2], 0, jobs, k, err, err, err, ws,
                                                           stream=s), 1),
    ]


@pytest.mark.parametrize("stream", [None, FakeStream(), RawStream()])
def test_own_buffers_belong_to_the_calls_stream(dsde, monkeypatch, stream):
    """A workspace that a call makes goes back to the allocator when the call
    returns, with its kernels still to run: unless it was made on their stream,
    the next tensor of the current stream can take its memory from under them."""
    stack = ["current"]

    class On:
        def __init__(self, s):
            self.s = s

        def __enter__(self):
            stack.append(self.s)

        def __exit__(self, *exc):
            stack.pop()

    monkeypatch.setattr(dsde, "_native", FakeNative())
    monkeypatch.setattr(torch.cuda, "stream", On)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: "current")
    monkeypatch.setattr(torch.cuda, "Stream", FakeStream)
    monkeypatch.setattr(torch.cuda, "ExternalStream", lambda handle: handle)
    want = "current" if stream is None else 78 if isinstance(stream, RawStream) else stream
    for name, f, n in calls_with_own_buffers(dsde):
        with Recorder(stack) as seen:
            f(stream)
        assert seen.seen == [want] * n, name
        assert stack == ["current"]
    with Recorder(stack) as seen:  # calibrate_sl_max calls the library itself, which refuses the CPU's tensors
        with pytest.raises(dsde.DsdeError, match="GPU tensor"):
            dsde.calibrate_sl_max(dsde.new_calibration_state(3, device="cpu"), stream=stream)
    assert seen.seen == [want]


def test_the_loaded_library_serves_every_call(dsde, tmp_path):
    """load(path) decides which library runs, for the marshalled calls too: with a
    copy loaded from elsewhere the package's own is not even mapped."""
    copy = tmp_path / "copy_of_the_library.so"
    copy.write_bytes(open(dsde.LIB_PATH, "rb").read())
    code = ("import sys, torch, paper_2509_01083_amd as d\n"
            "d.load(sys.argv[1]); d._bind()\n"
            "print([l.split()[-1] for l in open('/proc/self/maps') if 'r-xp' in l and l.rstrip().endswith('.so')])\n")
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    maps = subprocess.run([sys.executable, "-c", code, str(copy)], cwd=root, capture_output=True, text=True,
                          check=True).stdout
    assert str(copy) in maps
    assert dsde.LIB_PATH not in maps
