"""Host-side checks of the Python binding (no GPU needed): what it refuses before
it looks at a device pointer."""
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
