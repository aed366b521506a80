"""GPU parity on rows under a vocabulary mask (a constrained decoder's finite
mask value on most tokens), where most of a row is one value."""
import numpy as np
import pytest
import torch

from tests.test_gpu_shard import check_sharded
from tests.test_gpu_verify import check_step, random_arrays, step_from_arrays

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("V", [5, 300, 8192, 8200, 25000])
def test_greedy_ties_over_whole_chunks(gpu_lib, V, dtype):
    """Greedy rows whose maximum, or whose chunk maxima, are held by many lanes
    and wavefronts at once: constant rows (the smallest token wins), rows with
    one to three tokens unmasked at ends of chunks, and a tie across chunks."""
    rng = np.random.default_rng(V)
    sls = [2, 1, 3, 0, 2, 1]
    target, draft, tokens, u_acc, u_res = random_arrays(rng, sls, V)
    rows = target.shape[0]
    keep = [0, V - 1, V // 2, min(V - 1, 8191), min(V - 1, 8192)]
    want = np.zeros(rows, np.int64)
    for r in range(rows):
        target[r] = -1e4 if r % 2 else 0.25  # a mask, or a constant row
        if r % 2:
            held = sorted({keep[r % 5], keep[(r + 1) % 5], keep[(r + 3) % 5]})
            target[r, held] = 2.0
            want[r] = held[0]
    draft[:] = -1e4
    seq = np.repeat(np.arange(len(sls)), sls)
    tokens = want[np.arange(len(seq)) + seq]  # every draft is the argmax: all accepted, the bonus row's emitted
    draft[np.arange(len(seq)), tokens] = 1.0
    step = step_from_arrays(target, draft, sls, tokens, [0.0] * len(sls), u_acc, u_res, 3, dtype)
    got, _, _ = check_step(gpu_lib, step, f"greedy ties V={V} {dtype}")
    assert got["accepted"].tolist() == sls
    bonus = np.cumsum(np.asarray(sls) + 1) - 1
    assert got["tokens"][np.arange(len(sls)), sls].tolist() == want[bonus].tolist()
    tokens[:] = (tokens + 1) % V  # none accepted: the first rejected row's argmax
    step = step_from_arrays(target, draft, sls, tokens, [0.0] * len(sls), u_acc, u_res, 3, dtype)
    got, _, _ = check_step(gpu_lib, step, f"greedy ties, rejected V={V} {dtype}")
    assert (got["accepted"] == 0).all()
    assert got["tokens"][:, 0].tolist() == want[bonus - np.asarray(sls)].tolist()


@pytest.mark.parametrize("mask", ["lowest", -1e18, -1e10, -3e9])
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("V", [3000, 8192, 8200, 25000])
def test_masked_units_of_a_bonus_row_weigh_nothing(gpu_lib, V, dtype, mask):
    """Bonus rows under a mask that covers whole units of the draw, down to the
    type's lowest value, whose product with log2(e) / T overflows or rounds by far
    more than any exponent: such units weigh nothing and are not an error."""
    value = float(torch.finfo(torch.bfloat16 if dtype == "bf16" else torch.float32).min) if mask == "lowest" else mask
    rng = np.random.default_rng(V)
    B = 15
    none = np.zeros((0, V), np.float32)
    target = np.full((B, V), value, np.float32)
    allowed = sorted({0, 700, min(8191, V - 1), min(8192, V - 1), V - 1} | set(range(8192 + 100, V, 8192)))
    for b in range(B):
        keep = allowed if b < 8 else allowed[b % 3::2]  # from 8 on, some chunks hold no token at all
        target[b, keep] = rng.normal(0, 1, len(keep))
    temps = [(0.7, 1.0, 1.3, 2.0, 0.0)[b % 5] for b in range(B)]
    step = step_from_arrays(target, none, [0] * B, [], temps, [], rng.random(B), 2, dtype)
    got, _, rep = check_step(gpu_lib, step, f"mask {mask} V={V} {dtype}")
    assert rep["errored"] == 0
    check_sharded(gpu_lib, step, gpu_lib.slice_bounds(V, 3), f"mask {mask}, slices V={V} {dtype}")
    # nothing unmasked: an error, or a token of the row
    target[:] = value
    temps = [(0.7, 1.0, 1.3, 2.0)[b % 4] for b in range(B)]
    step = step_from_arrays(target, none, [0] * B, [], temps, [], rng.random(B), 2, dtype)
    out = gpu_lib.verify(step.target, step.draft, step.sl, step.cu_sl, step.draft_tokens, step.temperature,
                         step.u_acc, step.u_res, 2)
    err, drawn = out["seq_err"].cpu().numpy(), out["tokens"][:, 0].cpu().numpy()
    assert np.isin(err, (0, 4)).all()
    assert (drawn[err != 0] == -1).all() and (drawn[err == 0] >= 0).all() and (drawn[err == 0] < V).all()
