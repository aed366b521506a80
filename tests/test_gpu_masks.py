"""GPU parity on rows under a vocabulary mask (a constrained decoder's finite
mask value on most tokens), where most of a row is one value."""
import numpy as np
import pytest

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
