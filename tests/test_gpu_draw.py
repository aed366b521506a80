"""GPU parity of the draw where its division of the work changes: rows that end
at, before and after a unit of 2048 logits and a sub-block of 512, one logit
row per workgroup and several, more than 64 units (two rounds of the unit
search), and batches drawn in more than one pass over the workspace's cells.
The oracle and the tie rules are those of the other parity tests."""
import numpy as np
import pytest
import torch

from tests.test_gpu_verify import check_step, random_arrays, step_from_arrays

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("V", [504, 512, 2040, 2047, 2048, 2049, 2056, 4608, 131072, 131080, 133121])
@pytest.mark.parametrize("B", [1, 5])
def test_draw_unit_edges(gpu_lib, V, dtype, B):
    rng = np.random.default_rng(V + B)
    sls = [2, 0, 3, 1, 1][:B]
    target, draft, tokens, u_acc, u_res = random_arrays(rng, sls, V, sigma=1.0, noise=0.5)
    u_res = np.array([0.999999, 0.0, 0.9, 0.5, 0.05], np.float32)[:B]
    temps = [1.0, 0.7, 0.0, 1.3, 1.0][:B]
    step = step_from_arrays(target, draft, sls, tokens, temps, u_acc, u_res, 3, dtype)
    check_step(gpu_lib, step, f"draw units V={V} B={B} {dtype}")


def test_draw_in_two_passes(gpu_lib):
    """More sequences than one pass of the draw kernels holds (32,768): the
    second pass reuses the cells of the first."""
    rng = np.random.default_rng(5)
    B, V = 32768 + 77, 24
    sls = rng.integers(0, 3, B).tolist()
    target, draft, tokens, u_acc, u_res = random_arrays(rng, sls, V, noise=0.8)
    temps = rng.choice([0.0, 0.7, 1.0], B).tolist()
    step = step_from_arrays(target, draft, sls, tokens, temps, u_acc, u_res, 2)
    _, _, rep = check_step(gpu_lib, step, f"two passes B={B} V={V}")
    assert rep["compared"] >= 0.9 * B
    # the fused step takes its SL rule from the last pass: same bits as the separate calls
    dev = "cuda"
    ring = [(torch.zeros(B, 8, device=dev), torch.zeros(B, dtype=torch.int32, device=dev),
             torch.zeros(B, dtype=torch.int32, device=dev)) for _ in range(2)]
    smax = torch.full((B,), 8.0, device=dev)
    args = (step.target, step.draft, step.sl, step.cu_sl, step.draft_tokens, step.temperature, step.u_acc, step.u_res,
            step.k_max)
    got = gpu_lib.step(*args, *ring[0], smax)
    ver = gpu_lib.verify(*args)
    sig = gpu_lib.kld_signal(step.sl, step.cu_sl, ver["kld"], *ring[1])
    rule = gpu_lib.next_sl(sig["sf"], sig["wvir"], smax, 2.0, step.k_max)
    for k in ("accepted", "tokens"):
        assert torch.equal(got[k], ver[k]), k
    for k in ("sl_hat", "sl_cap"):
        assert torch.equal(got[k].view(torch.int32), rule[k].view(torch.int32)), k
    assert torch.equal(got["sl_next"], rule["sl_next"])


@pytest.mark.parametrize("B", [1024, 1025])
def test_draw_around_the_merged_workgroups(gpu_lib, B):
    """On both sides of the number of sequences above which the workgroups that
    write the outputs stream as well, with rows of two workgroups' units there."""
    rng = np.random.default_rng(B)
    V = 100008
    sls = (rng.integers(0, 3, B) * (rng.random(B) < 0.2)).tolist()
    # peaked rows: in flat ones (sigma 1) a token weighs about 1e-5, of which the tie
    # band around its boundaries (1e-6 on each side) takes a fifth
    target, draft, tokens, u_acc, u_res = random_arrays(rng, sls, V, sigma=4.0, noise=1.5)
    temps = rng.choice([0.0, 0.7, 1.0], B).tolist()
    step = step_from_arrays(target, draft, sls, tokens, temps, u_acc, u_res, 2)
    _, _, rep = check_step(gpu_lib, step, f"merged workgroups B={B} V={V}")
    assert rep["compared"] >= 0.9 * B


@pytest.mark.parametrize("B,k_max,V", [(64, 8, 8192), (1024, 4, 9000), (1024, 5, 8192), (1025, 1, 512)])
def test_statistics_with_and_without_the_setup_kernel(gpu_lib, B, k_max, V):
    """Batches on both sides of the rule that drops the set-up kernel (at most
    4,096 workgroups past the sequences' ends, at most 1,024 sequences), and a
    broken layout on each, which flags every sequence."""
    rng = np.random.default_rng(B + k_max)
    sls = rng.integers(0, k_max + 1, B).tolist()
    target, draft, tokens, u_acc, u_res = random_arrays(rng, sls, V, sigma=1.0, noise=0.5)
    temps = rng.choice([0.0, 0.7, 1.0], B).tolist()
    step = step_from_arrays(target, draft, sls, tokens, temps, u_acc, u_res, k_max)
    _, _, rep = check_step(gpu_lib, step, f"set-up rule B={B} k_max={k_max} V={V}")
    assert rep["compared"] >= 0.9 * B
    step.cu_sl[B // 2] += 1
    got = gpu_lib.verify(step.target, step.draft, step.sl, step.cu_sl, step.draft_tokens, step.temperature,
                         step.u_acc, step.u_res, k_max)
    torch.cuda.synchronize()
    assert (got["seq_err"] == 1).all() and (got["accepted"] == 0).all() and (got["tokens"] == -1).all()


def _shifted(t, by):
    """A contiguous copy of t that starts `by` elements into its allocation."""
    flat = torch.empty(t.numel() + by, dtype=t.dtype, device=t.device)
    flat[by:] = t.reshape(-1)
    return flat[by:].view(t.shape)


@pytest.mark.parametrize("dtype,widths", [("bf16", (8, 9, 15, 23, 8185, 8191, 8193, 8199, 10247)),
                                          ("fp32", (4, 5, 7, 11, 8189, 8191, 8193, 8195, 10243))])
def test_unaligned_rows(gpu_lib, dtype, widths):
    """Row widths that are no whole number of 16-byte loads, from one load up:
    the last load of a row starts inside the one before it."""
    for V in widths:
        rng = np.random.default_rng(V)
        sls = [3, 0, 1, 4, 2]
        target, draft, tokens, u_acc, u_res = random_arrays(rng, sls, V, sigma=1.0, noise=0.5)
        tokens[:4] = [V - 1, V - 2, 0, V - 1]  # logits gathered from the moved last load
        step = step_from_arrays(target, draft, sls, tokens, [1.0, 0.7, 0.0, 1.3, 0.0], u_acc, u_res, 4, dtype)
        check_step(gpu_lib, step, f"unaligned rows V={V} {dtype}")


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("V", [64, 2048, 8192, 10240, 20000])
def test_row_alignment_changes_no_bit(gpu_lib, V, dtype):
    """The same logits from a 16-byte aligned base and from one shifted by
    single elements (target and draft by different ones)."""
    rng = np.random.default_rng(V)
    sls = [3, 0, 1, 4, 2]
    target, draft, tokens, u_acc, u_res = random_arrays(rng, sls, V, sigma=1.0, noise=0.5)
    step = step_from_arrays(target, draft, sls, tokens, [1.0, 0.7, 0.0, 1.3, 0.0], u_acc, u_res, 4, dtype)
    rest = (step.sl, step.cu_sl, step.draft_tokens, step.temperature, step.u_acc, step.u_res, 4)

    def run(target, draft):
        lse = torch.zeros(step.N, 2, dtype=torch.float64, device="cuda")
        out = gpu_lib.verify(target, draft, *rest, row_lse=lse, draft_entropy=True)
        return dict(out, row_lse=lse)
    want = run(step.target, step.draft)
    for a, b in ((1, 0), (0, 3), (2, 1)):
        got = run(_shifted(step.target, a), _shifted(step.draft, b))
        for k in want:
            x, y = got[k], want[k]
            if x.dtype.is_floating_point:
                x, y = x.view(torch.uint8), y.view(torch.uint8)
            assert torch.equal(x, y), f"{k} differs at offsets {a}, {b}"


@pytest.mark.parametrize("G", [8, 9, 17, 33, 65])
def test_shard_counts_around_the_group_sizes(gpu_lib, G):
    """The sharded acceptance gives each position a group of 8, 16, 32 or 64
    lanes, one slice per lane; more slices than lanes take several each."""
    from tests.test_gpu_shard import check_sharded
    rng = np.random.default_rng(G)
    V = 16 * G + 3
    sls = [5, 0, 1, 40, 3]
    target, draft, tokens, u_acc, u_res = random_arrays(rng, sls, V, sigma=1.0, noise=0.3)
    step = step_from_arrays(target, draft, sls, tokens, [1.0, 0.7, 0.0, 1.3, 0.0], u_acc, u_res, 40)
    bounds = [16 * g for g in range(G)] + [V]
    check_sharded(gpu_lib, step, list(zip(bounds[:-1], bounds[1:])), f"{G} slices")


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("V", [5, 1001, 2048, 3000, 10248, 2048 * 70 + 8, 2048 * 70 + 3])
def test_draw_without_residual_mass(gpu_lib, V, dtype):
    """A rejected pair whose residual has no mass at all: the draw falls back to p of
    the target row.  Target and draft are equal (one weight on some tokens, none on
    the rest, so that p - q is exactly 0) but for the drafted token, of weight 0 in
    both and e times more likely under the draft, which u = 0.9 rejects.  u' lies
    in the middle of each token's interval."""
    from tests.test_gpu_shard import check_sharded
    rng = np.random.default_rng(V)
    edges = {0, 1, 511, 512, 2047, 2048, 2049, 8191, 8192, 64 * 2048 - 1, 64 * 2048, V // 3, V - 2, V - 1}
    x = 2 if V < 100 else 700  # the drafted token
    hot = np.array(sorted(t for t in edges if t < V and t != x))
    H = len(hot)
    B = 2 * H
    sls = [1] * H + [2] * H  # the second half accepts a draft first
    seq = np.repeat(np.arange(B), sls)
    N = len(seq)
    target, draft = np.full((N + B, V), -100.0, np.float32), np.full((N, V), -100.0, np.float32)
    target[:, hot] = 0.0
    draft[:, hot] = 0.0
    tokens, u_acc = np.full(N, x), np.full(N, 0.9, np.float32)
    for b in range(H, B):
        first = H + 2 * (b - H)
        tokens[first], u_acc[first] = hot[b % H], 0.5
    at = np.nonzero(tokens == x)[0]
    draft[at, x] = -99.0
    u_res = ((np.arange(B) % H + 0.5) / H).astype(np.float32)
    temps = [1.0, 0.9] * H
    step = step_from_arrays(target, draft, sls, tokens, temps, u_acc, u_res, 2, dtype)
    want = [0] * H + [1] * H

    def check(got, rep):
        assert got["accepted"].tolist() == want and rep["compared"] == B
        assert got["tokens"][np.arange(B), want].tolist() == hot[np.arange(B) % H].tolist()
    got, _, rep = check_step(gpu_lib, step, f"no residual mass V={V} {dtype}")
    check(got, rep)
    for G in (1, 3, 70):
        slices = gpu_lib.slice_bounds(V, G)
        got, _, rep = check_sharded(gpu_lib, step, slices, f"no residual mass, {len(slices)} slices V={V} {dtype}")
        check(got, rep)
