"""The signal's rings: what their unheld slots may hold, and rings larger than a
wavefront keeps in registers, through every call that updates the signal
(dsde_kld_signal, dsde_step, dsde_step_static, dsde_shard_accept_step)."""
import numpy as np
import pytest
import torch

import oracle
from tests.test_gpu_signal import close, compare_signal
from tests.test_gpu_verify import random_arrays, step_from_arrays

pytestmark = pytest.mark.gpu

SIGNAL = ("mu_last", "var_short", "var_long", "wvir", "sf", "sl_hat", "sl_cap", "sl_next", "seq_err")
CALLS = ("kld_signal", "step", "step_static", "shard_accept_step")
SLS = [3, 0, 1, 4, 0, 2, 1, 3]


def make_step(seed=1):
    rng = np.random.default_rng(seed)
    target, draft, tokens, u_acc, u_res = random_arrays(rng, SLS, 512, sigma=1.0, noise=0.4)
    return step_from_arrays(target, draft, SLS, tokens, [1.0] * len(SLS), u_acc, u_res, 4)


def make_ring(W_, counts, unheld, seed=2):
    """Rings with `counts` entries held at various heads; every other slot holds `unheld`."""
    rng = np.random.default_rng(seed)
    B = len(counts)
    head = rng.integers(0, W_, B).astype(np.int32)
    hist = np.full((B, W_), unheld, np.float32)
    for b, c in enumerate(counts):
        hist[b, (head[b] - 1 - np.arange(c)) % W_] = rng.gamma(0.6, 0.5, c)
    return [torch.as_tensor(x, device="cuda") for x in (hist, head, np.asarray(counts, np.int32))]


def run(gpu_lib, call, step, ring, n_short=10, n_long=30):
    """Signal, rule and updated ring of one call on a copy of `ring`."""
    ring = [t.clone() for t in ring]
    rows = (step.sl, step.cu_sl, step.draft_tokens, step.temperature, step.u_acc, step.u_res, step.k_max)
    smax = torch.full((step.B,), 9.0, device="cuda")
    win = dict(n_short=n_short, n_long=n_long)
    if call in ("step", "step_static"):
        out = getattr(gpu_lib, call)(step.target, step.draft, *rows, *ring, smax, **win)
    elif call == "shard_accept_step":
        base = gpu_lib.verify_sharded(step.target, step.draft, *rows, gpu_lib.slice_bounds(step.V, 2))
        out = gpu_lib.shard_accept_step(base["parts"], step.V, *rows, base["shard_seq_err"][0].clone(), *ring, smax,
                                        **win)
    else:
        v = gpu_lib.verify(step.target, step.draft, *rows)
        s = gpu_lib.kld_signal(step.sl, step.cu_sl, v["kld"], *ring, **win)
        r = gpu_lib.next_sl(s["sf"], s["wvir"], smax, 2.0, step.k_max)
        out = {**r, **s, "seq_err": v["seq_err"] | s["seq_err"] | r["seq_err"]}
    torch.cuda.synchronize()
    return {k: out[k].cpu().numpy() for k in SIGNAL}, [t.cpu().numpy() for t in ring]


def same_bits(a, b):
    return np.array_equal(a.view(np.uint32), b.view(np.uint32))


@pytest.mark.parametrize("unheld", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("W_", [8, 32, 100])
@pytest.mark.parametrize("call", CALLS)
def test_unheld_slots_are_not_used(gpu_lib, call, W_, unheld):
    """A slot the ring does not hold may contain anything (a caller may zero head
    and count alone): the bits of a ring that holds zeros there."""
    step = make_step()
    counts = [0, 0, 5, 5, 3, 1, W_ - 1, W_]
    want, ring_want = run(gpu_lib, call, step, make_ring(W_, counts, 0.0))
    got, ring_got = run(gpu_lib, call, step, make_ring(W_, counts, unheld))
    assert (want["seq_err"] == 0).all()
    for k in SIGNAL:
        assert same_bits(got[k], want[k]), k
    assert np.array_equal(ring_got[1], ring_want[1]) and np.array_equal(ring_got[2], ring_want[2])
    for b, c in enumerate(ring_got[2]):
        held = (ring_got[1][b] - 1 - np.arange(c)) % W_
        assert same_bits(ring_got[0][b, held], ring_want[0][b, held])


@pytest.mark.parametrize("call", CALLS)
def test_entries_past_the_short_window_leave_it_alone(gpu_lib, call):
    """A non-finite entry that only the long window holds: the short variance is
    that of a finite entry there, the long one is NaN."""
    step = make_step()
    ring = make_ring(16, [16] * len(SLS), 0.0)
    want, _ = run(gpu_lib, call, step, ring, n_short=3, n_long=12)
    hist, head = ring[0].cpu().numpy(), ring[1].cpu().numpy()
    for b in range(len(SLS)):
        hist[b, (head[b] - 6) % 16] = np.inf
    got, _ = run(gpu_lib, call, step, [torch.as_tensor(hist, device="cuda"), *ring[1:]], n_short=3, n_long=12)
    assert same_bits(got["var_short"], want["var_short"])
    assert np.isnan(got["var_long"]).all()


@pytest.mark.parametrize("W_, n_short, n_long", [(64, 10, 64), (65, 10, 30), (100, 70, 90), (256, 10, 200),
                                                 (257, 64, 65), (300, 10, 300)])
def test_rings_above_a_wavefronts_registers(gpu_lib, W_, n_short, n_long):
    """Rings of more than 64 entries (the fused step keeps 64 in registers, the other
    calls 256) and windows of more than 64: the oracle's signal, and the same bits
    from every call."""
    step = make_step()
    counts = [0, 1, 5, 63, 64, 65 % (W_ + 1), W_ - 1, W_]
    ring = make_ring(W_, counts, 0.0)
    want, ring_want = run(gpu_lib, "kld_signal", step, ring, n_short, n_long)
    v = gpu_lib.verify(step.target, step.draft, step.sl, step.cu_sl, step.draft_tokens, step.temperature, step.u_acc,
                       step.u_res, step.k_max)
    ref = oracle.kld_signal(step.sl.cpu().numpy(), step.cu_sl.cpu().numpy(), v["kld"].cpu().numpy().astype(np.float64),
                            *[t.cpu().numpy() for t in ring], n_short, n_long)
    compare_signal(want, ref, f"ring {W_}")
    close(ring_want[0], ref["hist"], rel=1e-7, label="ring")  # one rounding to fp32
    assert np.array_equal(ring_want[1], ref["head"]) and np.array_equal(ring_want[2], ref["count"])
    for call in CALLS[1:3]:
        got, ring_got = run(gpu_lib, call, step, ring, n_short, n_long)
        for k in SIGNAL:
            assert same_bits(got[k], want[k]), (call, k)
        for a, b in zip(ring_got, ring_want):
            assert same_bits(a, b), call
    # the sharded KLD is summed slice by slice: its own signal, from the separate calls on it
    base = gpu_lib.verify_sharded(step.target, step.draft, step.sl, step.cu_sl, step.draft_tokens, step.temperature,
                                  step.u_acc, step.u_res, step.k_max, gpu_lib.slice_bounds(step.V, 2))
    ring_a = [t.clone() for t in ring]
    sig = gpu_lib.kld_signal(step.sl, step.cu_sl, base["kld"], *ring_a, n_short, n_long)
    got, ring_got = run(gpu_lib, "shard_accept_step", step, ring, n_short, n_long)
    for k in ("mu_last", "var_short", "var_long", "wvir", "sf"):
        assert same_bits(got[k], sig[k].cpu().numpy()), k
    for a, b in zip(ring_got, ring_a):
        assert same_bits(a, b.cpu().numpy())
