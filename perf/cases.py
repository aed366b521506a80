"""The verification work whose speed is followed: a list of typical calls, how to
draw more of the same ranges, and how to make, run and check one.

A case is a dict of plain values:

  call     step      dsde.step, the fused call of a serving loop
           calls     dsde.verify, calibration_update, kld_signal and next_sl one after
                     another, as a program that calibrates SL_max while serving does
           verify    dsde.verify alone with the optional entropy and log-normalisers
           shard     one GPU's four vocabulary-shard calls of a step (the other
                     shards' exchanged records are made by prepare)
  B, V     sequences, vocabulary (for shard: the whole vocabulary)
  lo, hi   speculation lengths are uniform in lo..hi (hi is also k_max)
  dtype    bf16 or fp32 logits
  temp     one: T = 1; mixed: 0.7 and 1.0 in turn; greedy: 0; half: 0 and 1 in turn
  sigma_lo, sigma_hi   per-sequence noise of the draft logits around the target's;
           weak: true takes 0.5 z + noise instead (a drafter that agrees poorly)
  W        ring capacity of the signal; filled: whether the rings start full
  G        shards (shard only)

Logits are Gaussian with a Zipf rank bias per row, drafted tokens are sampled
from the tempered draft distribution (greedy sequences: its argmax).
"""
import math
import random

import torch

import paper_2509_01083_amd as dsde

SL_MIN, N_SHORT, N_LONG, DELTA, EPS = 2.0, 10, 30, 0.85, 1e-6
ROWS = 256  # rows made or checked at once


def _case(name, call, B, V, lo, hi, dtype="bf16", temp="one", sigma=(0.2, 4.0), weak=False, W=32, filled=True, G=0):
    c = dict(call=call, B=B, V=V, lo=lo, hi=hi, dtype=dtype, temp=temp, sigma_lo=sigma[0], sigma_hi=sigma[1],
             weak=weak, W=W, filled=filled, G=G)
    return dict(c, name=name) if name else c


def listed():
    return [
        # one user's request: nothing but latency
        _case("single", "step", 1, 128256, 5, 5),
        # a handful of sequences on fp32 logits (the smallest benchmark workload)
        _case("tiny_fp32", "step", 4, 32000, 4, 4, dtype="fp32", sigma=(1.0, 1.0), W=8),
        # a small server: 32 sequences on the large vocabulary (also one GPU's share
        # of the 256-sequence batch split eight ways)
        _case("b32", "step", 32, 128256, 1, 8, temp="mixed"),
        # a mid-sized batch on a 32,000-token vocabulary
        _case("b64", "step", 64, 32000, 1, 8, sigma=(0.3, 3.0), W=16),
        # a sampler that upcasts its logits to fp32
        _case("b64_fp32", "step", 64, 128256, 1, 8, dtype="fp32", temp="mixed"),
        # a vocabulary whose rows are not 16-byte aligned; some sequences draft
        # nothing, half are greedy; entropy and log-normalisers wanted
        _case("odd_vocab", "verify", 64, 50257, 0, 8, temp="half", sigma=(0.3, 3.0)),
        # calibration while serving: the separate calls, close drafts
        _case("calls", "calls", 256, 32000, 1, 8, sigma=(0.05, 0.6)),
        # the benchmark's workload: 256 sequences, large vocabulary
        _case("b256", "step", 256, 128256, 1, 8, temp="mixed"),
        # the same batch at temperature 0
        _case("b256_greedy", "step", 256, 128256, 1, 8, temp="greedy"),
        # many sequences whose lengths the controller has cut to 2 or 3
        _case("b1024_short", "step", 1024, 128256, 2, 3),
        # long drafts from a drafter that agrees poorly: the most rows
        _case("b512_long", "step", 512, 152064, 1, 16, sigma=(3.0, 3.0), weak=True),
        # one of eight GPUs of a target model split by vocabulary
        _case("shard8", "shard", 256, 128256, 1, 8, temp="mixed", G=8),
    ]


MOST_BYTES = 2 * 512 * 8.5 * 152064 * 2  # of b512_long's drafted rows


def draw(rng):
    call = rng.choice(["step", "step", "step", "verify", "calls", "shard"])
    B = round(math.exp(rng.uniform(0, math.log(1024))))
    V = round(math.exp(rng.uniform(math.log(8192), math.log(152064))))
    dtype = rng.choice(["bf16", "bf16", "bf16", "fp32"])
    if rng.random() < 0.6:
        V -= V % 64
    hi = rng.choice([2, 3, 4, 5, 8, 8, 16])
    lo = rng.choice([0, 1, 2, hi])
    lo = max(min(lo, hi), 1 if call == "shard" else 0)
    while 2 * B * (lo + hi) / 2 * V * (2 if dtype == "bf16" else 4) > MOST_BYTES:
        B = (B + 1) // 2
    weak = rng.random() < 0.2
    sigma = (3.0, 3.0) if weak else rng.choice([(0.2, 4.0), (0.3, 3.0), (0.05, 0.6)])
    return _case(None, call, B, V, lo, hi, dtype, rng.choice(["one", "mixed", "greedy", "half"]), sigma, weak,
                 rng.choice([8, 16, 32, 32]), rng.random() < 0.7, rng.choice([2, 4, 8]) if call == "shard" else 0)


def _lengths(case, seed=None):
    """The case's speculation lengths (their sum does not depend on the seed, their order does)."""
    r = random.Random(repr(sorted((k, v) for k, v in case.items() if k != "name")))
    sl = [r.randint(case["lo"], case["hi"]) for _ in range(case["B"])]
    if seed is not None:
        random.Random(seed).shuffle(sl)
    return sl


def _temperatures(case):
    two = {"one": (1.0, 1.0), "mixed": (0.7, 1.0), "greedy": (0.0, 0.0), "half": (0.0, 1.0)}[case["temp"]]
    return [two[b % 2] for b in range(case["B"])]


def _inputs(case, seed):
    dev = torch.device("cuda")
    g = torch.Generator(device=dev)
    g.manual_seed(1_000_003 * seed + 17)
    r = random.Random(seed)
    B, V, W = case["B"], case["V"], case["W"]
    sl = _lengths(case, seed)
    cu = [0]
    for s in sl:
        cu.append(cu[-1] + s)
    N = cu[-1]
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    temp = _temperatures(case)
    sigma = [r.uniform(case["sigma_lo"], case["sigma_hi"]) for _ in range(B)]
    seq = [b for b in range(B) for _ in range(sl[b])]
    f32 = dict(dtype=torch.float32, device=dev)

    def rand(*shape):
        return torch.rand(shape, generator=g, **f32)

    def randn(*shape):
        return torch.randn(shape, generator=g, **f32)

    # target rows: Gaussian logits plus -s ln(rank) under a random affine ranking per row
    steps = [r.randrange(1, V) for _ in range(N + B)]
    steps = torch.tensor([a if math.gcd(a, V) == 1 else 1 for a in steps], device=dev)[:, None]
    shift = torch.randint(0, V, (N + B, 1), generator=g, device=dev)
    ids = torch.arange(V, device=dev)[None, :]
    target = torch.empty((N + B, V), dtype=dt, device=dev)
    for i in range(0, N + B, ROWS):
        j = min(i + ROWS, N + B)
        rank = (steps[i:j] * ids + shift[i:j]) % V + 1
        target[i:j] = 4.0 * randn(j - i, V) - 1.05 * rank.float().log()
    # draft rows and drafted tokens
    draft = torch.empty((N, V), dtype=dt, device=dev)
    tokens = torch.empty(N, dtype=torch.int32, device=dev)
    rows = torch.tensor([k + b for k, b in enumerate(seq)], dtype=torch.int64, device=dev)
    noise = torch.tensor([sigma[b] for b in seq], **f32)[:, None]
    t_row = torch.tensor([temp[b] for b in seq], **f32)[:, None]
    for i in range(0, N, ROWS):
        j = min(i + ROWS, N)
        z = target[rows[i:j]].float()
        draft[i:j] = (0.5 * z if case["weak"] else z) + noise[i:j] * randn(j - i, V)
        gumbel = -torch.log(-torch.log(rand(j - i, V).clamp_(min=1e-30)))
        t = t_row[i:j]
        tokens[i:j] = torch.argmax(draft[i:j].float() / torch.where(t > 0, t, 1.0) + gumbel * (t > 0), dim=1).int()
    hist = torch.zeros((B, W), **f32)
    head = torch.zeros(B, dtype=torch.int32, device=dev)
    count = torch.zeros(B, dtype=torch.int32, device=dev)
    if case["filled"]:
        hist = torch.exp(math.log(0.2) + 2.0 * rand(B, 1) + 0.5 * randn(B, W))
        head = torch.randint(0, W, (B,), generator=g, device=dev, dtype=torch.int32)
        count.fill_(W)
    return dict(target=target, draft=draft, sl=torch.tensor(sl, dtype=torch.int32, device=dev),
                cu_sl=torch.tensor(cu, dtype=torch.int32, device=dev), draft_tokens=tokens,
                temperature=torch.tensor(temp, **f32), u_acc=rand(N), u_res=rand(B), hist=hist, head=head,
                count=count, sl_max=8.0 + 8.0 * rand(B),
                budget=torch.randint(1, 40, (B,), generator=g, device=dev, dtype=torch.int32))


def prepare(case, seed):
    x = _inputs(case, seed)
    B, V, N, k = case["B"], case["V"], int(x["draft"].shape[0]), case["hi"]
    dev = x["target"].device
    s = dict(x, call=case["call"], k_max=k, V=V, N=N)
    if case["call"] == "shard":
        slices = dsde.slice_bounds(V, case["G"])
        v0, v1 = slices[0]
        full = dsde.verify_sharded(x["target"], x["draft"], x["sl"], x["cu_sl"], x["draft_tokens"], x["temperature"],
                                   x["u_acc"], x["u_res"], k, slices)
        s.update(v0=v0, target=x["target"][:, v0:v1].contiguous(), draft=x["draft"][:, v0:v1].contiguous(),
                 parts=full["parts"].clone(), masses=full["masses"].clone(),
                 err=torch.empty(B, dtype=torch.int32, device=dev), drawn=torch.empty(B, dtype=torch.int32, device=dev),
                 workspace=dsde.new_shard_workspace(B, N, v1 - v0, k, device=dev), out=None)
        s["part_sums"] = s["parts"][0][:, 8:40].view(torch.float64)  # this shard's sums, as the exchange carries them
        s["mass_sums"] = s["masses"][0][:, 0:16].view(torch.float64)
        return s
    s.update(workspace=dsde.new_workspace(B, N, V, k, device=dev), out=None, signal=None, rule=None,
             calibration=dsde.new_calibration_state(B, device=dev),
             row_lse=torch.empty((N, 2), dtype=torch.float64, device=dev))
    return s


def run(s):
    rows = (s["sl"], s["cu_sl"], s["draft_tokens"], s["temperature"], s["u_acc"], s["u_res"], s["k_max"])
    ring = (s["hist"], s["head"], s["count"])
    if s["call"] == "step":
        s["out"] = dsde.step(s["target"], s["draft"], *rows, *ring, s["sl_max"], out=s["out"], workspace=s["workspace"])
        return dict(s["out"], hist=s["hist"], head=s["head"], count=s["count"])
    if s["call"] == "verify":
        s["out"] = dsde.verify(s["target"], s["draft"], *rows, out=s["out"], workspace=s["workspace"],
                               row_lse=s["row_lse"], draft_entropy=True)
        return dict(s["out"], row_lse=s["row_lse"])
    if s["call"] == "calls":
        o = s["out"] = dsde.verify(s["target"], s["draft"], *rows, out=s["out"], workspace=s["workspace"])
        dsde.calibration_update(s["sl"], s["cu_sl"], o["accepted"], o["kld"], o["seq_err"], s["calibration"])
        sig = s["signal"] = dsde.kld_signal(s["sl"], s["cu_sl"], o["kld"], *ring, out=s["signal"])
        s["rule"] = dsde.next_sl(sig["sf"], sig["wvir"], s["sl_max"], SL_MIN, s["k_max"], budget=s["budget"],
                                 out=s["rule"])
        return dict(verify=o, calibration=s["calibration"], signal=sig, rule=s["rule"], hist=s["hist"],
                    head=s["head"], count=s["count"])
    dsde.shard_stats(s["target"], s["draft"], s["v0"], s["V"], *rows[:4], s["k_max"], s["workspace"],
                     part=s["parts"][0], seq_err=s["err"])
    o = s["out"] = dsde.shard_accept_step(s["parts"], s["V"], *rows, s["err"], *ring, s["sl_max"], out=s["out"])
    dsde.shard_draw_mass(s["target"], s["draft"], s["v0"], s["parts"][0], o["jobs"], s["k_max"], s["workspace"],
                         mass=s["masses"][0])
    dsde.shard_draw_pick(0, s["masses"], s["target"], s["draft"], s["v0"], o["jobs"], s["k_max"], o["accepted"],
                         o["tokens"], s["err"], s["workspace"], drawn=s["drawn"])
    return dict({k: v for k, v in o.items() if k != "jobs"}, drawn=s["drawn"], hist=s["hist"], head=s["head"],
                count=s["count"], part_sums=s["part_sums"], mass_sums=s["mass_sums"])


def work(case):
    """Every drafted pair of rows once (bonus rows only count where they are
    sampled, which the logits decide: left out), the small arrays, and per pair
    of logits two exponentials and the sums of p, q and the divergence."""
    N, B, V, k = sum(_lengths(case)), case["B"], case["V"], case["hi"]
    if case["call"] == "shard":
        v0, v1 = dsde.slice_bounds(V, case["G"])[0]
        V = v1 - v0
    e = 2 if case["dtype"] == "bf16" else 4
    small = 16 * N + 4 * B * (k + 12 + 2 * min(case["W"], N_LONG))
    if case["call"] == "shard":
        small += case["G"] * (64 * N + 32 * B) + 44 * B
    return {"bytes": 2 * max(N, 1) * V * e + small, "flops": 14 * max(N, 1) * V}


def tolerance(case):
    return {"rel": 1e-5, "max": 4e-4, "differ": 0.004}


def _windows(x, mu, sl, eps):
    """Signal and pushed rings (float64) from the step's mean divergences."""
    hist, head, count = x["hist"].double().clone(), x["head"].long().clone(), x["count"].long().clone()
    B, W = hist.shape
    dev = hist.device
    live = sl > 0
    at = torch.arange(B, device=dev)
    hist[at[live], head[live]] = mu[live]
    head = torch.where(live, (head + 1) % W, head)
    count = torch.where(live, (count + 1).clamp(max=W), count)
    newest = hist[at, (head - 1) % W]
    mu = torch.where(live, mu, torch.where(count > 0, newest, 0.0))
    i = torch.arange(N_LONG, device=dev)[None, :]
    h = hist.gather(1, (head[:, None] - 1 - i) % W) - newest[:, None]
    got = {}
    for name, n in (("var_short", N_SHORT), ("var_long", N_LONG)):
        a = torch.where(i < count.clamp(max=n)[:, None], DELTA ** i.double(), 0.0)
        tot = a.sum(1).clamp(min=1e-300)
        m = (a * h).sum(1) / tot
        got[name] = (a * (h - m[:, None]) ** 2).sum(1) / tot
    got["mu_last"] = mu
    got["wvir"] = got["var_short"] / torch.where(got["var_long"] > 0, got["var_long"], eps)
    got["sf"] = torch.expm1(2 * mu)
    return got, dict(hist=hist, head=head.int(), count=count.int())


def _rule(sig, sl_max, k_max, budget=None):
    pen = sig["sf"] * sig["wvir"]
    hat = torch.where(pen <= 1, (1 - pen) * (sl_max.double() - SL_MIN) + SL_MIN, SL_MIN)
    cap = hat.mean()
    nxt = torch.floor(torch.minimum(hat, cap) + 0.5).clamp(SL_MIN, k_max)
    if budget is not None:
        nxt = torch.minimum(nxt, (budget.double() - 1).clamp(min=0))
    return dict(sl_hat=hat, sl_cap=cap.reshape(1), sl_next=nxt.int())


def exact(case, seed):
    x = _inputs(case, seed)
    B, V, k = case["B"], case["V"], case["hi"]
    sl, temp = x["sl"].tolist(), _temperatures(case)
    cu = x["cu_sl"].tolist()
    N = cu[-1]
    dev = x["target"].device
    f64 = dict(dtype=torch.float64, device=dev)
    kld, ent, lse = torch.empty(N, **f64), torch.empty(N, **f64), torch.empty((N, 2), **f64)
    accepted = torch.zeros(B, dtype=torch.int32, device=dev)
    tokens = torch.full((B, k + 1), -1, dtype=torch.int32, device=dev)
    mu = torch.zeros(B, **f64)
    for b in range(B):
        s, f, T = sl[b], cu[b], temp[b] or 1.0
        zt = x["target"][f + b:f + b + s + 1].double()
        lt = torch.log_softmax(zt / T, dim=1)
        toks = x["draft_tokens"][f:f + s].long()
        if s:
            zd = x["draft"][f:f + s].double() / T
            ld = torch.log_softmax(zd, dim=1)
            kld[f:f + s] = (lt[:s].exp() * (lt[:s] - ld)).sum(1).clamp(min=0)
            ent[f:f + s] = -(ld.exp() * ld).sum(1)
            lse[f:f + s, 0], lse[f:f + s, 1] = torch.logsumexp(zt[:s] / T, dim=1), torch.logsumexp(zd, dim=1)
            mu[b] = kld[f:f + s].mean()
            best = (zt[:s] == zt[:s].max(dim=1, keepdim=True).values).int().argmax(dim=1)
            j = torch.arange(s, device=dev)
            ok = best == toks if temp[b] == 0 else x["u_acc"][f:f + s].double() < (lt[j, toks] - ld[j, toks]).exp()
            a = int(torch.cumprod(ok.int(), 0).sum())
        else:
            a = 0
        if temp[b] == 0:
            drawn = int((zt[a] == zt[a].max()).int().argmax())
        else:
            w = lt[a].exp() if a == s else (lt[a].exp() - ld[a].exp()).clamp(min=0)
            c = torch.cumsum(w, 0)
            drawn = min(int(torch.searchsorted(c, x["u_res"][b].double() * c[-1], right=True)), V - 1)
        accepted[b] = a
        tokens[b, :a] = toks[:a].int()
        tokens[b, a] = drawn
    zero = torch.zeros(B, dtype=torch.int32, device=dev)
    out = dict(accepted=accepted, tokens=tokens, kld=kld, seq_err=zero)
    if case["call"] == "verify":
        return dict(out, draft_entropy=ent, row_lse=lse)
    sig, ring = _windows(x, mu, x["sl"], EPS)
    if case["call"] == "calls":
        most = torch.zeros(B, **f64)
        for b in range(B):
            if sl[b]:
                most[b] = kld[cu[b]:cu[b + 1]].max()
        cal = dict(a_max=accepted, kld_sum=mu * x["sl"].double(), kld_count=x["sl"].long(), kld_max=most)
        return dict(verify=out, calibration=cal, signal=dict(sig, seq_err=zero),
                    rule=dict(_rule(sig, x["sl_max"], k, x["budget"]), seq_err=zero), **ring)
    out.update(sig, **_rule(sig, x["sl_max"], k), **ring)
    if case["call"] == "shard":  # tokens and drawn hold this shard's own draws alone; the records are not computed here
        out.update(tokens=None, drawn=None, part_sums=None, mass_sums=None)
    return out
