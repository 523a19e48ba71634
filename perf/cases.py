"""Benchmark cases of the decision step: what a serving program has it do.

Each case is one call of ``paper_2608_26004_amd.fuse_verify`` over a batch of
B requests with K drafts, through the Python entry point with a Workspace that
the program keeps.  The inputs follow the seeded generator of ``synth.py``
(shared prior per position, verifier and drafter noise around it, a
per-request divergence scale rho between the drafter's two views), drawn on
the GPU so that they are quick to make.
"""

import math

import torch

import paper_2608_26004_amd as asp

LN2 = math.log(2.0)

# rho and tau: "a" or "lo:hi" (uniform per request) or "even/odd" (alternating)
_BASE = dict(B=8, K=4, V=128256, dtype="bf16", prior="gauss", rho="1", tau="1", gate="cda",
             beta=1.0, want_gate=False, want_full=False, early_exit=0, fuse_bonus=False,
             Vd=0, shared=0)


def _case(**kw):
    c = dict(_BASE)
    c.update(kw)
    return c


def listed():
    return [
        # one interactive request, small vocabulary, fp32 logits: pure latency
        _case(name="single_fp32", B=1, K=4, V=32000, dtype="fp32", rho="0.5"),
        # the paper's operating point: two drafts, greedy, a few agents
        _case(name="greedy_b8", B=8, K=2, V=151936, tau="0"),
        # a small sampling batch
        _case(name="sample_b8", B=8, K=5, V=128256, tau="0.8"),
        # a medium batch with a peaked prior and mixed divergence
        _case(name="zipf_b32", B=32, K=8, V=151936, prior="zipf", rho="0:2", tau="0.7"),
        # fp32 logits and an odd vocabulary size (rows start mid-vector), half
        # of the requests greedy, the bonus row fused, the KL gate
        _case(name="ragged_fp32_kl", B=24, K=5, V=50257, dtype="fp32", rho="0:2", tau="0/1",
              gate="kl", fuse_bonus=True),
        # the throughput batch: half of the requests with identical views
        _case(name="batch_b128", B=128, K=6, V=151936, rho="0/3"),
        # the same batch with the per-draft divergence and threshold returned
        # (acceptance diagnostics)
        _case(name="batch_b128_gate", B=128, K=6, V=151936, rho="0/3", want_gate=True),
        # the same batch, the later rows read only where the first two decide
        # nothing
        _case(name="batch_b128_early", B=128, K=6, V=151936, rho="0/3", early_exit=2),
        # every element's fused log-probability (scoring, distillation targets)
        _case(name="full_b128", B=128, K=6, V=151936, rho="0/3", want_full=True),
        # a drafter of another model family, reached through a vocabulary map:
        # a few greedy agents, and the throughput batch
        _case(name="cross_greedy_b8", B=8, K=2, V=151936, tau="0", Vd=128256, shared=109566),
        _case(name="cross_b128", B=128, K=6, V=151936, rho="0/3", Vd=128256, shared=109566),
        # the largest: 512 requests, 256000-token vocabulary, greedy and sampling
        _case(name="large_b512", B=512, K=8, V=256000, rho="0:2", tau="0/1"),
    ]


_VOCABS = (32000, 50257, 128256, 151936, 256000)
_LARGEST = 512 * 25 * 256000 * 2      # logit bytes of the largest listed case
_CROSS_LARGEST = 128 * 21 * 151936 * 2


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    c = _case(B=_logint(rng, 1, 512), K=rng.randint(1, 8),
              dtype=rng.choice(["bf16", "bf16", "bf16", "fp32"]),
              prior=rng.choice(["gauss", "gauss", "zipf"]),
              rho=rng.choice(["1", "0:2", "0/3", "0.5"]),
              tau=rng.choice(["0", "1", "0.8", "0/1", "0.7"]),
              gate=rng.choice(["cda", "cda", "cda", "fixed", "kl", "lambda"]),
              beta=rng.choice([1.0, 1.0, 1.0, 0.5]),
              fuse_bonus=rng.random() < 0.2)
    # real vocabulary sizes, or any size of their range, odd ones among them
    c["V"] = rng.choice(_VOCABS) if rng.random() < 0.5 else _logint(rng, 32000, 256000)
    what = rng.choice(["plain", "plain", "plain", "gate", "early", "full", "cross"])
    most = _LARGEST
    if what == "gate":
        c["want_gate"] = True
    elif what == "early":
        c["early_exit"] = rng.randint(1, 3)
    elif what == "full":
        c["want_full"] = True
        most //= 4
    elif what == "cross":
        c["Vd"] = _logint(rng, 32000, 256000)
        c["shared"] = int(rng.uniform(0.6, 0.95) * min(c["V"], c["Vd"]))
        most = _CROSS_LARGEST
    per = (3 * c["K"] + 3) * max(c["V"], c["Vd"]) * (2 if c["dtype"] == "bf16" else 4)
    c["B"] = max(1, min(c["B"], most // per))
    return c


# ------------------------------------------------------------------ inputs --
def _per_request(spec, B, gen):
    if "/" in spec:
        even, odd = (float(s) for s in spec.split("/"))
        r = torch.arange(B, device="cuda") % 2
        return torch.where(r == 0, even, odd).double()
    if ":" in spec:
        lo, hi = (float(s) for s in spec.split(":"))
        return lo + (hi - lo) * torch.rand(B, device="cuda", dtype=torch.float64, generator=gen)
    return torch.full((B,), float(spec), device="cuda", dtype=torch.float64)


def prepare(case, seed):
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    B, K, V, Vd = case["B"], case["K"], case["V"], case["Vd"] or case["V"]
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    rho = _per_request(case["rho"], B, gen).float()
    tau = _per_request(case["tau"], B, gen).float()

    def randn(*shape):
        return torch.randn(*shape, device=dev, generator=gen)

    vmap = xs = js = None
    if case["Vd"]:
        # the shared tokens, each with a drafter id of its own
        xs = torch.randperm(V, device=dev, generator=gen)[:case["shared"]].sort().values
        js = torch.randperm(Vd, device=dev, generator=gen)[:case["shared"]]
        vmap = torch.full((V,), -1, dtype=torch.int32, device=dev)
        vmap[xs] = js.int()
    t = torch.empty(B, K + 1, V, dtype=dt, device=dev)
    a = torch.empty(B, K + 1, Vd, dtype=dt, device=dev)
    b = torch.empty(B, K + 1, Vd, dtype=dt, device=dev)
    d = torch.zeros(B, K, dtype=torch.int32, device=dev)
    q = torch.ones(B, K, dtype=torch.float32, device=dev)
    n = max(1, min(B, (1 << 26) // ((K + 1) * V)))
    for lo in range(0, B, n):
        hi = min(B, lo + n)
        shape = (hi - lo, K + 1, V)
        if case["prior"] == "zipf":
            rank = torch.rand(shape, device=dev, generator=gen).argsort(dim=-1).float() + 1.0
            z = -6.0 * rank.log().sqrt() + randn(*shape)
        else:
            z = 3.0 * randn(*shape)
        t[lo:hi] = (z + randn(*shape)).to(dt)
        full = z + randn(*shape)
        comp = (full + rho[lo:hi, None, None] * randn(*shape)).to(dt)
        full = full.to(dt)
        if vmap is None:
            a[lo:hi], b[lo:hi] = full, comp
            w = full[:, :K].float()
        else:
            a[lo:hi] = (3.0 * randn(hi - lo, K + 1, Vd)).to(dt)
            b[lo:hi] = (3.0 * randn(hi - lo, K + 1, Vd)).to(dt)
            a[lo:hi, :, js] = full[:, :, xs]
            b[lo:hi, :, js] = comp[:, :, xs]
            w = torch.full_like(full[:, :K], -math.inf).float()     # shared tokens are drafted
            w[:, :, xs] = full[:, :K, xs].float()
        # the drafter's own choice from its full view: the argmax, or a draw
        # from softmax(a / tau) (Gumbel) and its probability
        tl = tau[lo:hi, None, None]
        samp = tl > 0
        w = torch.where(samp, w / torch.where(samp, tl, 1.0), w)
        noise = -torch.rand(w.shape, device=dev, generator=gen).clamp_min_(1e-20).log_().neg_().log_()
        pick = torch.where(samp, w + noise, w).argmax(dim=-1)
        p = (w.gather(-1, pick[..., None]).squeeze(-1).double() - w.double().logsumexp(-1)).exp()
        d[lo:hi] = pick.int()
        q[lo:hi] = torch.where(samp[..., 0], p.float(), 1.0)
        del z, full, comp, w, noise
    u = torch.rand(B, K + 1, device=dev, generator=gen)
    gates = {"cda": asp.GATE_CDA, "fixed": asp.GATE_FIXED, "kl": asp.GATE_KL, "lambda": asp.GATE_LAMBDA}
    kw = dict(beta=case["beta"], gate_mode=gates[case["gate"]], return_gate=case["want_gate"],
              return_full=case["want_full"], early_exit=case["early_exit"],
              fuse_bonus=case["fuse_bonus"], vocab_map=vmap, workspace=asp.Workspace(dev))
    return dict(args=(t, a, b, d, q, u, tau), kw=kw)


def run(state):
    out = asp.fuse_verify(*state["args"], **state["kw"])
    # the drafts' log-probabilities, which no draw decides, also on their own
    return {"out": out, "drafts": out[2][:, :-1]}


def work(case):
    """Each logit the outputs depend on read once (t rows 0..K, a and b rows
    0..K-1, or 0..K with the fused bonus; through a map only the shared
    drafter entries; with early exit the first rows alone), outputs written
    once.  Operations: an exponential's argument, the exponential and its sum
    per stream, and the fused logit."""
    B, K, V = case["B"], case["K"], case["V"]
    el = 2 if case["dtype"] == "bf16" else 4
    rows_ab = K + 1 if case["fuse_bonus"] else K
    rows_t = K + 1
    if case["early_exit"] and case["early_exit"] <= K:
        rows_ab = rows_t = case["early_exit"]
    n_ab = case["shared"] or V
    out = 4 * B * (2 + (K + 1)) + (8 * B * K if case["want_gate"] else 0)
    out += 4 * B * (K + 1) * V if case["want_full"] else 0
    small = 4 * B * (3 * K + 2) + (4 * V if case["Vd"] else 0)
    return {"bytes": B * el * (rows_t * V + 2 * rows_ab * n_ab) + out + small,
            "flops": B * (3 * rows_t * V + 8 * rows_ab * n_ab)}


def tolerance(case):
    """fp32 sums behind log-probabilities of size 1 to 30: up to 5e-7 off fp64
    as measured.  An inverse-CDF draw over 10^5 tokens lands within fp32
    rounding of a step boundary in about 0.5% of the requests and may then
    take the neighbouring token, whose log-probability is another one."""
    if case["tau"] != "0" and case["B"] >= 100:
        return {"rel": 0.015, "max": 0.99, "differ": 0.01}
    return {"rel": 2e-6, "max": 2e-5, "differ": 0.004}


# ------------------------------------------------------------- 64-bit check --
def exact(case, seed):
    """The outputs that no draw decides (the drafts' log-probabilities, the
    gate, the full rows) in fp64 torch; f = t + beta (a - b) in fp32 as the
    step defines it."""
    s = prepare(case, seed)
    t, a, b, d, q, u, tau = s["args"]
    vmap = s["kw"]["vocab_map"]
    B, K, V = case["B"], case["K"], case["V"]
    gamma, lam, beta = 0.5, 0.1, case["beta"]
    neg = -math.inf
    flp = torch.zeros(B, K, dtype=torch.float64, device=t.device)
    gate = torch.zeros(B, K, 2, dtype=torch.float64, device=t.device)
    full = (torch.empty(B, K + 1, V, dtype=torch.float64, device=t.device) if case["want_full"] else None)
    d, u64, taus = d.long(), u.double(), tau.tolist()
    rows = torch.arange(K, device=t.device)
    for r in range(B):
        T, A, Bv = t[r].float(), a[r].float(), b[r].float()
        if vmap is not None:
            ok = vmap >= 0
            j = vmap.long().clamp_min(0)
            T = torch.where(ok, T, neg)
            A = torch.where(ok, A[:, j], neg)
            Bv = torch.where(ok, Bv[:, j], neg)
        F = T + beta * (A - Bv)
        F = torch.where(F.isnan(), neg, F)
        if not case["fuse_bonus"]:
            F[K] = T[K]
        samp = taus[r] > 0
        # (the fp32 temperature of the call)
        th = taus[r] if samp else 1.0
        LF = (F.double() / th).log_softmax(-1)
        if full is not None:
            full[r] = LF
        Ad, Bd = A[:K].double(), Bv[:K].double()
        LA, LB = Ad.log_softmax(-1), Bd.log_softmax(-1)
        P, Q = LA.exp(), LB.exp()
        at = lambda x: x[rows, d[r]]     # noqa: E731
        if case["gate"] == "kl":
            D = torch.where(P > 0, P * (LA - LB), 0.0).sum(-1)
        elif case["gate"] == "lambda":
            D = lam * (at(LA) - at(LB))
        else:
            LM = (0.5 * (P + Q)).log()
            D = 0.5 * (torch.where(P > 0, P * (LA - LM), 0.0) + torch.where(Q > 0, Q * (LB - LM), 0.0)).sum(-1)
            D = D.clamp(0.0, LN2)
        fixed = case["gate"] == "fixed"
        De = torch.zeros_like(D) if fixed else D
        gate[r, :, 0] = D
        gate[r, :, 1] = gamma * (-De).exp()
        flp[r] = at(LF[:K])
        if samp:
            x = at(LF[:K]) - q[r].double().log() - math.log(gamma)
            lhs = u64[r, :K].log()
        else:
            x = at(T[:K].double().log_softmax(-1)) - at(LB) - math.log(gamma)
            lhs = torch.zeros_like(x)
        G = case["early_exit"]
        if 0 < G <= K:
            # the later rows are not read after a sure rejection (whatever D
            # within its bounds) among the first
            known = case["gate"] in ("fixed", "kl", "lambda")
            same = (A[:K] == Bv[:K]).all(-1)
            most = De if known else torch.where(same, 0.0, LN2)
            if bool((lhs >= x + most)[:G].any()):
                flp[r, G:K] = math.nan
                gate[r, G:] = math.nan
    out = (None, None, None)
    out += (gate,) if case["want_gate"] else ()
    out += (full,) if case["want_full"] else ()
    return {"out": out, "drafts": flp}
