"""Performance cases of the policy-gradient path, each run through the package's entry points.

A case is one call (or one short sequence of calls) of an agentic-RL update: the loss with its
gradients (`pg`), the log-prob pass of the trainer (`logprob`), advantages and value loss of the PPO
path (`ppo`), the linear value head forward and backward (`head`), group advantages (`advantage`) and
the prefix-tree packing of recorded model calls (`tree`).  Shapes are those of the benchmark
workloads and of their micro-batches, with ragged ones beside them.
"""
import math

import numpy as np
import torch

import paper_2608_16798_amd as rlk

DEV = "cuda"
F64 = torch.float64


def _pg(name, **kw):
    base = dict(name=name, kind="pg", dtype="bf16", groups=8, per_group=8, len_min=2048, len_max=2048, d=4096, V=151936,
                masked=0.5, segment=64.0, equal_groups=0, excluded=0, eps_high=0.2, entropy=0.0, kl=0.0, tis=0.0,
                agg="seq", planned=True)
    base.update(kw)
    return base


def listed():
    return [
        # The fp32 debugging batch: launches and latency count, ~1,000 trained tokens.
        _pg("pg_tiny_fp32", dtype="f32", groups=2, per_group=4, len_min=256, len_max=256, d=256, V=4096, segment=32.0),
        # One gradient-accumulation micro-batch of an 8B-sized model: 8 short rollouts against the whole
        # vocabulary, ~770 trained tokens; W and dW move as much as the matrix cores work.
        _pg("pg_micro", groups=2, per_group=4, len_min=240, len_max=240, masked=0.6),
        # A small model's whole update, token-mean objective.
        _pg("pg_small", d=2048, V=32768, masked=0.4, agg="token"),
        # Sizes that fill no tile: hidden size and vocabulary off every power of two, rollouts of all
        # lengths, one failed rollout, importance weights and the KL term on, no bound on the trained tokens.
        _pg("pg_ragged", groups=5, per_group=6, len_min=301, len_max=2999, d=2568, V=50021, excluded=1, kl=0.05, tis=2.0,
            planned=False),
        # Large-batch update with the entropy bonus (logit gradient formed explicitly), rollouts of
        # mixed length.
        _pg("pg_entropy", groups=2, per_group=16, len_min=1024, len_max=8192, entropy=1e-3),
        # The benchmark's update: 128 rollouts x 4096 tokens, 60 % tool tokens, two groups of equal rewards.
        _pg("pg_update", groups=16, len_min=4096, len_max=4096, masked=0.6, equal_groups=2, eps_high=0.28),
        # The trainer's log-probs of one micro-batch, latency of a small call ...
        dict(name="logprob_micro", kind="logprob", dtype="bf16", rollouts=2, len_min=150, len_max=250, d=4096, V=151936,
             masked=0.6, segment=64.0, planned=True),
        # ... and of long-horizon rollouts of a larger model.
        dict(name="logprob_long", kind="logprob", dtype="bf16", rollouts=8, len_min=8192, len_max=32768, d=5120,
             V=151936, masked=0.7, segment=256.0, planned=True),
        # PPO targets of a whole update: advantages and returns, then the value loss and its gradient.
        dict(name="ppo_targets", kind="ppo", rollouts=128, len_min=1024, len_max=7168, masked=0.6, segment=64.0,
             gamma=1.0, lam=0.95),
        # The critic's linear head on the policy's hidden states, forward and backward.
        dict(name="value_head", kind="head", dtype="bf16", rollouts=64, len_min=1024, len_max=3072, d=4096, masked=0.6,
             segment=64.0),
        # Group advantages of the largest batch that a call takes.
        dict(name="advantage_16384", kind="advantage", rollouts=16384, per_group=8),
        # The recorded calls of 32 rollouts packed into prefix trees (host arrays, host code).
        dict(name="tree_pack", kind="tree", rollouts=32, calls=8, prompt=512, response=256, observation=64),
    ]


def _log(rng, lo, hi):
    return lo * (hi / lo) ** rng.random()


def draw(rng):
    kind = rng.choice(["pg", "pg", "pg", "pg", "logprob", "logprob", "ppo", "head", "advantage", "tree"])
    if kind in ("pg", "logprob"):
        fp32 = kind == "pg" and rng.random() < 0.2
        d = 8 * int(_log(rng, 32, 64 if fp32 else 640))
        V = int(_log(rng, 1000, 6000 if fp32 else 152000))
        # trained tokens ~ half of the batch; at most a quarter of the largest listed case's work
        most = 1e9 if fp32 else 3e13
        tokens = int(_log(rng, 300, max(600, min(6e4, most / (d * V)))))
        masked = round(rng.uniform(0.3, 0.7), 2)
        if kind == "logprob":
            R = int(_log(rng, 1, 32))
            mean = max(16, tokens // R)
            return dict(kind="logprob", dtype="bf16", rollouts=R, len_min=mean // 2, len_max=mean + mean // 2, d=d, V=V,
                        masked=masked, segment=float(rng.choice([32, 64, 256])), planned=rng.random() < 0.7)
        Q, G = rng.randint(2, 8), rng.randint(2, 12)
        mean = max(16, tokens // (Q * G))
        c = _pg("", dtype="f32" if fp32 else "bf16", groups=Q, per_group=G, len_min=mean // 2, len_max=mean + mean // 2,
                d=d, V=V, masked=masked, segment=float(rng.choice([32, 64])), equal_groups=rng.choice([0, 0, 1]),
                excluded=rng.choice([0, 0, 1]), eps_high=rng.choice([0.2, 0.28]), entropy=rng.choice([0.0, 0.0, 1e-3]),
                kl=rng.choice([0.0, 0.0, 0.05]), tis=rng.choice([0.0, 0.0, 2.0]), agg=rng.choice(["seq", "token"]),
                planned=rng.random() < 0.7)
        del c["name"]
        return c
    R = int(_log(rng, 4, 512))
    mean = int(_log(rng, 64, min(16384, 1e6 / R)))
    if kind == "ppo":
        return dict(kind="ppo", rollouts=R, len_min=mean // 2, len_max=mean + mean // 2, masked=round(rng.uniform(0.3, 0.7), 2),
                    segment=64.0, gamma=rng.choice([1.0, 0.99]), lam=rng.choice([1.0, 0.95]))
    if kind == "head":
        d = 8 * int(_log(rng, 32, 640))
        mean = max(16, min(mean, int(1e9 / (R * d))))
        return dict(kind="head", dtype=rng.choice(["bf16", "f32"]), rollouts=R, len_min=mean // 2, len_max=mean + mean // 2,
                    d=d, masked=round(rng.uniform(0.3, 0.7), 2), segment=64.0)
    if kind == "advantage":
        return dict(kind="advantage", rollouts=int(_log(rng, 8, 16384)), per_group=rng.randint(2, 16))
    return dict(kind="tree", rollouts=int(_log(rng, 2, 48)), calls=rng.randint(2, 10), prompt=int(_log(rng, 32, 1024)),
                response=int(_log(rng, 16, 512)), observation=int(_log(rng, 8, 256)))


# ---- inputs ----

def _lengths(case, R, rng):
    """Rollout lengths evenly spread over the case's range (the total does not depend on the seed)."""
    return rng.permutation(np.linspace(case["len_min"], case["len_max"], R).round().astype(np.int64))


def _tokens(case):
    """(rollouts, packed tokens, trained tokens expected)."""
    R = case["rollouts"] if "rollouts" in case else case["groups"] * case["per_group"]
    N = int(np.linspace(case["len_min"], case["len_max"], R).round().sum())
    return R, N, int(N * (1 - case["masked"]))


def _mask(case, lengths, rng):
    """1 = token sampled by the policy.  Each rollout opens with a prompt; then policy and tool segments of
    geometric length alternate, with the case's share of tool tokens."""
    tool, policy = case["segment"], case["segment"] * (1 - case["masked"]) / case["masked"]
    out = []
    for T in lengths:
        k = int(2 * T / (tool + policy)) + 8
        while True:
            seg = np.stack([rng.geometric(min(1.0, 1 / tool), k), rng.geometric(min(1.0, 1 / policy), k)], 1).reshape(-1)
            if seg.sum() >= T:
                break
            k *= 2
        out.append(np.repeat(np.tile(np.array([0, 1], np.uint8), k), seg)[:T])
    return np.concatenate(out)


def _batch(case, rng):
    R, _, _ = _tokens(case)
    lengths = _lengths(case, R, rng)
    cu = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    return lengths, cu, _mask(case, lengths, rng)


def _randn(rows, cols, std, dtype, gen):
    out = torch.empty(rows, cols, dtype=dtype, device=DEV)
    for r in range(0, rows, 65536):
        out[r:r + 65536] = torch.randn(min(65536, rows - r), cols, generator=gen, device=DEV) * std
    return out


def _dev(a, dtype):
    return torch.as_tensor(a, dtype=dtype, device=DEV)


def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _head_tensors(case, N, seed):
    """Hidden states of unit scale and an LM head whose logits have a standard deviation of 1.28."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    h = _randn(N, case["d"], 1.0, _dtype(case), gen)
    W = _randn(case["V"], case["d"], 1.28 / math.sqrt(case["d"]), _dtype(case), gen)
    return h, W, gen


def _about_logp(h, W, targets, w_std):
    """Log-probs of the sampled tokens to a few hundredths (h.W_y - ln V - w_std^2 |h|^2 / 2, the log of
    the expected sum over a random vocabulary), computed for a small vocabulary, where that estimate is poorer."""
    out = torch.empty(h.shape[0], device=DEV)
    for r in range(0, h.shape[0], 32768):
        x, y = h[r:r + 32768].float(), targets[r:r + 32768].long()
        z = (x * W[y].float()).sum(1)
        if W.shape[0] <= 40000:
            out[r:r + 32768] = z - torch.logsumexp(x @ W.float().T, 1)
        else:
            out[r:r + 32768] = z - math.log(W.shape[0]) - 0.5 * w_std ** 2 * (x * x).sum(1)
    return out


def _rewards(case, rng):
    """Rewards of {0, 1} by group, every group mixed but the first `equal_groups`, keys in no order, the
    first `excluded` rollouts failed (key -1), groups interleaved in the packed order."""
    Q, G = case["groups"], case["per_group"]
    rew = (rng.random((Q, G)) < 0.3).astype(np.float32)
    rew[:, 0], rew[:, 1] = 1.0, 0.0
    rew[:case["equal_groups"]] = 0.0
    keys = rng.permutation(np.arange(1, 4 * Q + 1, dtype=np.int32))[:Q] * 1009
    order = rng.permutation(Q * G)
    gid = np.repeat(keys, G)[order]
    gid[:case["excluded"]] = -1
    return rew.reshape(-1)[order], gid


def _advantages(rew, gid, eps=1e-6):
    A = np.zeros(len(rew))
    for k in np.unique(gid[gid >= 0]):
        at = gid == k
        r = rew[at].astype(np.float64)
        if r.max() > r.min():
            A[at] = (r - r.mean()) / (r.std() + eps)
    return A


def _pg_inputs(case, seed):
    """Everything a loss call reads.  The policy has moved since the rollouts: log-ratios lean towards each
    token's advantage, most lie well inside the clip range and a tenth well beyond it (none on a bound,
    where the last bit of a log-prob would decide whether a token has a gradient)."""
    rng = np.random.default_rng(seed)
    lengths, cu, mask = _batch(case, rng)
    N = int(cu[-1])
    rew, gid = _rewards(case, rng)
    h, W, gen = _head_tensors(case, N, seed)
    targets = torch.randint(0, case["V"], (N,), generator=gen, device=DEV, dtype=torch.int32)
    sign = torch.repeat_interleave(_dev(np.sign(_advantages(rew, gid)), torch.float32), _dev(lengths, torch.int64))
    u = torch.rand(4, N, generator=gen, device=DEV)
    near, far = 0.1 * (u[0] - 0.5), (0.35 + 0.15 * u[1]) * torch.where(u[2] < 0.5, -1.0, 1.0)
    ratio = 0.06 * sign + torch.where(u[3] < 0.1, far, near)
    old = _about_logp(h, W, targets, 1.28 / math.sqrt(case["d"])) - ratio
    old = old * _dev(mask, torch.float32)
    more = {}
    if case["tis"]:
        more["rollout_logp"] = old + 0.1 * torch.randn(N, generator=gen, device=DEV)
    if case["kl"]:
        more["ref_logp"] = old + 0.2 * torch.randn(N, generator=gen, device=DEV)
    return dict(h=h, W=W, targets=targets, mask=_dev(mask, torch.uint8), cu=_dev(cu, torch.int32), old=old,
                rewards=_dev(rew, torch.float32), gid=_dev(gid, torch.int32), more=more, lengths=lengths,
                host=(cu, mask, rew, gid))


def _calls(case, seed):
    """Recorded calls: each call's context is the history so far; every fourth rollout retries one call."""
    rng = np.random.default_rng(seed)
    rolls = []
    for r in range(case["rollouts"]):
        hist = rng.integers(0, 151936, case["prompt"]).astype(np.int32)
        calls = []
        for c in range(case["calls"]):
            resp = rng.integers(0, 151936, case["response"]).astype(np.int32)
            calls.append((hist, resp))
            if r % 4 == 0 and c == 1:
                calls.append((hist, resp))
            hist = np.concatenate([hist, resp, rng.integers(0, 151936, case["observation"]).astype(np.int32)])
        rolls.append(calls)
    return rolls


def prepare(case, seed):
    kind, f32 = case["kind"], torch.float32
    if kind == "tree":
        return dict(kind=kind, calls=_calls(case, seed))
    if kind == "advantage":
        rng = np.random.default_rng(seed)
        R = case["rollouts"]
        gid = rng.permutation(np.arange(R) // case["per_group"]).astype(np.int32) * 7 + 3
        return dict(kind=kind, rewards=_dev(rng.integers(0, 9, R) / 8, f32), gid=_dev(gid, torch.int32),
                    adv=torch.empty(R, device=DEV), index=torch.empty(R, dtype=torch.int32, device=DEV),
                    count=torch.empty(1, dtype=torch.int32, device=DEV),
                    ws=rlk.alloc_workspace(rlk.advantage_workspace_size(R), DEV))
    if kind == "pg":
        s = _pg_inputs(case, seed)
        cu, mask, rew, gid = s["host"]
        bound = int((mask * np.repeat(gid >= 0, s["lengths"])).sum()) if case["planned"] else 0
        hint = rlk.grad_token_hint(mask, cu, rew, gid) if case["planned"] else 0
        p = rlk.make_params(eps_low=0.2, eps_high=case["eps_high"], entropy_coef=case["entropy"], kl_coef=case["kl"],
                            tis_cap=case["tis"], agg=rlk.AGG_TOKEN if case["agg"] == "token" else rlk.AGG_SEQ,
                            grad_tokens=hint)
        N = s["h"].shape[0]
        ws = rlk.alloc_workspace(rlk.workspace_size(rlk.make_batch(s["h"], s["W"], s["cu"], max_policy_tokens=bound), p), DEV)
        s.update(kind=kind, params=p, bound=bound, ws=ws, loss=torch.empty(1, device=DEV), dhidden=torch.empty_like(s["h"]),
                 dW=torch.empty(s["W"].shape, dtype=f32, device=DEV), logp=torch.empty(N, device=DEV),
                 entropy=torch.empty(N, device=DEV), stats=rlk.stats_buffer(DEV))
        return s
    rng = np.random.default_rng(seed)
    lengths, cu, mask = _batch(case, rng)
    N, R = int(cu[-1]), len(lengths)
    s = dict(kind=kind, cu=_dev(cu, torch.int32), mask=_dev(mask, torch.uint8), lengths=lengths)
    if kind == "logprob":
        h, W, gen = _head_tensors(case, N, seed)
        bound = int(mask.sum()) if case["planned"] else 0
        ws = rlk.alloc_workspace(rlk.workspace_size(rlk.make_batch(h, W, s["cu"], max_policy_tokens=bound)), DEV)
        s.update(h=h, W=W, targets=torch.randint(0, case["V"], (N,), generator=gen, device=DEV, dtype=torch.int32),
                 bound=bound, ws=ws, logp=torch.empty(N, device=DEV), entropy=torch.empty(N, device=DEV))
        return s
    gen = torch.Generator(device=DEV).manual_seed(seed)
    s["gid"] = _dev(rng.permutation(np.arange(R) // 8).astype(np.int32), torch.int32)
    if kind == "ppo":
        s.update(values=0.3 * torch.randn(N, generator=gen, device=DEV) + 0.3, gamma=case["gamma"], lam=case["lam"],
                 rewards=_dev(rng.integers(0, 2, R), f32), adv=torch.empty(N, device=DEV), returns=torch.empty(N, device=DEV),
                 loss=torch.empty(1, device=DEV), dvalues=torch.empty(N, device=DEV),
                 ws=rlk.alloc_workspace(rlk.value_workspace_size(R), DEV))
        return s
    d, dt = case["d"], _dtype(case)
    h = _randn(N, d, 1.0, dt, gen)
    s.update(h=h, w=_randn(1, d, 0.02, dt, gen)[0], dvalues=torch.randn(N, generator=gen, device=DEV) / N,
             values=torch.empty(N, device=DEV), dhidden=torch.empty_like(h), dw=torch.empty(d, device=DEV),
             db=torch.empty(1, device=DEV), ws=rlk.alloc_workspace(rlk.value_head_workspace_size(h, s["cu"]), DEV))
    return s


def run(s):
    kind = s["kind"]
    if kind == "pg":
        rlk.pg_loss_fwd_bwd(s["h"], s["W"], s["targets"], s["mask"], s["cu"], s["old"], s["rewards"], s["gid"], s["params"],
                            loss=s["loss"], dhidden=s["dhidden"], dW=s["dW"], logp_out=s["logp"], entropy_out=s["entropy"],
                            stats=s["stats"], ws=s["ws"], max_policy_tokens=s["bound"], **s["more"])
        # of the statistics, those that do not depend on how the call is cut into chunks
        return dict({k: s[k] for k in ("loss", "dhidden", "dW", "logp", "entropy")},
                    means=s["stats"][:20].view(torch.float32), counts=s["stats"][20:28].view(torch.int32),
                    tokens=s["stats"][32:40].view(torch.int64))
    if kind == "logprob":
        rlk.logprob_fwd(s["h"], s["W"], s["targets"], s["mask"], s["cu"], logp=s["logp"], entropy=s["entropy"], ws=s["ws"],
                        max_policy_tokens=s["bound"])
        return dict(logp=s["logp"], entropy=s["entropy"])
    if kind == "ppo":
        rlk.gae(s["values"], s["rewards"], s["mask"], s["cu"], s["gid"], gamma=s["gamma"], lam=s["lam"], adv=s["adv"],
                returns=s["returns"])
        rlk.value_loss(s["values"], s["returns"], s["mask"], s["cu"], s["gid"], loss=s["loss"], dvalues=s["dvalues"], ws=s["ws"])
        return {k: s[k] for k in ("adv", "returns", "loss", "dvalues")}
    if kind == "head":
        rlk.value_head_fwd(s["h"], s["w"], 0.1, s["mask"], s["cu"], s["gid"], values=s["values"])
        rlk.value_head_bwd(s["h"], s["w"], s["mask"], s["cu"], s["gid"], s["dvalues"], dhidden=s["dhidden"], dw_v=s["dw"],
                           db_v=s["db"], ws=s["ws"])
        return {k: s[k] for k in ("values", "dhidden", "dw", "db")}
    if kind == "advantage":
        rlk.group_advantage(s["rewards"], s["gid"], adv=s["adv"], group_index=s["index"], n_groups=s["count"], ws=s["ws"])
        return dict(adv=s["adv"], index=s["index"], count=s["count"])
    return rlk.tree_pack(s["calls"])


# ---- what a pass cannot do without ----

def work(case):
    kind = case["kind"]
    if kind == "tree":
        # every token of the recorded calls read; packed positions and rows (13 bytes each) written
        history = case["response"] + case["observation"]
        calls = case["rollouts"] * case["calls"]
        context = case["rollouts"] * sum(case["prompt"] + c * history for c in range(case["calls"]))
        packed = case["rollouts"] * (case["prompt"] + case["calls"] * case["response"] + (case["calls"] - 1) * case["observation"])
        return dict(bytes=4 * (context + calls * case["response"]) + 25 * packed, flops=0)
    if kind == "advantage":
        return dict(bytes=16 * case["rollouts"], flops=0)
    R, N, n = _tokens(case)
    if kind == "ppo":
        # values and mask read, advantages and returns written; values, returns and mask read, gradient written
        return dict(bytes=26 * N, flops=0)
    e = 4 if case["dtype"] == "f32" else 2
    d = case["d"]
    if kind == "head":
        # trained rows read once by each direction, every gradient row written
        return dict(bytes=2 * n * d * e + N * d * e + 10 * N, flops=4 * n * d)
    V = case["V"]
    if kind == "logprob":
        return dict(bytes=(n * d + V * d) * e + 13 * N, flops=2 * n * d * V)
    grad = n if case["entropy"] or case["kl"] else n * (1 - case["equal_groups"] / case["groups"])
    return dict(bytes=(n * d + V * d + N * d) * e + V * d * 4 + 25 * N, flops=2 * V * d * (n + 2 * grad))


def tolerance(case):
    kind = case["kind"]
    if kind == "tree":
        return "exact"
    if kind == "pg":
        # bf16: the gradients are rounded to bf16 from operands rounded to bf16; fp32: sums of up to 4,096 terms
        return dict(rel=1e-2) if case["dtype"] == "bf16" else dict(rel=1e-5)
    if kind == "head" and case["dtype"] == "bf16":
        return dict(rel=1e-2)
    return dict(rel=1e-5)


# ---- the same in 64 bits ----

def _exact_pg(case, seed):
    s = _pg_inputs(case, seed)
    _, mask, rew, gid = s["host"]
    N, (V, d) = s["h"].shape[0], s["W"].shape
    A_r = _advantages(rew, gid)
    roll = np.repeat(np.arange(len(rew)), s["lengths"])
    kept = (mask != 0) & (gid >= 0)[roll]
    idx = torch.as_tensor(np.flatnonzero(kept), device=DEV)
    n_r = np.bincount(roll[kept], minlength=len(rew))
    keys = np.unique(gid[gid >= 0])
    size = np.array([(gid == g).sum() for g in gid])
    if case["agg"] == "token":
        w_tok = np.full(kept.sum(), 1.0 / kept.sum())
    else:
        w_tok = (1.0 / (len(keys) * size * np.maximum(n_r, 1)))[roll[kept]]
    w_tok = _dev(w_tok, F64)
    A = _dev(A_r[roll[kept]], F64)
    W = s["W"].to(F64)
    dW = torch.zeros(V, d, dtype=F64, device=DEV)
    dh = torch.zeros(N, d, dtype=F64, device=DEV)
    logp, ent = torch.zeros(N, dtype=F64, device=DEV), torch.zeros(N, dtype=F64, device=DEV)
    loss = torch.zeros((), dtype=F64, device=DEV)
    lo, hi, c, beta = 1 - np.float64(np.float32(0.2)), 1 + np.float64(np.float32(case["eps_high"])), case["entropy"], case["kl"]
    c, beta = float(np.float32(c)), float(np.float32(beta))
    for r in range(0, len(idx), 2048):
        at = idx[r:r + 2048]
        x = s["h"][at].to(F64)
        z = x @ W.T
        lse = torch.logsumexp(z, 1)
        y = s["targets"][at].long()
        k = torch.arange(len(at), device=DEV)
        lp = z[k, y] - lse
        z -= lse[:, None]
        p = z.exp()
        H = -(p * z).sum(1)
        a, w = A[r:r + 2048], w_tok[r:r + 2048]
        old = s["old"][at].to(F64)
        rho = (lp - old).exp()
        sur = torch.minimum(rho * a, rho.clamp(lo, hi) * a)
        cut = ((a > 0) & (rho > hi)) | ((a < 0) & (rho < lo))
        if case["tis"]:
            w = w * (old - s["more"]["rollout_logp"][at].to(F64)).exp().clamp(max=case["tis"])
        g = torch.where(cut, 0.0, a * rho)
        obj = sur + c * H
        if beta:
            q = s["more"]["ref_logp"][at].to(F64) - lp
            obj = obj - beta * (q.exp() - q - 1)
            g = g + beta * (q.exp() - 1)
        loss -= (w * obj).sum()
        g, e = -w * g, -w * c
        if c:
            p *= g[:, None] + e[:, None] * (z + H[:, None])
        else:
            p *= g[:, None]
        p.neg_()
        p[k, y] += g
        dh[at] = p @ W
        dW += p.T @ x
        logp[at], ent[at] = lp, H
    return dict(loss=loss.reshape(1), dhidden=dh, dW=dW, logp=logp, entropy=ent, means=None, counts=None, tokens=None)


def _exact_logprob(case, seed):
    s = prepare(case, seed)
    N = s["h"].shape[0]
    W = s["W"].to(F64)
    logp, ent = torch.zeros(N, dtype=F64, device=DEV), torch.zeros(N, dtype=F64, device=DEV)
    idx = torch.nonzero(s["mask"])[:, 0]
    for r in range(0, len(idx), 2048):
        at = idx[r:r + 2048]
        z = torch.log_softmax(s["h"][at].to(F64) @ W.T, 1)
        logp[at] = z[torch.arange(len(at), device=DEV), s["targets"][at].long()]
        ent[at] = -(z.exp() * z).sum(1)
    return dict(logp=logp, entropy=ent)


def _exact_ppo(case, seed):
    s = prepare(case, seed)
    v, mask, rew = s["values"].double().cpu().numpy(), s["mask"].cpu().numpy() != 0, s["rewards"].double().cpu().numpy()
    cu = s["cu"].cpu().numpy().astype(np.int64)
    gamma, lam = float(np.float32(case["gamma"])), float(np.float32(case["lam"]))
    R = len(rew)
    adv, ret = np.zeros(len(v)), np.zeros(len(v))
    # all rollouts at once, from their last tokens backwards
    nv, later, A = rew.copy(), np.zeros(R, bool), np.zeros(R)
    for k in range(int(np.diff(cu).max())):
        t = cu[1:] - 1 - k
        on = t >= cu[:-1]
        on[on] = mask[t[on]]
        if not on.any():
            continue
        at = t[on]
        delta = np.where(later[on], gamma * nv[on], rew[on]) - v[at]
        A[on] = delta + gamma * lam * np.where(later[on], A[on], 0.0)
        adv[at], ret[at] = A[on], A[on] + v[at]
        nv[on], later[on] = v[at], True
    diff = np.where(mask, v - ret, 0.0)
    n = mask.sum()
    return dict(adv=adv, returns=ret, loss=np.array([(diff ** 2).sum() / n]), dvalues=2 * diff / n)


def _exact_head(case, seed):
    s = prepare(case, seed)
    N, d = s["h"].shape
    on = s["mask"].to(F64)
    g, w = s["dvalues"].to(F64) * on, s["w"].to(F64)
    values, dw = torch.empty(N, dtype=F64, device=DEV), torch.zeros(d, dtype=F64, device=DEV)
    dh = torch.empty(N, d, dtype=F64, device=DEV)
    for r in range(0, N, 16384):
        x = s["h"][r:r + 16384].to(F64)
        values[r:r + 16384] = (x @ w + float(np.float32(0.1))) * on[r:r + 16384]
        dw += g[r:r + 16384] @ x
        dh[r:r + 16384] = g[r:r + 16384, None] * w
    return dict(values=values, dhidden=dh, dw=dw, db=g.sum().reshape(1))


def exact(case, seed):
    kind = case["kind"]
    if kind == "pg":
        return _exact_pg(case, seed) if work(case)["flops"] < 3e14 else None
    if kind == "logprob":
        return _exact_logprob(case, seed)
    if kind == "ppo":
        return _exact_ppo(case, seed)
    if kind == "head":
        return _exact_head(case, seed)
    if kind == "advantage":
        s = prepare(case, seed)
        gid = s["gid"].cpu().numpy()
        rew = s["rewards"].cpu().numpy().astype(np.float64)
        _, index = np.unique(gid, return_inverse=True)
        n = np.bincount(index)
        mu = np.bincount(index, rew) / n
        sd = np.sqrt(np.bincount(index, (rew - mu[index]) ** 2) / n)
        equal = sd[index] == 0
        return dict(adv=np.where(equal, 0.0, (rew - mu[index]) / (sd[index] + float(np.float32(1e-6)))), index=None, count=None)
    return None
