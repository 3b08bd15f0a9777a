"""Timed cases of the library's public calls: the learner's loss forward and
backward, the calls that build its teacher-score cache, and the diagnostics.

A case is one call on one batch.  Sizes follow the learner this library is
for: a vocabulary of 151,936 entries, rollouts of up to 2,048 tokens, 1 to 64
Monte-Carlo draws or a top-32 support per token, bf16 logits with fp32
gradients; and, beside them, fp32 logits, bf16 gradients, narrower and odd
vocabularies, and batches from the few rows left at the end of a step to
8,192 tokens.

  op     "loss" (loss_fwd_bwd), "sample", "topk", "score", "diag"
  N, V   tokens and vocabulary; rows are padded to a multiple of 8 elements
  K      cached ids per token: support size, draws or ids to score
  dtype  of the logits; grad: dtype of the gradient
  ragged rollouts of unequal length, padded and masked
  more   the optional outputs are wanted too (lse, gathered logits, coverage)
  kept   the call is prepared once and re-issued on the same buffers
"""
import math

import torch

import paper_2606_24143_amd as opd

DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
BYTES = {"bf16": 2, "f32": 4}
SUPPORT = ("fkl_topk", "rkl_topk", "fkl_topk_trunc", "rkl_topk_trunc")
DENSE = ("fkl_dense", "rkl_dense")
# (the clipped surrogates run the same kernels; where a ratio falls within
# rounding of the clip's edge their gradient jumps by a whole spike, so no
# tolerance describes two correct results)
MC = ("rkl_mc", "rkl_mc_old", "rkl_mc_nois")
GROUPS = (2, 4, 8)
SEQ = 2048
CLIP = 0.2
# most elements of a [N, V] array, and most bytes moved, by a drawn case
MOST_ELEMENTS = 8192 * 151936
MOST_BYTES = 7.0e9


def _loss(est, N, V, K, dtype="bf16", grad="f32", ragged=False, more=False, kept=False, **name):
    return dict(op="loss", est=est, N=N, V=V, K=K, dtype=dtype, grad=grad, ragged=ragged, more=more,
                kept=kept, **name)


def listed():
    return [
        # the rows left over at the end of a step: latency and launches count
        _loss("rkl_mc", 24, 151936, 16, kept=True, name="mc16-24-rows"),
        # the smallest micro-batch
        _loss("rkl_mc", 256, 151936, 16, name="mc16-256-rows"),
        # an ordinary learner micro-batch: four full rollouts, with the outputs
        # that the diagnostics read
        _loss("rkl_mc", 8192, 151936, 16, more=True, name="mc16-8192-rows"),
        # one draw per token over ragged rollouts, gradients in bf16 for a bf16
        # LM head, a vocabulary that does not fill its padded rows
        _loss("rkl_mc1", 4096, 151933, 1, grad="bf16", ragged=True, name="mc1-ragged-bf16"),
        # logits that the model hands over in fp32
        _loss("rkl_mc", 1024, 151936, 64, dtype="f32", name="mc64-fp32"),
        # the sparse support: only the cached logits are read
        _loss("fkl_topk", 4096, 151936, 32, name="topk32"),
        # a small model's vocabulary, with the support's coverage logged
        _loss("rkl_topk", 512, 32000, 16, dtype="f32", more=True, name="topk16-small-fp32"),
        # full teacher logits
        _loss("rkl_dense", 2048, 151936, 0, name="dense"),
        # building the cache: the rollout's draws, the teacher's support, its
        # scores at the draws
        dict(op="sample", N=4096, V=151936, K=16, dtype="bf16", ragged=False, name="draws16"),
        dict(op="topk", N=4096, V=151936, K=32, dtype="bf16", ragged=False, name="support32"),
        dict(op="score", N=2048, V=100003, K=16, dtype="bf16", ragged=True, name="score16-odd"),
        # the estimator's diagnostics over a whole batch
        dict(op="diag", N=32768, V=0, K=16, dtype="f32", ragged=True, name="diagnostics"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        op = rng.choice(("loss", "loss", "loss", "loss", "loss", "sample", "topk", "score", "diag"))
        if op == "diag":
            return dict(op=op, N=_log_int(rng, 256, 65536), V=0, K=rng.choice((16, 32, 64)),
                        dtype="f32", ragged=rng.random() < 0.5)
        N = _log_int(rng, 8, 8192)
        # half of the draws at a vocabulary of full width, some a little short of it
        V = (151936 - rng.choice((0, 0, 1, 7, 267)) if rng.random() < 0.5
             else _log_int(rng, 2000, 160000))
        dtype = rng.choice(("bf16", "bf16", "f32"))
        ragged = rng.random() < 0.3
        if op != "loss":
            c = dict(op=op, N=N, V=V, K=_log_int(rng, 1, 64), dtype=dtype, ragged=ragged)
        else:
            est = rng.choice(SUPPORT + DENSE + MC + ("rkl_mc1", "rkl_mc", "fkl_topk"))
            K = (0 if est in DENSE else 1 if est == "rkl_mc1"
                 else _log_int(rng, 4 if est in SUPPORT else 1, 128))
            c = _loss(est, N, V, K, dtype, rng.choice(("f32", "f32", "bf16")), ragged,
                      rng.random() < 0.4, rng.random() < 0.3)
        if N * V <= MOST_ELEMENTS and work(c)["bytes"] <= MOST_BYTES:
            return c


# ---------------------------------------------------------------- inputs

def _rows(N, V):
    """Row blocks of about 2^26 elements: what the inputs are made in."""
    step = max(1, (1 << 26) // max(V, 1))
    return [(r, min(r + step, N)) for r in range(0, N, step)]


def _mask(N, gen):
    """Right-padded rollouts of 2,048 tokens (of N, in a smaller batch), an
    eighth of the length to the whole of it valid."""
    L = min(SEQ, N)
    n = -(-N // L)
    lens = torch.randint(max(1, L // 8), L + 1, (n,), generator=gen, device="cuda")
    return (torch.arange(L, device="cuda")[None, :] < lens[:, None]).reshape(-1)[:N].to(torch.uint8)


def prepare(case, seed):
    c = case
    op, N, V, K = c["op"], c["N"], c["V"], c["K"]
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def randn(*shape):
        return torch.randn(*shape, device="cuda", generator=gen)

    s = {"case": c, "mask": _mask(N, gen) if c["ragged"] else None}
    if op == "diag":
        # what a Monte-Carlo loss call returned and the cache it read: the
        # student a little off the behaviour policy, the teacher further
        logp = -2.0 - 2.5 * randn(N, K).abs()
        s["lse"] = 16.0 + 0.5 * randn(N)
        s["gathered"] = logp + s["lse"][:, None]
        s["teacher_logp"] = logp + randn(N, K)
        s["behav_logp"] = logp + 0.4 * randn(N, K)
        return s
    dt, ld = DTYPES[c["dtype"]], -(-V // 8) * 8
    # bulk logits of spread 3; supports come from peaked rows, one entry in a
    # hundred 8 higher
    est = c.get("est", "")
    peaked = op == "topk" or est in SUPPORT
    logits = torch.zeros(N, ld, device="cuda", dtype=dt)[:, :V]
    teacher = torch.zeros(N, ld, device="cuda", dtype=dt)[:, :V] if est in DENSE else None
    ids = torch.empty(N, K, device="cuda", dtype=torch.int32)
    tau, beta = torch.empty(N, K, device="cuda"), torch.empty(N, K, device="cuda")
    for a, b in _rows(N, V):
        z = 3.0 * randn(b - a, V)
        if peaked:
            z += 8.0 * (torch.rand(b - a, V, device="cuda", generator=gen) < 0.01)
        logits[a:b] = z
        if op in ("sample", "topk"):
            continue
        z = logits[a:b].float()
        y = z + randn(b - a, V)  # the teacher
        if est in DENSE:
            teacher[a:b] = y
        elif est in SUPPORT:
            ids[a:b] = y.topk(K).indices
            tau[a:b] = torch.log_softmax(y, 1).gather(1, ids[a:b].long())
        else:
            old = torch.log_softmax(z + 0.5 * randn(b - a, V), 1)  # the stale policy
            ids[a:b] = torch.multinomial(old.exp(), K, replacement=True, generator=gen)
            beta[a:b] = old.gather(1, ids[a:b].long())
            tau[a:b] = torch.log_softmax(y, 1).gather(1, ids[a:b].long())
    s["logits"] = logits
    if op == "sample":
        # uniforms on the grid that a 24-bit generator gives
        s["uniforms"] = torch.randint(0, 1 << 24, (N, K), device="cuda", generator=gen) * 2.0 ** -24
    elif op == "score":
        s["ids"] = ids
    elif op == "loss":
        if est in DENSE:
            s["cache"] = {"teacher_logits": teacher}
        elif est in SUPPORT:
            s["cache"] = {"idx": ids, "teacher_logp": tau}
        else:
            s["cache"] = {"sampled_ids": ids, "teacher_logp": tau, "behav_logp": beta}
        s["options"] = dict(mask=s["mask"], grad_scale=1.0 / N, dlogits_dtype=DTYPES[c["grad"]],
                            want_lse=c["more"],
                            want_gathered=c["more"] and est not in DENSE,
                            want_coverage=c["more"] and est in SUPPORT)
        if c["kept"]:
            s["call"] = opd.prepare_loss_fwd_bwd(logits, est, **s["cache"], **s["options"])
    return s


def run(state):
    c = state["case"]
    op, mask = c["op"], state["mask"]
    if op == "loss":
        if c["kept"]:
            return state["call"]()
        return opd.loss_fwd_bwd(state["logits"], c["est"], **state["cache"], **state["options"])
    if op == "sample":
        return opd.sample_actions(state["logits"], state["uniforms"], mask=mask, want_lse=True)
    if op == "topk":
        return opd.topk_support(state["logits"], c["K"], mask=mask, want_lse=True)
    if op == "score":
        return opd.score_actions(state["logits"], state["ids"], mask=mask, want_lse=True)
    return opd.mc_diagnostics(state["lse"], state["gathered"], state["teacher_logp"],
                              state["behav_logp"], mask=mask, clip_eps=CLIP, group_sizes=GROUPS,
                              seq_len=SEQ)


# ---------------------------------------------------------------- work and tolerance

def work(case):
    c = case
    op, N, V, K = c["op"], c["N"], c["V"], c["K"]
    n = N * 9 / 16 if c["ragged"] else N  # valid rows: 1/8 to the whole of a rollout
    inb = BYTES[c["dtype"]]
    if op == "diag":
        return {"bytes": n * (4 + 12 * K) + N * 12, "flops": n * K * 20}
    if op != "loss":
        return {"bytes": n * V * inb + N * 8 * K + (N * 4 * K if op == "sample" else 0) + 4 * N,
                "flops": n * V * 4}
    est = c["est"]
    if est in DENSE:
        read, flops = 2 * V * inb, 16 * V
    elif est in ("fkl_topk", "rkl_topk") and not c["more"]:
        read, flops = K * inb + 8 * K, 20 * K
    else:
        read, flops = V * inb + (8 if est in SUPPORT else 12) * K, 8 * V
    return {"bytes": n * read + N * (V * BYTES[c["grad"]] + 4), "flops": n * flops}


def tolerance(case):
    """About four times what the calls are off the 64-bit results by."""
    c = case
    if c["op"] == "loss" and c["grad"] == "bf16":
        return {"rel": 7e-3, "max": 2e-2}  # one rounding to bf16
    if c["op"] == "loss":
        return {"rel": 8e-6, "max": 1e-4}
    if c["op"] == "diag":
        # a ratio within rounding of the clip's edge may count on either side
        return {"rel": 2e-5, "max": 1e-4}
    # draws of a double-precision distribution function: two of them part only
    # where a uniform falls within rounding of a cumulative value
    return {"rel": 1e-6, "max": 1e-5, "differ": 1e-5 if c["op"] == "sample" else 0.0}


# ---------------------------------------------------------------- in 64 bits

def _mc_weights(est, lp, tau, beta):
    """Per-draw gradient weight and loss term of the surrogates."""
    if est == "rkl_mc_nois":
        return tau - lp, (tau - lp) * lp
    w = (lp - beta).exp() * (tau - beta if est == "rkl_mc_old" else tau - lp)
    return w, w


def _exact_loss(c, s):
    est, N, V, K = c["est"], c["N"], c["V"], c["K"]
    gamma = s["options"]["grad_scale"]
    f64 = dict(device="cuda", dtype=torch.float64)
    out = {"loss": torch.zeros(N, **f64), "dlogits": torch.zeros(N, V, **f64)}
    if c["more"]:
        out["lse"] = torch.zeros(N, **f64)
        if est not in DENSE:
            out["gathered"] = torch.zeros(N, K, **f64)
        if est in SUPPORT:
            out["coverage"] = torch.zeros(N, 2, **f64)
    cache = s["cache"]
    for a, b in _rows(N, V):
        keep = torch.ones(b - a, **f64) if s["mask"] is None else s["mask"][a:b].double()
        z = s["logits"][a:b].double()
        L = torch.logsumexp(z, 1)
        p = (z - L[:, None]).exp()
        if est in DENSE:
            y = cache["teacher_logits"][a:b].double()
            lr = z - L[:, None] - (y - torch.logsumexp(y, 1)[:, None])
            q = (z - L[:, None] - lr).exp()
            loss = (p * lr).sum(1) if est == "rkl_dense" else -(q * lr).sum(1)
            g = p * (lr - loss[:, None]) if est == "rkl_dense" else p - q
        else:
            ids = cache["idx" if est in SUPPORT else "sampled_ids"][a:b].long()
            tau = cache["teacher_logp"][a:b].double()
            zk = z.gather(1, ids)
            lp = zk - L[:, None]
            if est in ("fkl_topk", "rkl_topk"):
                lpt = zk - torch.logsumexp(zk, 1, True)
                lqt = tau - torch.logsumexp(tau, 1, True)
                pt, qt = lpt.exp(), lqt.exp()
                loss = (qt * (lqt - lpt) if est == "fkl_topk" else pt * (lpt - lqt)).sum(1)
                spike = pt - qt if est == "fkl_topk" else pt * (lpt - lqt - loss[:, None])
                coef = torch.zeros_like(loss)
            elif est in SUPPORT:
                pk, q = lp.exp(), tau.exp()
                if est == "fkl_topk_trunc":
                    loss, spike, coef = (q * (tau - lp)).sum(1), -q, q.sum(1)
                else:
                    spike = pk * (lp - tau + 1)
                    loss, coef = (pk * (lp - tau)).sum(1), -spike.sum(1)
            else:
                w, term = _mc_weights(est, lp, tau, cache["behav_logp"][a:b].double())
                loss, spike, coef = -term.mean(1), -w / K, w.mean(1)
            g = p.mul_(coef[:, None]).scatter_add_(1, ids, spike)
            if c["more"]:
                out["gathered"][a:b] = zk * keep[:, None]
                if est in SUPPORT:
                    out["coverage"][a:b] = torch.stack((lp.exp().sum(1), tau.exp().sum(1)), 1) * keep[:, None]
        out["loss"][a:b] = loss * keep
        out["dlogits"][a:b] = g * (gamma * keep)[:, None]
        if c["more"]:
            out["lse"][a:b] = L * keep
    return out


def _exact_rows(c, s):
    N, V, K = c["N"], c["V"], c["K"]
    f64 = dict(device="cuda", dtype=torch.float64)
    lse, logp = torch.zeros(N, **f64), torch.zeros(N, K, **f64)
    for a, b in _rows(N, V):
        z = s["logits"][a:b].double()
        L = torch.logsumexp(z, 1)
        if c["op"] == "topk":
            zk = z.topk(K).values
        elif c["op"] == "score":
            zk = z.gather(1, s["ids"][a:b].long())
        else:
            cdf = (z - z.amax(1, True)).exp().cumsum(1)
            t = s["uniforms"][a:b].double() * cdf[:, -1:]
            zk = z.gather(1, torch.searchsorted(cdf, t, right=True).clamp_(max=V - 1))
        keep = torch.ones(b - a, **f64) if s["mask"] is None else s["mask"][a:b].double()
        lse[a:b], logp[a:b] = L * keep, (zk - L[:, None]) * keep[:, None]
    out = {"logp": logp, "lse": lse}
    if c["op"] != "score":
        out["ids" if c["op"] == "sample" else "idx"] = None
    return out


def _exact_diag(c, s):
    N, K = c["N"], c["K"]
    f64 = dict(device="cuda", dtype=torch.float64)
    keep = torch.ones(N, device="cuda", dtype=torch.bool) if s["mask"] is None else s["mask"].bool()
    lp = s["gathered"].double() - s["lse"].double()[:, None]
    rho = (lp - s["behav_logp"].double()).exp()
    X = -rho * (s["teacher_logp"].double() - lp)
    zero = torch.zeros(N, **f64)
    flat = rho[keep].reshape(-1).sort().values
    q = float(torch.tensor(0.99, dtype=torch.float32))
    rank = max(1, math.ceil(q * flat.numel()))
    groups = {m: X.reshape(N, K // m, m).mean(2) for m in (1,) + GROUPS}
    local = {m: y.var(1)[keep].sum() for m, y in groups.items()}
    seq = {}
    for m, y in groups.items():
        total = 0.0
        for t in range(0, N, SEQ):
            v = keep[t:t + SEQ]
            if bool(v.any()):
                total = total + y[t:t + SEQ][v].mean(0).var()
        seq[m] = total
    return {"row_mean": torch.where(keep, X.mean(1), zero), "row_var": torch.where(keep, X.var(1), zero),
            "row_rho_max": torch.where(keep, rho.amax(1), zero),
            "rho_quantile": flat[rank - 1].reshape(1),
            "clip_frac": ((flat - 1).abs() > CLIP).double().mean().reshape(1),
            "ratio_local": torch.stack([local[m] / local[1] for m in GROUPS]),
            "ratio_seq": torch.stack([seq[m] / seq[1] for m in GROUPS])}


def exact(case, seed):
    s = prepare(case, seed)
    if case["op"] == "loss":
        return _exact_loss(case, s)
    return _exact_diag(case, s) if case["op"] == "diag" else _exact_rows(case, s)
