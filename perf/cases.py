"""The work this library is asked to do, as cases that can be timed and compared.

A training update with the multi-step GRPO loss makes these calls: the loss and its gradient from logits (on one
device, or on one device's columns of a split vocabulary), the proximal log-probs and entropies recomputed before an
update, and the same from hidden states and the LM-head weight.  The cases go through the public entry points of
``paper_2606_05597_amd`` on batches shaped like the rollouts the loss is for: groups of G trajectories, failures
longer than successes, ragged steps and tokens, policies that are sure of most tokens and unsure of some.

``listed()`` holds the fixed cases, ``draw(rng)`` gives others of the same ranges.
"""
import math

import numpy as np
import torch

import paper_2606_05597_amd as grpo

EPS, DUAL_C, K = 0.2, 3.0, 10.0
MAX_BYTES = 9.2e9    # logits of the largest logits case
MAX_FLOPS = 5.4e13   # products of the largest fused case


# ---- the cases ----------------------------------------------------------------------------------------------------

def listed():
    return [
        # a smoke-sized step, as in unit tests and debugging runs: launches and host time are all there is
        {"name": "loss_tiny", "kind": "loss", "dtype": "f32", "T": 192, "V": 1024, "ld": 1024, "G": 4, "prox": False,
         "norm": "k", "aux": False},
        # an update of a model with a 32,000-word vocabulary, the paper's baseline normaliser, metrics collected
        {"name": "loss_32k", "kind": "loss", "dtype": "bf16", "T": 32411, "V": 32000, "ld": 32000, "G": 8,
         "prox": False, "norm": "steps", "aux": True},
        # the same size of model after tokens were added to its tokenizer: an odd vocabulary, rows that start anywhere
        {"name": "loss_32k_odd", "kind": "loss", "dtype": "bf16", "T": 9001, "V": 32003, "ld": 32003, "G": 8,
         "prox": True, "norm": "k", "aux": False},
        # the large-vocabulary model of the paper, one micro-batch of an update, proximal log-probs given
        {"name": "loss_152k", "kind": "loss", "dtype": "bf16", "T": 30000, "V": 151936, "ld": 151936, "G": 8,
         "prox": True, "norm": "k", "aux": False},
        # its tokenizer's words alone, in the columns of a head that is padded for the hardware
        {"name": "loss_152k_padded", "kind": "loss", "dtype": "bf16", "T": 6007, "V": 151669, "ld": 151936, "G": 8,
         "prox": True, "norm": "k", "aux": False},
        # a trainer that keeps its logits in 32 bits
        {"name": "loss_152k_f32", "kind": "loss", "dtype": "f32", "T": 6000, "V": 151936, "ld": 151936, "G": 8,
         "prox": True, "norm": "k", "aux": False},
        # proximal log-probs and entropies recomputed before an update, from logits
        {"name": "logp_152k", "kind": "logp", "dtype": "bf16", "T": 24000, "V": 151936, "ld": 151936, "entropy": True},
        # one device's eighth of the vocabulary: its records, then the loss and its columns of the gradient
        {"name": "shard_19k", "kind": "shard", "dtype": "bf16", "T": 32768, "V": 18992, "ld": 18992, "G": 8,
         "n_shards": 8, "prox": True, "norm": "k"},
        # the LM head and the loss in one, a large batch in token blocks on two streams
        {"name": "fused_16k", "kind": "fused", "T": 16384, "H": 3584, "V": 151936, "G": 8, "schedule": "blocked",
         "streams": 2, "autograd": False, "prox": True, "norm": "k"},
        # a micro-batch of a few hundred tokens through autograd, the gradients in the parameters' type
        {"name": "fused_autograd_700", "kind": "fused", "T": 700, "H": 3584, "V": 151936, "G": 8,
         "schedule": "blocked", "streams": 1, "autograd": True, "prox": False, "norm": "k"},
        # proximal log-probs and entropies from hidden states
        {"name": "fused_logp_4k", "kind": "fused_logp", "T": 4001, "H": 3584, "V": 151936, "entropy": True},
        # one device's eighth of the LM head: its records, then its columns of dW and its share of dhidden
        {"name": "fused_shard_8k", "kind": "fused_shard", "T": 8192, "H": 3584, "V": 18992, "G": 8, "n_shards": 8,
         "keep": True, "prox": True, "norm": "k"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["loss", "loss", "loss", "logp", "shard", "fused", "fused", "fused_logp", "fused_shard"])
    common = {"G": rng.choice([4, 8, 16]), "prox": rng.random() < 0.5, "norm": rng.choice(["k", "steps"])}
    if kind in ("loss", "logp", "shard"):
        dtype = rng.choice(["bf16", "bf16", "f32"])
        top = 33000 if kind == "shard" else 262144
        V = _log_int(rng, 1000, top)
        form = rng.choice(["whole", "odd", "padded"])
        if form == "whole":
            V = max(8, V // 8 * 8)
        ld = (V + 255) // 256 * 256 if form == "padded" else V
        T = _log_int(rng, 64, max(65, min(40000, int(MAX_BYTES / (ld * (2 if dtype == "bf16" else 4))))))
        case = {"kind": kind, "dtype": dtype, "T": T, "V": V, "ld": ld}
        if kind == "logp":
            return {**case, "entropy": rng.random() < 0.7}
        if kind == "shard":
            return {**case, **common, "n_shards": rng.choice([2, 4, 8])}
        return {**case, **common, "aux": rng.random() < 0.3}
    H = 64 * _log_int(rng, 8, 64)
    V = 8 * _log_int(rng, 250, 2400 if kind == "fused_shard" else 18992)
    products = 1 if kind == "fused_logp" else 3
    T = _log_int(rng, 48, max(49, min(16384, int(MAX_FLOPS / (2 * products * H * V)))))
    case = {"kind": kind, "T": T, "H": H, "V": V}
    if kind == "fused_logp":
        return {**case, "entropy": rng.random() < 0.7}
    if kind == "fused_shard":
        return {**case, **common, "n_shards": rng.choice([2, 4, 8]), "keep": rng.random() < 0.7}
    schedule = rng.choice(["blocked", "blocked", "chunked"])
    return {**case, **common, "schedule": schedule, "streams": rng.choice([1, 2]) if schedule == "blocked" else 1,
            "autograd": rng.random() < 0.3}


# ---- inputs --------------------------------------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _row_chunks(T, V, elements=1 << 27):
    rows = max(1, elements // V)
    return [(r, min(T, r + rows)) for r in range(0, T, rows)]


def _rollouts(case, seed):
    """Rewards, the CSR offsets and the advantages of a batch of T action tokens: mixed groups, failures longer."""
    T, G = case["T"], case["G"]
    rng = np.random.default_rng(seed)
    n_groups = max(1, min(16, T // 2000))
    n = n_groups * G
    rewards = np.zeros(n, np.float32)
    for g in range(n_groups):
        won = rng.integers(1, max(2, G // 2 + 1))
        rewards[g * G + rng.permutation(G)[:won]] = 1.0
    steps = np.where(rewards > 0, rng.integers(3, 13, n), rng.integers(8, 31, n))
    share = rng.geometric(1.0 / 96.0, int(steps.sum())).astype(np.float64)
    cum = np.concatenate([[0.0], np.cumsum(share)])
    sto = np.floor(cum * (T / cum[-1]) + 1e-9).astype(np.int32)
    sto[-1] = T
    tso = np.concatenate([[0], np.cumsum(steps)]).astype(np.int32)
    r = torch.from_numpy(rewards).double().reshape(n_groups, G)
    adv = ((r - r.mean(1, keepdim=True)) / r.std(1, keepdim=True)).reshape(-1)
    return {"rewards": torch.from_numpy(rewards).cuda(), "sto": torch.from_numpy(sto).cuda(),
            "tso": torch.from_numpy(tso).cuda(), "adv": adv.float().cuda()}


def _policy_rows(z, seed):
    """Raises one word of three rows in four by 4 to 20, so that the policy is sure of most tokens, in place."""
    T, V = z.shape
    g = _gen(seed)
    at = torch.randint(0, V, (T, 1), generator=g, device="cuda")
    up = 4 + 16 * torch.rand((T, 1), generator=g, device="cuda")
    up = torch.where(torch.rand((T, 1), generator=g, device="cuda") < 0.75, up, torch.zeros_like(up))
    z.scatter_add_(1, at, up.to(z.dtype))


def _sample(z, seed):
    """Actions drawn from softmax(z), int32, and their log-probs in float32."""
    u = torch.rand(z.shape, generator=_gen(seed), device="cuda").clamp_(min=1e-30).log_().neg_().log_().neg_()
    act = torch.argmax(u.add_(z), dim=1)
    z = z.float()
    return act.to(torch.int32), z.gather(1, act[:, None])[:, 0] - torch.logsumexp(z, dim=1)


def _off_the_kinks(new, old):
    """`old`, moved where pi/pi_old lies within 1e-3 of the clip range's ends or of the dual clip's factor, where
    rounding alone would decide which branch a token takes."""
    for _ in range(2):
        r = torch.exp(new - old)
        near = ((r - (1 - EPS)).abs() < 1e-3) | ((r - (1 + EPS)).abs() < 1e-3) | ((r - DUAL_C).abs() < 1e-2)
        old = torch.where(near, old + 0.02, old)
    return old


def _old_logps(case, logp, seed):
    """The rollout's log-probs (a slightly older policy, a few tokens far off) and the proximal ones, or None."""
    g = _gen(seed)
    n = torch.randn(logp.shape, generator=g, device="cuda")
    far = torch.rand(logp.shape, generator=g, device="cuda") < 0.02
    behave = _off_the_kinks(logp, logp + torch.where(far, 0.6, 0.05) * n)
    prox = None
    if case["prox"]:
        prox = _off_the_kinks(logp, behave + 0.05 * torch.randn(logp.shape, generator=g, device="cuda"))
    return behave.contiguous(), prox


def _logits_inputs(case, seed):
    T, V, ld = case["T"], case["V"], case["ld"]
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    logits = torch.zeros((T, ld), dtype=dt, device="cuda") if ld != V else torch.empty((T, V), dtype=dt, device="cuda")
    act = torch.empty(T, dtype=torch.int32, device="cuda")
    logp = torch.empty(T, device="cuda")
    for c, (a, b) in enumerate(_row_chunks(T, V)):
        z = torch.randn((b - a, V), generator=_gen(seed * 7919 + c), device="cuda").mul_(2.0)
        _policy_rows(z, seed * 6007 + c)
        logits[a:b, :V] = z
        act[a:b], logp[a:b] = _sample(logits[a:b, :V], seed * 104729 + c)
    return logits, act, logp


def _hidden_inputs(case, seed):
    """Hidden states and a weight whose product is sure of most tokens, actions drawn from it and their log-probs."""
    T, H, V = case["T"], case["H"], case["V"]
    W = torch.empty((H, V), dtype=torch.bfloat16, device="cuda").normal_(0.0, 1.2 / math.sqrt(H), generator=_gen(seed * 13 + 2))
    g = _gen(seed * 13 + 1)
    h = torch.randn((T, H), generator=g, device="cuda")
    at = torch.randint(0, V, (T,), generator=g, device="cuda")
    up = (4 + 16 * torch.rand((T, 1), generator=g, device="cuda")) / 1.2
    up = torch.where(torch.rand((T, 1), generator=g, device="cuda") < 0.75, up, torch.zeros_like(up))
    dirs = W[:, at].float().t()
    h = (h + up * dirs / dirs.norm(dim=1, keepdim=True)).to(torch.bfloat16)
    act = torch.empty(T, dtype=torch.int32, device="cuda")
    logp = torch.empty(T, device="cuda")
    Wf = W.float()
    for c, (a, b) in enumerate(_row_chunks(T, V)):
        act[a:b], logp[a:b] = _sample(h[a:b].float() @ Wf, seed * 977 + c)
    return h, W, act, logp


def _other_shards(case, own, seed):
    """The records of the n_shards - 1 devices that hold the rest of the vocabulary: (max, sum, action logit), of
    logits like this shard's; a token in n_shards has its action here, the others have it there."""
    T, n = case["T"], case["n_shards"]
    g = _gen(seed)
    m = own[None, :, 0] + 2.0 * torch.randn((n - 1, T), generator=g, device="cuda", dtype=torch.float64)
    s = 1.0 + torch.rand((n - 1, T), generator=g, device="cuda", dtype=torch.float64) * 20.0
    return m, s


def _shard_records(case, z_of_rows, act_local, seed):
    """All shards' records [n_shards, T, 3] in float64, this device's among them (shard 0), the global action ids and
    their log-probs over the whole vocabulary."""
    T, V, n = case["T"], case["V"], case["n_shards"]
    own = torch.empty((T, 3), dtype=torch.float64, device="cuda")
    for a, b in _row_chunks(T, V, 1 << 26):
        z = z_of_rows(a, b).double()
        own[a:b, 0] = z.max(1).values
        own[a:b, 1] = torch.exp(z - own[a:b, :1]).sum(1)
        own[a:b, 2] = z.gather(1, act_local[a:b].long()[:, None])[:, 0]
    m, s = _other_shards(case, own, seed * 17 + 3)
    g = _gen(seed * 17 + 4)
    owner = torch.randint(0, n, (T,), generator=g, device="cuda")
    here = owner == 0
    own[:, 2] = torch.where(here, own[:, 2], -math.inf)
    rec = torch.empty((n, T, 3), dtype=torch.float64, device="cuda")
    rec[0] = own
    rec[1:, :, 0], rec[1:, :, 1] = m, s
    rec[1:, :, 2] = -math.inf
    for k in range(1, n):
        rec[k, :, 2] = torch.where(owner == k, m[k - 1] - torch.rand(T, generator=g, device="cuda", dtype=torch.float64), -math.inf)
    act = torch.where(here, act_local, (owner * V + act_local.long() % V).to(torch.int32)).to(torch.int32)
    M = rec[:, :, 0].max(0).values
    lse = M + torch.log((rec[:, :, 1] * torch.exp(rec[:, :, 0] - M)).sum(0))
    return rec, act, (rec[:, :, 2].max(0).values - lse).float()


def _as_records(rec):
    return rec.contiguous().view(torch.uint8).reshape(rec.shape[0], rec.shape[1], 24)


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind in ("loss", "logp", "shard"):
        s["logits"], s["act"], logp = _logits_inputs(case, seed)
        if kind == "shard":
            rec, s["act"], logp = _shard_records(case, lambda a, b: s["logits"][a:b, :case["V"]], s["act"], seed)
            s["others"] = _as_records(rec)
    else:
        s["h"], s["W"], s["act"], logp = _hidden_inputs(case, seed)
        if kind == "fused_shard":
            Wf = s["W"].float()
            rec, s["act"], logp = _shard_records(case, lambda a, b: s["h"][a:b].float() @ Wf, s["act"], seed)
            del Wf
            s["others"] = _as_records(rec)
            if case["keep"]:
                s["kept"] = grpo.vocab_shard_logits_buffer(case["T"], case["V"], "cuda")
    if kind not in ("logp", "fused_logp"):
        s.update(_rollouts(case, seed * 31 + 7))
        s["behave"], s["prox"] = _old_logps(case, logp, seed * 31 + 2)
        n_traj = s["tso"].numel() - 1
        if case.get("aux"):
            s["aux"] = grpo.LossAux.alloc(case["T"], n_traj, "cuda", which=("token_logp", "traj_loss", "clip_counts",
                                                                            "ratio_stats", "error_flags"))
    if kind == "fused" and case["autograd"]:
        s["h"].requires_grad_(True)
        s["W"].requires_grad_(True)
    if kind == "fused" and case["streams"] == 2:
        s["aux_stream"] = torch.cuda.Stream()
    return s


# ---- one pass ------------------------------------------------------------------------------------------------------

def _opts(s):
    return {"prox_logp": s["prox"], "norm": grpo.GRPO_NORM_CONST_K if s["case"]["norm"] == "k" else
            grpo.GRPO_NORM_TRAJ_STEPS, "k": K, "eps_low": EPS, "eps_high": EPS, "dual_clip_c": DUAL_C}


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "loss":
        aux = s.get("aux")
        loss, dl = grpo.loss(s["logits"], s["act"], s["behave"], s["rewards"], s["sto"], s["tso"], c["G"], V=c["V"],
                             aux=aux, **_opts(s))
        out = {"loss": loss, "dlogits": dl[:, :c["V"]] if c["V"] < c["ld"] else dl}  # columns past V aren't written
        if aux is not None:
            out.update(logp=aux.token_logp, traj_loss=aux.traj_loss, clips=aux.clip_counts, ratios=aux.ratio_stats,
                       flags=aux.error_flags)
        return out
    if kind == "logp":
        logp, ent = grpo.grpo_token_logp(s["logits"], s["act"], V=c["V"], entropy=c["entropy"])
        return {"logp": logp, "entropy": ent}
    if kind == "shard":
        every = s["others"]
        grpo.grpo_vocab_shard_stats(s["logits"], s["act"], 0, V=c["V"], stats=every[0])
        loss, dl = grpo.grpo_loss_fwd_bwd_vocab_shard(s["logits"], every, 0, c["V"] * c["n_shards"], s["act"],
                                                      s["behave"], s["adv"], s["sto"], s["tso"], c["G"], V=c["V"],
                                                      **_opts(s))
        m, za, sm = grpo.vocab_stats_fields(every[0])
        return {"loss": loss, "dlogits": dl[:, :c["V"]] if c["V"] < c["ld"] else dl, "m": m, "sum": sm, "z_a": za}
    if kind == "fused_logp":
        logp, ent = grpo.fused_lmhead_token_logp(s["h"], s["W"], s["act"], entropy=c["entropy"])
        return {"logp": logp, "entropy": ent}
    if kind == "fused_shard":
        every, kept = s["others"], s.get("kept")
        grpo.fused_lmhead_vocab_shard_stats(s["h"], s["W"], s["act"], 0, stats=every[0], logits_out=kept)
        loss, dh, dw = grpo.fused_lmhead_grpo_vocab_shard(s["h"], s["W"], every, 0, c["V"] * c["n_shards"], s["act"],
                                                          s["behave"], s["adv"], s["sto"], s["tso"], c["G"],
                                                          logits_in=kept, **_opts(s))
        m, za, sm = grpo.vocab_stats_fields(every[0])
        return {"loss": loss, "dhidden": dh, "dW": dw, "m": m, "sum": sm, "z_a": za}
    args = (s["h"], s["W"], s["act"], s["behave"], s["adv"], s["sto"], s["tso"], c["G"])
    opts = _opts(s)
    if c["schedule"] == "blocked" and c["streams"] == 2:
        opts["aux_stream"] = s["aux_stream"]
    if c["autograd"]:
        s["h"].grad = s["W"].grad = None
        loss = grpo.FusedLmHeadGrpoLoss.apply(*args, {**opts, "schedule": c["schedule"]})
        loss.backward()
        return {"loss": loss.detach(), "dhidden": s["h"].grad, "dW": s["W"].grad}
    entry = grpo.fused_lmhead_grpo_blocked if c["schedule"] == "blocked" else grpo.fused_lmhead_grpo
    loss, dh, dw = entry(*args, **opts)
    return {"loss": loss, "dhidden": dh, "dW": dw}


# ---- what a pass cannot do without ------------------------------------------------------------------------------------

def work(case):
    kind, T, V = case["kind"], case["T"], case["V"]
    if kind in ("loss", "logp", "shard"):
        e = 2 if case["dtype"] == "bf16" else 4
        if kind == "logp":
            return {"bytes": T * (e * V + 12), "flops": 4 * T * V}
        if kind == "loss":
            return {"bytes": T * (2 * e * V + 16), "flops": 6 * T * V}
        return {"bytes": T * (3 * e * V + 24 * (case["n_shards"] + 1) + 16), "flops": 8 * T * V}
    H = case["H"]
    if kind == "fused_logp":
        return {"bytes": 2 * (T + V) * H + 12 * T, "flops": 2 * T * H * V}
    # h and W read once, dhidden and dW written once
    dh = 4 if kind == "fused_shard" else 2
    dw = 2 if case.get("autograd") else 4
    return {"bytes": (2 + dh) * T * H + (2 + dw) * H * V, "flops": 6 * T * H * V}


def tolerance(case):
    kind = case["kind"]
    if kind in ("loss", "shard"):
        # float32: the exponent's argument and the log-sum-exp carry a few 1e-7 of values up to 30; bfloat16: values
        # next to a rounding boundary go either way
        return {"rel": 5e-6, "max": 2e-4} if case["dtype"] == "f32" else {"rel": 4e-3, "max": 2e-2}
    if kind == "logp":
        return {"rel": 1e-6, "max": 1e-4}
    if kind == "fused_logp":
        return {"rel": 5e-6, "max": 1e-3}
    # dlogits are rounded to bfloat16 before the two products of the gradients
    return {"rel": 1e-2, "max": 5e-2}


# ---- the same in 64 bits, in plain torch --------------------------------------------------------------------------------

def _token_terms(s, logp, adv):
    """Per token, in float64: its share of the loss, and minus d(loss)/d(log-prob)."""
    c = s["case"]
    sto, tso = s["sto"].long(), s["tso"].long()
    n = tso.numel() - 1
    start = sto[tso]
    traj = torch.searchsorted(start, torch.arange(c["T"], device="cuda"), right=True) - 1
    traj = traj.clamp(max=n - 1)
    den = (tso[1:] - tso[:-1]).double() if c["norm"] == "steps" else torch.full((n,), K, device="cuda", dtype=torch.float64)
    w = (1.0 / (n * den))[traj]
    A = adv.double()[traj]
    b = s["behave"].double()
    p = b if s["prox"] is None else s["prox"].double()
    rho, r, omega = torch.exp(logp - b), torch.exp(logp - p), torch.exp(p - b)
    u1, u2 = rho * A, omega * r.clamp(1 - EPS, 1 + EPS) * A
    inside = (r >= 1 - EPS) & (r <= 1 + EPS)
    eps_cut = (u2 < u1) & ~inside
    term = torch.minimum(u1, u2)
    dual_cut = (A < 0) & (term < DUAL_C * A)
    term = torch.where(dual_cut, DUAL_C * A, term)
    g = torch.where(eps_cut | dual_cut, torch.zeros_like(w), w * u1)
    share = -w * term
    return {"share": share, "g": g, "traj": traj, "n": n, "rho": rho, "r": r, "eps_cut": eps_cut, "dual_cut": dual_cut,
            "outside": ~inside}


def _dlogits_rows(z, lse, g, act, here=None):
    d = torch.exp(z - lse[:, None])
    hot = torch.ones_like(lse) if here is None else here.double()
    d.scatter_add_(1, act[:, None], -hot[:, None])
    return d.mul_(g[:, None])


def _exact_rows(s, z_of_rows, entropy=False):
    c = s["case"]
    T, V = c["T"], c["V"]
    lse = torch.empty(T, dtype=torch.float64, device="cuda")
    za, ent = torch.empty_like(lse), torch.empty_like(lse)
    for a, b in _row_chunks(T, V, 1 << 26):
        z = z_of_rows(a, b)
        lse[a:b] = torch.logsumexp(z, 1)
        za[a:b] = z.gather(1, s["act"][a:b].long().clamp(max=V - 1)[:, None])[:, 0]
        if entropy:
            l = z - lse[a:b, None]
            ent[a:b] = -(torch.exp(l) * l).sum(1)
    return lse, za, ent


def exact(case, seed):
    kind, T, V = case["kind"], case["T"], case["V"]
    s = prepare(case, seed)
    if kind in ("loss", "logp", "shard"):
        z_of_rows = lambda a, b: s["logits"][a:b, :V].double()  # noqa: E731
    else:
        W = s["W"].detach().double()
        z_of_rows = lambda a, b: s["h"][a:b].detach().double() @ W  # noqa: E731
    act = s["act"].long()
    if kind in ("logp", "fused_logp"):
        lse, za, ent = _exact_rows(s, z_of_rows, case["entropy"])
        return {"logp": za - lse, "entropy": ent if case["entropy"] else None}
    out = {}
    here = None
    if kind in ("shard", "fused_shard"):
        here = act < V
        rec = s["others"].view(torch.float64).clone()
        own, za, _ = _exact_rows(s, z_of_rows)
        for a, b in _row_chunks(T, V, 1 << 26):
            rec[0, a:b, 0] = z_of_rows(a, b).max(1).values
        rec[0, :, 1] = torch.exp(own - rec[0, :, 0])
        rec[0, :, 2] = torch.where(here, za, -math.inf)
        M = rec[:, :, 0].max(0).values
        lse = M + torch.log((rec[:, :, 1] * torch.exp(rec[:, :, 0] - M)).sum(0))
        logp = rec[:, :, 2].max(0).values - lse
        out.update(m=rec[0, :, 0], sum=rec[0, :, 1], z_a=rec[0, :, 2])
    else:
        lse, za, _ = _exact_rows(s, z_of_rows)
        logp = za - lse
    t = _token_terms(s, logp, s["adv"])
    out["loss"] = t["share"].sum().reshape(() if case.get("autograd") else (1,))
    col = act.clamp(max=V - 1)
    if kind in ("loss", "shard"):
        dl = torch.empty((T, V), dtype=torch.float64, device="cuda")
        for a, b in _row_chunks(T, V, 1 << 26):
            dl[a:b] = _dlogits_rows(z_of_rows(a, b), lse[a:b], t["g"][a:b], col[a:b], None if here is None else here[a:b])
        out["dlogits"] = dl
        if case.get("aux"):
            r, rho = t["r"], t["rho"]
            out["logp"] = logp
            out["traj_loss"] = torch.zeros(t["n"], dtype=torch.float64, device="cuda").index_add_(0, t["traj"], t["share"])
            out["ratios"] = torch.stack([r.sum(), r.min(), r.max(), rho.sum(), rho.min(), rho.max(),
                                         t["outside"].sum().double(), torch.tensor(float(T), device="cuda", dtype=torch.float64)])
            out["clips"] = out["flags"] = None
        return out
    H = case["H"]
    dh = torch.empty((T, H), dtype=torch.float64, device="cuda")
    dW = torch.zeros((H, V), dtype=torch.float64, device="cuda")
    for a, b in _row_chunks(T, V, 1 << 28):
        D = _dlogits_rows(z_of_rows(a, b), lse[a:b], t["g"][a:b], col[a:b], None if here is None else here[a:b])
        dh[a:b] = D @ W.t()
        dW.addmm_(s["h"][a:b].detach().double().t(), D)
    out["dhidden"], out["dW"] = dh, dW
    return out
