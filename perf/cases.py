"""The framework's measured workloads: rollout steps, teacher-forced scoring, value estimates, the
learning phase's gradients and kernels, and the LoRA merge, each called as a training program calls them.

Sizes come from the presets of paper_2505_18719_amd/inputs.py (tiny, mid, the OpenVLA-7B decoder shape) and
from bench.py; where a case runs fewer decoder layers than its preset, the layers left out do the same work
as those that run.  `exact` is a plain torch implementation in 64 bits of what the calls compute."""
import math

import numpy as np
import torch

from paper_2505_18719_amd import inputs, vla

DEV = "cuda"
LR_KEYS = inputs.LORA_PROJECTIONS
W7B = {"d": 4096, "heads": 32, "ffn": 11008}
WMID = {"d": 1024, "heads": 16, "ffn": 2752}
MAX_SEQ = 320       # longest sequence of one environment
SCALE = 0.5         # alpha / rank of the LoRA adapters
EPS = 0.2           # PPO clipping parameter


def _case(name, kind, layers, batch, shape=W7B, n_visual=256, prompt_min=32, prompt_max=32, **more):
    return {"name": name, "kind": kind, "layers": layers, "batch": batch, "n_visual": n_visual,
            "prompt_min": prompt_min, "prompt_max": prompt_max, **shape, **more}


def listed():
    return [
        # rollout steps (prefill, 7-token decode, action extraction)
        # the tiny preset: a smoke-sized policy, where latency and launches count
        _case("step_tiny_b4", "step", 2, 4, {"d": 256, "heads": 4, "ffn": 688}, prompt_min=16, prompt_max=16),
        # the mid preset, whole
        _case("step_mid_b16", "step", 8, 16, WMID),
        # one robot: the evaluation of a policy in a single environment, the 7B decoder's layers
        _case("step_7b_b1", "step", 4, 1, prompt_min=21, prompt_max=21),
        # the batch-8 preset's layers
        _case("step_7b_b8", "step", 4, 8),
        # the headline workload, whole: 64 environments with ragged prompts through all 32 layers
        _case("step_7b_b64", "step", 32, 64, prompt_min=16, prompt_max=48),
        # the learner's scoring of stored actions: the 128-action PPO minibatch of the 7B decoder
        _case("score_7b_b128", "score", 4, 128),
        # the critic's forward over a small vectorised environment
        _case("value_7b_b24", "value", 4, 24, prompt_min=16, prompt_max=48),
        # one PPO update's gradient of every LoRA factor: the 7B decoder's layers with kept activations, and the
        # mid preset with adapters on the query and value projections only and its activations recomputed
        _case("grads_7b_b16", "grads", 4, 16, prompt_min=16, prompt_max=48, rank=32, adapt="all", keep=True),
        _case("grads_mid_b16", "grads", 8, 16, WMID, rank=16, adapt="qv", keep=False),
        # the merge of a layer's adapters before a rollout, and the merged weights read back
        _case("merge_7b_r32", "merge", 1, 1, rank=32),
        # the learner's kernels around the model, over a rollout window: GAE, then the PPO loss, its gradient and
        # the logits gradient of every stored action (a small window taken as one batch, and a large one)
        {"name": "learn_64x64", "kind": "learn", "envs": 64, "steps": 64, "bins": 256},
        {"name": "learn_256x256", "kind": "learn", "envs": 256, "steps": 256, "bins": 256},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw(rng):
    kind = rng.choice(["step", "step", "step", "score", "value", "grads", "grads", "merge", "learn"])
    if kind == "learn":
        envs = _log_int(rng, 1, 4096)
        return {"kind": kind, "envs": envs, "steps": _log_int(rng, 1, max(1, min(512, 65536 // envs))),
                "bins": rng.choice([256, 256, 200, 64])}
    d = 256 * _log_int(rng, 1, 16)
    hd = rng.choice([64, 128])
    c = {"kind": kind, "layers": rng.randint(1, 4), "batch": _log_int(rng, 1, 128), "n_visual": rng.choice([256, 256, 64]),
         "d": d, "heads": d // hd, "ffn": 8 * int(d * rng.uniform(2.0, 3.0) / 8)}
    c["prompt_min"] = rng.randint(0 if kind == "step" else 1, 24)
    c["prompt_max"] = rng.randint(c["prompt_min"], 57)
    if kind == "grads":
        c.update(batch=_log_int(rng, 1, 24), rank=rng.choice([8, 16, 32, 64, 12]), adapt=rng.choice(["all", "all", "qv"]),
                 keep=rng.random() < 0.6)
    if kind == "merge":
        c.update(batch=1, layers=1, rank=rng.choice([8, 16, 24, 32, 64]))
    return c


def _cost(c):
    w = work(c)
    return w["flops"] / 1e15 + w["bytes"] / 4e12


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        c = _draw(rng)
        if _cost(c) <= most:
            return c


# ------------------------------------------------------------------ the sizes
def _cfg(c):
    return inputs.VlaConfig("case", n_layers=c["layers"], d_model=c["d"], n_heads=c["heads"], d_ffn=c["ffn"],
                            n_visual=c["n_visual"], batch=c["batch"], prompt_min=c["prompt_min"],
                            prompt_max=c["prompt_max"])


def _adapted(c):
    return LR_KEYS if c["adapt"] == "all" else ("wq", "wv")


def work(case):
    """Bytes of the inputs, weights and outputs once per pass over them, and the flops that cannot be left out:
    of the last layer only the rows that are read afterwards need more than its keys and values."""
    if case["kind"] == "learn":
        n, na, a = case["envs"] * case["steps"], 7, case["bins"]
        gae = n * (4 + 4 + 1 + 4 + 4)
        ppo = n * (3 * na * 4 + 4)
        lpb = n * na * (2 * a * 4 + 8)
        return {"bytes": gae + ppo + lpb, "flops": n * (10.0 + 4 * na + 6.0 * na * a)}
    c = _cfg(case)
    d, f, L, B, na = c.d_model, c.d_ffn, c.n_layers, c.batch, c.n_actions
    attn_w, mlp_w = 4.0 * d * d, 3.0 * d * f
    per = attn_w + mlp_w
    if case["kind"] == "merge":
        r = case["rank"]
        merge = 2 * 2.0 * per + 2.0 * r * (4 * 2 * d + 3 * (d + f))
        return {"bytes": merge + 2 * 2.0 * per, "flops": 2.0 * r * per}  # the merge, and its result read back
    pre = c.n_visual + 0.5 * (c.prompt_min + c.prompt_max)
    tf = case["kind"] in ("score", "grads")
    rows = pre + (na if tf else 0)
    need = na if tf else 1  # rows of each sequence read after the last layer
    M = B * rows
    lin = 2.0 * M * per * (L - 1) + 2.0 * M * 2 * d * d + 2.0 * B * need * (2 * d * d + mlp_w)
    att = B * 2.0 * d * rows * (rows + 1) * (L - 1) + B * need * 4.0 * d * rows
    weights = 2.0 * per * L
    io = 2.0 * B * c.n_visual * d
    if case["kind"] == "grads":
        n = len(_adapted(case))
        fe = sum(d + (f if k in ("wgate", "wup", "wdown") else d) for k in _adapted(case))
        lora = 8.0 * M * case["rank"] * fe * L
        return {"bytes": 2 * weights + io + 2.0 * case["rank"] * fe * L * 3 + n, "flops": 2 * lin + 3 * att + lora}
    if case["kind"] != "step":
        return {"bytes": weights + io, "flops": lin + att}
    kv = sum(2.0 * 2.0 * d * (pre + i) for i in range(1, na)) * B * L
    passes = (na - 1) * ((B + 127) // 128)
    return {"bytes": weights * (1 + passes) + kv + io, "flops": lin + att + (na - 1) * 2.0 * B * per * L}


# ------------------------------------------------------------------ inputs
def _gen(seed, *key):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(np.random.SeedSequence([int(seed), *key]).generate_state(1, np.uint64)[0] >> np.uint64(1)))
    return g


def _policy(c, case, seed):
    """Weights (for "grads" with the adapters merged in, the policy a rollout runs) and adapters."""
    w = inputs.make_weights(c, seed=seed, device=DEV, gain_jitter=True)
    if case["kind"] not in ("grads", "merge"):
        return w, None
    ad = inputs.make_lora(c, case["rank"], seed=seed, device=DEV)
    if case["kind"] == "grads":
        keys = _adapted(case)
        ad = [{k: layer[k] for k in keys} for layer in ad]
        for lw, layer in zip(w["layers"], ad):
            for k, (a, b) in layer.items():
                lw[k] = (lw[k].float() + SCALE * (b.float() @ a.float())).to(torch.bfloat16).contiguous()
    return w, ad


def _batch(c, seed):
    inp = inputs.make_inputs(c, seed=seed, device=DEV)
    return inp, torch.from_numpy(inp.prompt_ids).to(DEV)


def _old_logp(case, seed, logp):
    """The rollout policy's log-probs of the stored actions: the current ones moved as a few updates move them (a
    ratio spread of 0.15 over actions), none on a clip edge, where rounding would decide the branch."""
    g = _gen(seed, 7)
    B, na = logp.shape
    shift = 0.15 * torch.randn(B, generator=g, device=DEV, dtype=torch.float64)
    for edge in (math.log(1 + EPS), math.log(1 - EPS)):
        near = (shift - edge).abs() < 0.06
        shift = torch.where(near, shift + torch.where(shift > edge, 0.08, -0.08), shift)
    tok = 0.05 * torch.randn(B, na, generator=g, device=DEV, dtype=torch.float64)
    tok = tok - tok.mean(1, keepdim=True) + shift[:, None] / na  # ratio = exp(shift)
    return (logp - tok).float().contiguous()


def _advantages(case, seed):
    return torch.randn(case["batch"], generator=_gen(seed, 8), device=DEV)


def _window(case, seed):
    """A rollout window: rewards, values, episode starts; then every stored action's old and new token log-probs,
    logits over the bins and token."""
    N, M, na, A = case["envs"], case["steps"], 7, case["bins"]
    g = _gen(seed, 9)
    r, v, dn = inputs.rollout_window(N, M, seed=seed)
    n = N * M
    z = 1.3 * torch.randn(n * na, A, generator=g, device=DEV)
    tokens = torch.randint(0, A, (n * na,), generator=g, device=DEV, dtype=torch.int32) + 31808
    new = -torch.empty(n, na, device=DEV).exponential_(0.25, generator=g)
    old = new + 0.05 * torch.randn(n, na, generator=g, device=DEV)
    return {"rewards": torch.from_numpy(r).to(DEV), "values": torch.from_numpy(v).to(DEV),
            "dones": torch.from_numpy(dn).to(DEV), "z": z, "tokens": tokens, "new": new, "old": old}


def prepare(case, seed):
    kind = case["kind"]
    if kind == "learn":
        return dict(_window(case, seed), kind=kind)
    c = _cfg(case)
    w, ad = _policy(c, case, seed)
    s = {"kind": kind, "cfg": c, "model": vla.VlaModel(c, w, device=DEV)}
    if kind == "merge":
        # a checkpoint stays resident beside the policy: every merge starts from it
        s.update(w0=w["layers"], ad=ad)
        d, fp = c.d_model, (c.d_ffn + 255) // 256 * 256
        s["sizes"] = [(r + 15) // 16 * (k // 32 + 1) * 512 for r, k in ((3 * d, d), (d, d), (2 * fp, d), (d, fp))]
        return s
    inp, ids = _batch(c, seed)
    s.update(vis=inp.vis, ids=ids, lens=inp.prompt_lens)
    if kind == "step":
        s["gumbel"] = torch.from_numpy(inp.gumbel).to(DEV)
        s["lo"] = torch.linspace(-1.0, -0.4, c.n_actions, device=DEV)
        s["hi"] = torch.linspace(0.5, 1.2, c.n_actions, device=DEV)
    if kind == "value":
        s["head"] = (0.02 * torch.randn(c.d_model, generator=_gen(seed, 6), device=DEV)).to(torch.bfloat16)
    if kind in ("score", "grads"):
        s["actions"] = torch.from_numpy(inputs.stored_actions(c, c.batch, seed=seed)).to(DEV)
    if kind == "grads":
        with torch.no_grad():
            logp = _score64(c, w, inp, s["actions"])[0]
        s.update(ad=ad, old=_old_logp(case, seed, logp), adv=_advantages(case, seed),
                 mode=vla.TRAIN_KEEP if case["keep"] else vla.TRAIN_RECOMPUTE)
    return s


# ------------------------------------------------------------------ one pass
def run(s):
    kind = s["kind"]
    if kind == "learn":
        adv, ret = vla.gae(s["rewards"], s["values"], s["dones"], 0.99, 0.95)
        stats, dlogp = vla.ppo_clip(s["new"], s["old"], adv.view(-1), EPS)
        dz = vla.logprob_backward(s["z"], s["tokens"], 31808, 1.5, dlogp.view(-1))
        return {"adv": adv, "ret": ret, "loss": stats, "dlogp": dlogp, "dz": dz}
    m = s["model"]
    if kind == "step":
        first = m.prefill(s["vis"], s["ids"], s["lens"])
        out = m.decode_actions(s["gumbel"], 1.5)
        act = vla.extract_actions(out["tokens"], s["cfg"].action_begin, s["cfg"].action_bins, s["lo"], s["hi"])
        return dict(out, first=first, act=act)
    if kind == "score":
        return m.token_logprobs(s["vis"], s["ids"], s["lens"], s["actions"], 1.5)
    if kind == "value":
        return m.value(s["vis"], s["ids"], s["lens"], s["head"])
    if kind == "grads":
        stats, logp, grads = m.ppo_lora_grads(s["vis"], s["ids"], s["lens"], s["actions"], s["old"], s["adv"], EPS, 1.5,
                                              s["ad"], SCALE, mode=s["mode"])
        return {"loss": stats, "logp": logp, "grads": grads}
    m.lora_merge_layer(0, s["w0"][0], s["ad"][0], SCALE)
    return [m.debug_read(5 + i, 0, torch.empty(n, dtype=torch.bfloat16, device=DEV)) for i, n in enumerate(s["sizes"])]


# ------------------------------------------------------------------ tolerances
def tolerance(case):
    """Of another correct implementation at the same precision: fp32 sums in another order, and where bf16 values
    are stored (all of the model's calls), the values that then round the other way, carried through the layers.
    An fp32 torch implementation with the same bf16 rounding points is 3e-3 (tiny), 7e-3 (four layers of 7B width)
    and 9e-3 (mid) from the framework's logits, 8e-3 from its values and up to 2e-2 from its gradients."""
    return {
        "step": {"rel": 0.03, "max": 0.2, "differ": 0.01},
        "score": {"rel": 0.03, "max": 0.15},
        "value": {"rel": 0.03, "max": 0.1},
        "grads": {"rel": 0.03, "max": 0.5},
        "merge": {"rel": 1e-4, "max": 0.01},  # rank sums in another order: a few values round the other way
        "learn": {"rel": 1e-5, "max": 1e-3},
    }[case["kind"]]


# ------------------------------------------------------------------ 64 bits
def _rms64(x, g, eps):
    return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + eps) * g.double()


def _rope64(x, pos, base):
    hd = x.shape[-1]
    ang = pos.double()[:, None] * base ** (-2.0 * torch.arange(hd // 2, device=DEV, dtype=torch.float64) / hd)
    c, s = ang.cos()[:, None], ang.sin()[:, None]
    a, b = x[..., :hd // 2], x[..., hd // 2:]
    return torch.cat([a * c - b * s, a * s + b * c], -1)


def _hidden64(c, w, inp, actions, params=None):
    """Residual rows of every sequence after the last layer, and where each sequence starts; `params`: per layer the
    projections to use in place of the weights."""
    xs, pos, at, o = [], [], [], 0
    for b in range(c.batch):
        ids = torch.from_numpy(np.asarray(inp.env_prompt(b), dtype=np.int64)).to(DEV)
        parts = [inp.vis[b].double(), w["embed"][ids].double()]
        if actions is not None:
            parts.append(w["embed"][actions[b].long()].double())
        x = torch.cat(parts)
        xs.append(x)
        pos.append(torch.arange(x.shape[0], device=DEV))
        at.append((o, o + x.shape[0]))
        o += x.shape[0]
    x, pos = torch.cat(xs), torch.cat(pos)
    H, hd = c.n_heads, c.head_dim
    for li, lw in enumerate(w["layers"]):
        W = params[li] if params is not None else {k: lw[k].double() for k in LR_KEYS}
        u = _rms64(x, lw["attn_norm"], c.rms_eps)
        q = _rope64((u @ W["wq"].T).view(-1, H, hd), pos, c.rope_base)
        k = _rope64((u @ W["wk"].T).view(-1, H, hd), pos, c.rope_base)
        v = (u @ W["wv"].T).view(-1, H, hd)
        outs = []
        for a, e in at:
            qb, kb, vb = (t[a:e].transpose(0, 1).contiguous() for t in (q, k, v))
            sc = torch.matmul(qb, kb.transpose(1, 2).contiguous()) / math.sqrt(hd)
            sc = sc.masked_fill(torch.ones(e - a, e - a, device=DEV, dtype=torch.bool).triu(1), -math.inf)
            outs.append(torch.matmul(sc.softmax(-1), vb).transpose(0, 1).reshape(e - a, -1))
        x = x + torch.cat(outs) @ W["wo"].T
        u = _rms64(x, lw["mlp_norm"], c.rms_eps)
        x = x + (torch.nn.functional.silu(u @ W["wgate"].T) * (u @ W["wup"].T)) @ W["wdown"].T
    return x, at


def _logits64(c, w, h):
    return _rms64(h, w["final_norm"], c.rms_eps) @ w["lm_head"][c.action_begin:c.action_begin + c.action_bins].double().T


def _score64(c, w, inp, actions, params=None):
    """Teacher-forced log-probs, entropies [B, n_actions] and logits [B, n_actions, bins]."""
    x, at = _hidden64(c, w, inp, actions, params)
    na = c.n_actions
    h = torch.cat([x[e - na - 1:e - 1] for _, e in at])
    z = _logits64(c, w, h).view(c.batch, na, -1)
    lp = (z / 1.5).log_softmax(-1)
    k = (actions.long() - c.action_begin).unsqueeze(-1)
    return lp.gather(-1, k).squeeze(-1), -(lp.exp() * lp).sum(-1), z


def _frag64(rows):
    """A matrix [R, K] in the packed layout that reading the weights back documents (one spare block per 16 rows)."""
    R, K = rows.shape
    t = rows.view(R // 16, 16, K // 32, 4, 8).permute(0, 2, 3, 1, 4).reshape(R // 16, K // 32, 512)
    return torch.cat([t, t.new_zeros(R // 16, 1, 512)], 1).reshape(-1)


def _merged64(case, seed):
    c = _cfg(case)
    w, ad = _policy(c, case, seed)
    W = {k: w["layers"][0][k].double() + SCALE * (b.double() @ a.double()) for k, (a, b) in ad[0].items()}
    d, f, hd = c.d_model, c.d_ffn, c.head_dim
    fp = (f + 255) // 256 * 256
    i = torch.arange(hd // 2, device=DEV).view(-1, 32)
    head = torch.stack([i, i + hd // 2], 1).reshape(-1)
    qk = (torch.arange(c.n_heads, device=DEV)[:, None] * hd + head).reshape(-1)
    up = {k: torch.cat([W[k], W[k].new_zeros(fp - f, d)]).view(fp // 32, 32, d) for k in ("wgate", "wup")}
    return [_frag64(torch.cat([W["wq"][qk], W["wk"][qk], W["wv"]])), _frag64(W["wo"]),
            _frag64(torch.stack([up["wgate"], up["wup"]], 1).reshape(2 * fp, d)),
            _frag64(torch.cat([W["wdown"], W["wdown"].new_zeros(d, fp - f)], 1))]


def _learn64(case, seed):
    s = _window(case, seed)
    r, v, go = s["rewards"].double(), s["values"].double(), 1.0 - (s["dones"][1:] != 0).double()
    n = r.numel()
    adv, a = torch.empty_like(r), torch.zeros_like(r[0])
    g, lam = float(np.float32(0.99)), float(np.float32(0.95))
    for t in reversed(range(r.shape[0])):
        a = r[t] + g * go[t] * v[t + 1] - v[t] + g * lam * go[t] * a
        adv[t] = a
    A = adv.reshape(-1)
    eps = float(np.float32(EPS))
    rho = (s["new"].double().sum(1) - s["old"].double().sum(1)).exp()
    loss = -torch.minimum(rho * A, rho.clamp(1 - eps, 1 + eps) * A).mean()
    cut = ((A > 0) & (rho > 1 + eps)) | ((A < 0) & (rho < 1 - eps))
    dl = torch.where(cut, 0.0, -rho * A / n)[:, None].expand(-1, 7).contiguous()
    p = (s["z"].double() / 1.5).softmax(-1)
    one = torch.nn.functional.one_hot(s["tokens"].long() - 31808, case["bins"]).double()
    dz = dl.reshape(-1, 1) * (one - p) / 1.5
    return {"adv": adv, "ret": adv + v[:-1], "loss": torch.stack([loss, cut.double().mean()]), "dlogp": dl, "dz": dz}


def exact(case, seed):
    kind = case["kind"]
    if kind == "learn":
        return _learn64(case, seed)
    if work(case)["flops"] > 4e14:  # minutes in 64 bits
        return None
    if kind == "merge":
        return _merged64(case, seed)
    c = _cfg(case)
    w, ad = _policy(c, case, seed)
    inp, _ = _batch(c, seed)
    if kind in ("step", "value"):
        with torch.no_grad():
            x, at = _hidden64(c, w, inp, None)
            h = torch.stack([x[e - 1] for _, e in at])
            if kind == "value":
                head = (0.02 * torch.randn(c.d_model, generator=_gen(seed, 6), device=DEV)).to(torch.bfloat16)
                return _rms64(h, w["final_norm"], c.rms_eps) @ head.double()
            # the tokens after the first depend on draws that rounding can decide: no 64-bit value stands for them
            return {"first": _logits64(c, w, h), "act": None, "tokens": None, "logp": None, "entropy": None,
                    "logits": None}
    actions = torch.from_numpy(inputs.stored_actions(c, c.batch, seed=seed)).to(DEV)
    if kind == "score":
        with torch.no_grad():
            lp, ent, z = _score64(c, w, inp, actions)
        return {"logp": lp, "entropy": ent, "logits": z}
    params = [{k: lw[k].double().requires_grad_(k in layer) for k in LR_KEYS} for lw, layer in zip(w["layers"], ad)]
    lp, _, _ = _score64(c, w, inp, actions, params)
    old, A = _old_logp(case, seed, lp.detach()).double(), _advantages(case, seed).double()
    eps = float(np.float32(EPS))
    rho = (lp.sum(1) - old.sum(1)).exp()
    loss = -torch.minimum(rho * A, rho.clamp(1 - eps, 1 + eps) * A).mean()
    with torch.no_grad():
        cut = ((A > 0) & (rho > 1 + eps)) | ((A < 0) & (rho < 1 - eps))
    loss.backward()
    grads = [{k: (SCALE * b.double().T @ p[k].grad, SCALE * p[k].grad @ a.double().T) for k, (a, b) in layer.items()}
             for p, layer in zip(params, ad)]
    return {"loss": torch.stack([loss.detach(), cut.double().mean()]), "logp": lp.detach(), "grads": grads}
