"""Timed cases of the rollout library, through its public calls.

The path decodes redundant trajectories, scores them and selects training
groups.  Its calls are the stateless kernels (paged decode attention, the fused
sampler, group selection with page reclaim, the decoder's projections) and the
rollout context (prefill, decode steps, selection).  The sizes are those of the
repository's own configurations: the Qwen3-8B- and Qwen3-30B-A3B-shaped
decoders, the tiny fp32 one, and the kernel sweep.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2605_30859_amd import binding as B

PAGE = 16
DEV = "cuda"

# Decoder widths of the repository's configurations.  A case takes a few layers
# of them: a layer is what repeats.
MODELS = {
    "tiny": dict(d_model=128, n_q_heads=4, n_kv_heads=4, head_dim=32, ffn_dim=512, dtype="f32",
                 rope_theta=1e4),
    "dense-small": dict(d_model=1024, n_q_heads=16, n_kv_heads=4, head_dim=64, ffn_dim=4096,
                        dtype="bf16", rope_theta=1e4),
    "qwen3-8b": dict(d_model=4096, n_q_heads=32, n_kv_heads=8, head_dim=128, ffn_dim=12288,
                     dtype="bf16", rope_theta=1e6),
    "qwen3-30b-a3b": dict(d_model=2048, n_q_heads=32, n_kv_heads=4, head_dim=128, ffn_dim=0,
                          dtype="bf16", rope_theta=1e6, n_experts=128, top_k=8, expert_ffn=768),
}

# Projections of those decoders: (N, K, epilogue).  Epilogues: 0 fp32 result (QKV,
# LM head), 2 residual add (O, down), 3 SwiGLU (gate/up).
PROJ = {
    "8b-qkv": (6144, 4096, 0), "8b-o": (4096, 4096, 2), "8b-gate-up": (24576, 4096, 3),
    "8b-down": (4096, 12288, 2), "8b-lm-head": (151936, 4096, 0),
    "moe-qkv": (5120, 2048, 0), "moe-o": (2048, 4096, 2), "moe-lm-head": (151936, 2048, 0),
    "small-qkv": (1536, 1024, 0), "small-gate-up": (8192, 1024, 3), "small-down": (1024, 4096, 2),
}


def listed():
    return [
        # a whole small rollout, run to its last kept set: launches and host calls
        # are what it costs (the tiny fp32 decoder, as smoke() runs it)
        dict(name="rollout-tiny-f32", kind="rollout", model="tiny", layers=2, vocab=512, prompts=4,
             prompt_len=16, m=8, k=4, steps=24),
        # decode attention over trajectories of any length (the kernel sweep)
        dict(name="attn-ragged-1024", kind="attn", rows=1024, hq=32, hkv=8, hd=128, ctx=1500, sigma=1.0),
        # a decode step of the MoE rollout while most trajectories are live
        dict(name="attn-decode-777", kind="attn", rows=777, hq=32, hkv=4, hd=128, ctx=1123, sigma=0.0),
        # the long tail of a rollout: a few long trajectories of the 8B decoder
        dict(name="attn-tail-19", kind="attn", rows=19, hq=32, hkv=8, hd=128, ctx=5211, sigma=0.0),
        # sampling and scoring a full decode batch (the kernel sweep)
        dict(name="sample-1024-bf16", kind="sample", rows=1024, vocab=151936, dtype="bf16",
             temperature=1.0, forced=0.0),
        # the same late in a rollout: few rows, fp32 logits, some tokens forced
        dict(name="sample-21-f32", kind="sample", rows=21, vocab=151936, dtype="f32", temperature=0.7,
             forced=0.25),
        # group selection with the pages of every finished group given back (the sweep)
        dict(name="select-4096-groups", kind="select", groups=4096, m=16, k=8, m_up=16, median=1000),
        # projections of a decode step: a large batch, the tail, and the prefill's
        # largest one.  A step walks the layers, so each pass takes several weights.
        dict(name="gemm-gate-up-389", kind="gemm", proj="8b-gate-up", rows=389, layers=3),
        dict(name="gemm-down-45", kind="gemm", proj="8b-down", rows=45, layers=5),
        dict(name="gemm-prefill-gate-up", kind="gemm", proj="8b-gate-up", rows=16384, layers=1),
        # the prefill of the MoE rollout: 64 prompts of 512 tokens, first tokens sampled
        dict(name="prefill-moe", kind="rollout", model="qwen3-30b-a3b", layers=2, vocab=151936,
             prompts=64, prompt_len=512, m=16, k=8, steps=0),
        # MoE decode steps with selection: the batch shrinks from 976 rows as members end
        dict(name="decode-moe", kind="rollout", model="qwen3-30b-a3b", layers=2, vocab=4096,
             prompts=61, prompt_len=48, m=16, k=8, steps=10),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["attn", "attn", "sample", "select", "gemm", "gemm", "rollout", "rollout"])
    if kind == "attn":
        hq, hkv, hd = rng.choice([(32, 8, 128), (32, 4, 128), (16, 4, 64)])
        rows, ragged = _log(rng, 1, 1024), rng.random() < 0.4
        ctx = _log(rng, 16, 1500 if ragged else min(16000, 2000000 // rows))
        return dict(kind=kind, rows=rows, hq=hq, hkv=hkv, hd=hd, ctx=ctx, sigma=1.0 if ragged else 0.0)
    if kind == "sample":
        return dict(kind=kind, rows=_log(rng, 1, 1024), vocab=rng.choice([512, 4096, 32000, 151936]),
                    dtype=rng.choice(["bf16", "f32"]), temperature=rng.choice([1.0, 1.0, 0.7]),
                    forced=rng.choice([0.0, 0.25]))
    if kind == "select":
        m = rng.choice([8, 12, 16, 32])
        return dict(kind=kind, groups=_log(rng, 4, 4096), m=m, k=m // 2, m_up=rng.choice([m, m + 1]),
                    median=_log(rng, 50, 1000) * 16 // max(m, 16))
    if kind == "gemm":
        proj = rng.choice(sorted(PROJ))
        rows = _log(rng, 1, 512 if "lm-head" in proj else 16384)
        return dict(kind=kind, proj=proj, rows=rows, layers=1 if rows > 512 or "lm-head" in proj else 4)
    model = rng.choice(["tiny", "dense-small", "qwen3-8b", "qwen3-30b-a3b"])
    big = model in ("qwen3-8b", "qwen3-30b-a3b")
    steps = 0 if rng.random() < 0.4 else rng.randint(2, 10)
    prompts = _log(rng, 1, 8 if model == "tiny" else 32 if steps else 48)
    plen = 16 * _log(rng, 1, 4 if model == "tiny" else 8 if steps else 32)
    m = rng.choice([8, 16])
    return dict(kind="rollout", model=model, layers=rng.choice([1, 2]), vocab=512 if model == "tiny" else 4096,
                prompts=prompts, prompt_len=plen, m=m, k=m // 2, steps=min(steps, 6) if big else steps)


def _gen(seed, salt=0):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 1000003 + salt)


def _rng(seed, *more):
    return np.random.default_rng([int(seed), *more])


# ------------------------------------------------------------------ attention
def _contexts(case):
    """Context lengths, ascending: the case's own, whatever the seed."""
    if case["sigma"] == 0.0:
        return np.full(case["rows"], case["ctx"], dtype=np.int64)
    p = (np.arange(case["rows"]) + 0.5) / case["rows"]
    z = math.sqrt(2.0) * torch.erfinv(torch.tensor(2 * p - 1)).numpy()
    return np.clip(np.rint(case["ctx"] * np.exp(case["sigma"] * z)), 16, 32768).astype(np.int64)


def _attn_inputs(case, seed):
    rng, g = _rng(seed, 1), _gen(seed, 1)
    ctx = rng.permutation(_contexts(case))
    npg = -(-ctx // PAGE)
    total = int(npg.sum())
    perm = rng.permutation(total).astype(np.int32)
    pt = np.full((case["rows"], int(npg.max())), -1, dtype=np.int32)
    off = 0
    for r, n in enumerate(npg):
        pt[r, :n] = perm[off:off + n]
        off += n
    hkv, hd = case["hkv"], case["hd"]
    # pools in the library's page layouts: K [page][kv head][hd/32][slot][32],
    # V [page][kv head][slot/8][hd][slot%8]
    k = torch.empty(total, hkv, hd // 32, PAGE, 32, dtype=torch.bfloat16, device=DEV).normal_(generator=g)
    v = torch.empty(total, hkv, 2, hd, 8, dtype=torch.bfloat16, device=DEV).normal_(generator=g)
    q = torch.empty(case["rows"], case["hq"], hd, dtype=torch.bfloat16, device=DEV).normal_(generator=g)
    return ctx, pt, q, k, v


def _attn_prepare(case, seed):
    ctx, pt, q, k, v = _attn_inputs(case, seed)
    rows, hq, hkv, hd = case["rows"], case["hq"], case["hkv"], case["hd"]
    mx = int(ctx.max())
    ws = torch.empty(B.darts_attn_workspace_bytes(rows, hq, hkv, hd, mx), dtype=torch.uint8, device=DEV)
    return SimpleNamespace(case=case, q=q, k=k, v=v, n_pages=k.shape[0], pt=torch.from_numpy(pt).to(DEV), mx=mx,
                           ctx=torch.from_numpy(ctx.astype(np.int32)).to(DEV) if case["sigma"] else None,
                           out=torch.empty_like(q), ws=ws)


def _attn_run(s):
    c = s.case
    B.darts_attn_decode(s.q, s.k, s.v, s.n_pages, s.pt, s.ctx, c["hq"], c["hkv"], c["hd"], s.mx, B.DARTS_BF16,
                        s.out, s.ws, n_rows=c["rows"])
    return s.out


def _attn_exact(case, seed):
    ctx, pt, q, k, v = _attn_inputs(case, seed)
    hq, hkv, hd = case["hq"], case["hkv"], case["hd"]
    out = torch.empty(q.shape, dtype=torch.float64, device=DEV)
    for r in range(case["rows"]):
        n = int(ctx[r])
        ids = torch.from_numpy(pt[r, :-(-n // PAGE)].astype(np.int64)).to(DEV)
        kr = k[ids].permute(1, 0, 3, 2, 4).reshape(hkv, -1, hd)[:, :n].double()
        vr = v[ids].permute(1, 0, 2, 4, 3).reshape(hkv, -1, hd)[:, :n].double()
        s = q[r].double().view(hkv, hq // hkv, hd) @ kr.transpose(1, 2).contiguous() / math.sqrt(hd)
        out[r] = (torch.softmax(s, -1) @ vr).reshape(hq, hd)
    return out


def _attn_work(case):
    ctx = _contexts(case).astype(np.float64)
    io = 2.0 * case["rows"] * case["hq"] * case["hd"] * 2
    kv = ctx.sum() * case["hkv"] * case["hd"] * 4
    return dict(bytes=kv + io + 4 * np.ceil(ctx / PAGE).sum(), flops=4.0 * ctx.sum() * case["hq"] * case["hd"])


# -------------------------------------------------------------------- sampler
def _sample_inputs(case, seed):
    g, rng = _gen(seed, 2), _rng(seed, 2)
    n, v = case["rows"], case["vocab"]
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    logits = torch.empty(n, v, dtype=dt, device=DEV).normal_(0.0, 3.0, generator=g)
    traj = torch.from_numpy(np.sort(rng.choice(4 * n, n, replace=False)).astype(np.int32)).to(DEV)
    step = torch.from_numpy(np.full(n, rng.integers(0, 4096), dtype=np.int32)).to(DEV)
    force = None
    if case["forced"]:
        f = np.where(rng.random(n) < case["forced"], rng.integers(0, v, n), -1).astype(np.int32)
        force = torch.from_numpy(f).to(DEV)
    return logits, traj, step, force


def _sample_prepare(case, seed):
    logits, traj, step, force = _sample_inputs(case, seed)
    n = case["rows"]
    return SimpleNamespace(case=case, seed=int(seed) + 11, logits=logits, traj=traj, step=step, force=force,
                           tok=torch.empty(n, dtype=torch.int32, device=DEV),
                           lp=torch.empty(n, device=DEV), ent=torch.empty(n, device=DEV))


def _sample_run(s):
    c = s.case
    B.darts_sample(s.logits, B.DARTS_BF16 if c["dtype"] == "bf16" else B.DARTS_F32, s.seed, s.traj, s.step,
                   c["temperature"], s.force, s.tok, s.lp, s.ent)
    return dict(token=s.tok, logprob=s.lp, entropy=s.ent)


def _philox(c0, c1, c2, c3, k0, k1):
    """Philox4x32-10 on int64 tensors holding 32-bit words."""
    m = 0xFFFFFFFF

    def mul(a, x):   # 32 x 32 -> (high, low), in halves that fit int64
        lo, hi = a * (x & 0xFFFF), a * (x >> 16)
        t = (lo >> 16) + (hi & m)
        return ((hi >> 32) * 65536 + (t >> 16)) & m, ((t & 0xFFFF) << 16) | (lo & 0xFFFF)

    for _ in range(10):
        h0, l0 = mul(0xD2511F53, c0)
        h1, l1 = mul(0xCD9E8D57, c2)
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & m, (k1 + 0xBB67AE85) & m
    return c0, c1, c2, c3


def _sample_exact(case, seed):
    logits, traj, step, force = _sample_inputs(case, seed)
    n, v = case["rows"], case["vocab"]
    t32 = torch.tensor(case["temperature"], dtype=torch.float32, device=DEV)
    lp = torch.empty(n, dtype=torch.float64, device=DEV)
    ent = torch.empty_like(lp)
    j = torch.arange(v // 4, device=DEV, dtype=torch.int64)
    for r in range(n):
        z = (logits[r].float() / t32).double()
        w = _philox(j, torch.full_like(j, int(traj[r])), torch.full_like(j, int(step[r])), torch.full_like(j, 2),
                    (seed + 11) & 0xFFFFFFFF, (seed + 11) >> 32)
        u = ((torch.stack(w, 1).reshape(-1) >> 8) | 1).double() / 2 ** 24
        tok = int(torch.argmax(z - torch.log(-torch.log(u))))
        if force is not None and int(force[r]) >= 0:
            tok = int(force[r])
        lse = torch.logsumexp(z, 0)
        p = torch.exp(z - lse)
        lp[r] = z[tok] - lse
        ent[r] = lse - (p * z).sum()
    return dict(token=None, logprob=lp, entropy=ent)


def _sample_work(case):
    n, v = case["rows"], case["vocab"]
    # a counter word, two logarithms, an exponential and the running sums per logit
    return dict(bytes=n * v * (2.0 if case["dtype"] == "bf16" else 4.0) + 24.0 * n, flops=40.0 * n * v)


# ------------------------------------------------------------------ selection
def _select_sizes(case):
    n = case["groups"] * case["m"]
    p = (np.arange(n) + 0.5) / n
    z = math.sqrt(2.0) * torch.erfinv(torch.tensor(2 * p - 1)).numpy()
    ln = np.clip(np.rint(case["median"] * np.exp(z)), 1, 8192).astype(np.int32)
    return np.random.default_rng(7).permutation(ln)


def _select_prepare(case, seed):
    rng = _rng(seed, 3)
    ln = _select_sizes(case).reshape(case["groups"], case["m"])
    ln = rng.permutation(ln, axis=0).reshape(-1)
    n = ln.size
    # most members have ended; one group in four still has live members, some of
    # them enough to hold it open
    st = np.where(ln >= 8192, 2, 1).astype(np.uint8)
    open_ = np.repeat(rng.random(case["groups"]) < 0.25, case["m"])
    st[open_ & (rng.random(n) < 0.5)] = 0
    mlp = -(np.floor(rng.random(n) * 3 * 1024) / 1024).astype(np.float32)
    npg = (ln.astype(np.int64) + PAGE - 1) // PAGE
    off = np.concatenate([[0], np.cumsum(npg)]).astype(np.int32)
    pages = rng.permutation(int(npg.sum())).astype(np.int32)
    t = lambda a: torch.from_numpy(a).to(DEV)  # noqa: E731
    i32 = dict(dtype=torch.int32, device=DEV)
    return SimpleNamespace(case=case, st=t(st), ln=t(ln), mlp=t(mlp), off=t(off), pages=t(pages),
                           kept=torch.full((case["groups"], case["k"]), -1, **i32),
                           done=torch.zeros(case["groups"], dtype=torch.uint8, device=DEV),
                           freed=torch.full((pages.size,), -1, **i32), nfree=torch.zeros(1, **i32),
                           work=torch.zeros(case["groups"] + 1, **i32))


def _select_run(s):
    c = s.case
    B.darts_select_groups(s.st, s.ln, s.mlp, c["m"], c["k"], 1, c["m_up"], 1, s.kept, s.done, s.off, s.pages,
                          s.freed, s.nfree, s.work)
    return dict(status=s.st, kept=s.kept, complete=s.done, freed=s.freed, n_freed=s.nfree)


def _select_work(case):
    ln = _select_sizes(case).astype(np.int64)
    pages = float(((ln + PAGE - 1) // PAGE).sum())
    return dict(bytes=ln.size * (1 + 4 + 4 + 4) + case["groups"] * (case["k"] * 4 + 1) + 8.0 * pages * 0.8,
                flops=0.0)


# ---------------------------------------------------------------- projections
def _gemm_inputs(case, seed):
    n, k, epi = PROJ[case["proj"]]
    g, m = _gen(seed, 4), case["rows"]
    a = torch.empty(m, k, dtype=torch.bfloat16, device=DEV).normal_(generator=g)
    lim = math.sqrt(3.0 / k)
    w = [torch.empty(n, k, dtype=torch.bfloat16, device=DEV).uniform_(-lim, lim, generator=g)
         for _ in range(case["layers"])]
    if epi == 2:
        c = [torch.empty(m, n, device=DEV).normal_(generator=g) for _ in w]
    elif epi == 3:
        c = [torch.empty(m, n // 2, dtype=torch.bfloat16, device=DEV) for _ in w]
    else:
        c = [torch.empty(m, n, device=DEV) for _ in w]
    return a, w, c


def _gemm_prepare(case, seed):
    a, w, c = _gemm_inputs(case, seed)
    n, k, epi = PROJ[case["proj"]]
    nb = B.darts_gemm_workspace_bytes(case["rows"], n, k)
    ws = torch.empty(nb, dtype=torch.uint8, device=DEV) if nb else None
    return SimpleNamespace(a=a, w=w, c=c, ws=ws, m=case["rows"], n=n, k=k, epi=epi)


def _gemm_run(s):
    for w, c in zip(s.w, s.c):
        B.darts_gemm(s.a, w, c, s.m, s.n, s.k, B.DARTS_BF16, s.epi, s.ws)
    return s.c


def _gemm_exact(case, seed):
    a, w, c = _gemm_inputs(case, seed)
    n, k, epi = PROJ[case["proj"]]
    if 2.0 * case["rows"] * n * k * case["layers"] > 2e14:
        return None
    a, out = a.double(), []
    for wl, cl in zip(w, c):
        y = a @ wl.double().T
        if epi == 2:
            y = y + cl.double()
        elif epi == 3:   # W rows: 16 gate rows, then the 16 up rows of the same features
            y = y.view(case["rows"], n // 32, 2, 16)
            y = (torch.nn.functional.silu(y[:, :, 0]) * y[:, :, 1]).reshape(case["rows"], n // 2)
        out.append(y)
    return out


def _gemm_work(case):
    n, k, epi = PROJ[case["proj"]]
    m = case["rows"]
    c = {0: 4.0 * m * n, 2: 8.0 * m * n, 3: 1.0 * m * n}[epi]
    return dict(bytes=case["layers"] * (2.0 * n * k + c) + 2.0 * m * k, flops=2.0 * m * n * k * case["layers"])


# -------------------------------------------------------------------- rollout
def _cfgs(case):
    mc = dict(n_experts=0, top_k=0, expert_ffn=0, rms_eps=1e-6, weight_seed=0)
    mc.update(MODELS[case["model"]], n_layers=case["layers"], vocab=case["vocab"])
    rc = dict(n_prompts=case["prompts"], prompt_len=case["prompt_len"], m=case["m"], k=case["k"],
              cap=case["steps"] + 64, L=1, m_up=None, kv_pool_gb=0.0, sample_seed=5, temperature=1.0)
    return SimpleNamespace(**mc), SimpleNamespace(**rc)


def _lengths(case):
    """Forced lengths: distinct inside a group, so that members end one by one."""
    rng = np.random.default_rng(9)
    start = rng.integers(1, 4, case["prompts"])
    return np.concatenate([s + rng.permutation(case["m"]) for s in start]).astype(np.int32)


def _schedule(case):
    """The rows of every sampling step: a trajectory runs to its length, or until
    its group has k that have ended."""
    m, k, ln = case["m"], case["k"], _lengths(case)
    gen, live, steps = np.zeros_like(ln), np.ones(ln.size, dtype=bool), []
    ended = np.zeros(ln.size, dtype=bool)
    for _ in range(case["steps"] + 1):
        if not live.any():
            break
        steps.append(np.flatnonzero(live))
        gen[live] += 1
        ended |= live & (gen == ln)
        full = np.repeat(ended.reshape(-1, m).sum(1) >= k, m)
        live &= ~ended & ~full
    return steps, gen


def _weights(mc, seed):
    """The decoder's tensors in the order darts_model_cfg.weights documents."""
    g = _gen(seed, 5)
    dt = torch.bfloat16 if mc.dtype == "bf16" else torch.float32

    def w(fan, *shape):
        lim = math.sqrt(3.0 / fan)
        return torch.empty(*shape, dtype=dt, device=DEV).uniform_(-lim, lim, generator=g)

    d, f, e = mc.d_model, mc.ffn_dim, mc.n_experts
    q, kv = mc.n_q_heads * mc.head_dim, mc.n_kv_heads * mc.head_dim
    out = [w(1, mc.vocab, d), w(d, mc.vocab, d)]
    for _ in range(mc.n_layers):
        out += [w(d, q, d), w(d, kv, d), w(d, kv, d), w(q, d, q)]
        if e:
            fe = mc.expert_ffn
            # the router three times wider than the rest: a trained one is peaked, so
            # that a near tie for the last place carries little weight
            out += [w(d / 9.0, e, d), w(d, e, fe, d), w(d, e, fe, d), w(fe, e, d, fe)]
        else:
            out += [w(d, f, d), w(d, f, d), w(f, d, f)]
    return out


def _rollout_inputs(case, seed):
    rng = _rng(seed, 6)
    n = case["prompts"] * case["m"]
    prompts = rng.integers(0, case["vocab"], case["prompts"] * case["prompt_len"]).astype(np.int32)
    force = rng.integers(0, case["vocab"] - 1, (case["steps"] + 1, n)).astype(np.int32)
    return prompts, force


def _rollout_prepare(case, seed):
    mc, rc = _cfgs(case)
    prompts, force = _rollout_inputs(case, seed)
    ro = B.Rollout(mc, rc, weights=_weights(mc, seed))
    t = lambda a: torch.from_numpy(a).to(DEV)  # noqa: E731
    return SimpleNamespace(case=case, ro=ro, prompts=t(prompts), force=t(force), forced_len=t(_lengths(case)))


def _rollout_run(s):
    # tokens are teacher-forced, as in a scored replay: a sample is a near tie away
    # from another one, and every later value would follow it
    ro, c = s.ro, s.case
    ro.darts_reset()
    rows = ro.darts_prefill(s.prompts, s.forced_len, s.force[0])
    lp, ent = [rows["logprob"].clone()], [rows["entropy"].clone()]
    ro.darts_select_and_prune()
    step = 0
    while step < c["steps"] and ro.n_live > 0:
        step += 1
        rows = ro.darts_decode_step(s.force[step])
        lp.append(rows["logprob"].clone())
        ent.append(rows["entropy"].clone())
        ro.darts_select_and_prune()
    ln, total, mean, status = ro.traj_scores()
    return dict(logits=ro.debug_logits(ro.run.n_prompts if step == 0 else rows["traj"].numel()),
                logprob=torch.cat(lp), entropy=torch.cat(ent), kept=ro.kept.clone(), done=ro.done_step.clone(),
                length=ln, sum_logprob=total, mean_logprob=mean, status=status)


def _norm(x, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps)


def _forward(mc, w, tokens):
    """Plain float64 decoder over [sequences, positions]: the final hidden states."""
    b, t = tokens.shape
    hq, hkv, hd, d = mc.n_q_heads, mc.n_kv_heads, mc.head_dim, mc.d_model
    x = w[0].double()[tokens]
    inv = mc.rope_theta ** (-2.0 * torch.arange(hd // 2, device=DEV, dtype=torch.float64) / hd)
    ang = torch.arange(t, device=DEV, dtype=torch.float64)[:, None] * inv
    cos, sin = ang.cos()[:, None], ang.sin()[:, None]

    def rope(y):
        a, c = y[..., :hd // 2], y[..., hd // 2:]
        return torch.cat([a * cos - c * sin, c * cos + a * sin], -1)

    mask = torch.full((t, t), -math.inf, dtype=torch.float64, device=DEV).triu(1)
    per = 8 if mc.n_experts else 7
    silu = torch.nn.functional.silu
    for l in range(mc.n_layers):
        wl = w[2 + per * l: 2 + per * (l + 1)]
        h = _norm(x, mc.rms_eps)
        q = rope((h @ wl[0].double().T).view(b, t, hq, hd))
        k = rope((h @ wl[1].double().T).view(b, t, hkv, hd))
        v = (h @ wl[2].double().T).view(b, t, hkv, hd)
        o = torch.empty(b, t, hq * hd, dtype=torch.float64, device=DEV)
        for i in range(b):
            qi = q[i].view(t, hkv, hq // hkv, hd).permute(1, 2, 0, 3).reshape(hkv, -1, hd)
            s = (qi @ k[i].permute(1, 2, 0).contiguous() / math.sqrt(hd)).view(hkv, hq // hkv, t, t) + mask
            y = torch.softmax(s, -1).view(hkv, -1, t) @ v[i].permute(1, 0, 2).contiguous()
            o[i] = y.view(hkv, hq // hkv, t, hd).permute(2, 0, 1, 3).reshape(t, hq * hd)
        x = x + o @ wl[3].double().T
        h = _norm(x, mc.rms_eps)
        if not mc.n_experts:
            x = x + (silu(h @ wl[4].double().T) * (h @ wl[5].double().T)) @ wl[6].double().T
            continue
        h = h.view(-1, d)
        top, ids = torch.softmax(h @ wl[4].double().T, -1).topk(mc.top_k, -1)
        top = top / top.sum(-1, keepdim=True)
        y = torch.zeros_like(h)
        for e in range(mc.n_experts):
            r, c = (ids == e).nonzero(as_tuple=True)
            he = h[r]
            he = (silu(he @ wl[5][e].double().T) * (he @ wl[6][e].double().T)) @ wl[7][e].double().T
            y.index_add_(0, r, he * top[r, c][:, None])
        x = x + y.view(b, t, d)
    return _norm(x, mc.rms_eps)


def _rollout_exact(case, seed):
    mc, _ = _cfgs(case)
    if _rollout_work(case)["flops"] > 4e13:
        return None
    w = _weights(mc, seed)
    prompts, force = _rollout_inputs(case, seed)
    steps, gen = _schedule(case)
    P, lp_, m, n = case["prompts"], case["prompt_len"], case["m"], case["prompts"] * case["m"]
    ln = _lengths(case)
    tok = force[:len(steps)].copy()
    for g in range(n):
        if ln[g] <= len(steps):
            tok[ln[g] - 1, g] = case["vocab"] - 1
    pr = torch.from_numpy(prompts.astype(np.int64)).to(DEV).view(P, lp_)
    tk = torch.from_numpy(tok.astype(np.int64)).to(DEV)
    if len(steps) == 1:
        h, rows_of = _forward(mc, w, pr), [np.arange(n) // m]
    else:
        h = _forward(mc, w, torch.cat([pr.repeat_interleave(m, 0), tk[:-1].T.contiguous()], 1))
        rows_of = steps
    head = w[1].double()
    logprob, entropy, total = [], [], torch.zeros(n, dtype=torch.float64, device=DEV)
    for s, live in enumerate(steps):
        at = torch.from_numpy(np.asarray(rows_of[s] if len(steps) == 1 else live)).to(DEV)
        uniq, back = torch.unique(at, return_inverse=True) if len(steps) == 1 else (at, torch.arange(len(at), device=DEV))
        z = h[uniq, lp_ - 1 + s] @ head.T
        lsm = torch.log_softmax(z, -1)
        g = torch.from_numpy(live).to(DEV)
        t = tk[s, g]
        logprob.append(lsm[back, t])
        entropy.append(-(lsm.exp() * lsm).sum(-1)[back])
        total[g] += logprob[-1]
    return dict(logits=z, logprob=torch.cat(logprob), entropy=torch.cat(entropy), kept=None, done=None, length=None,
                sum_logprob=total, mean_logprob=total / torch.from_numpy(gen.astype(np.float64)).to(DEV), status=None)


def _rollout_work(case):
    mc, _ = _cfgs(case)
    d, q, kv = mc.d_model, mc.n_q_heads * mc.head_dim, mc.n_kv_heads * mc.head_dim
    es = 2 if mc.dtype == "bf16" else 4
    steps, _ = _schedule(case)
    lp_, P, V = case["prompt_len"], case["prompts"], case["vocab"]
    attn_w = d * (q + 2 * kv) + q * d
    total_b = total_f = 0.0
    for s, live in enumerate(steps):
        rows, heads = (P * lp_, P) if s == 0 else (len(live), len(live))
        keys = P * lp_ * (lp_ + 1) / 2 if s == 0 else len(live) * (lp_ + s)
        kv_bytes = P * lp_ * 2 * kv * es if s == 0 else keys * 2 * kv * es
        if mc.n_experts:
            each = 3 * d * mc.expert_ffn
            ffn_w = min(mc.n_experts, rows * mc.top_k) * each + mc.n_experts * d
            ffn_f = 2.0 * rows * (mc.top_k * each + mc.n_experts * d)
        else:
            ffn_w, ffn_f = 3 * d * mc.ffn_dim, 2.0 * rows * 3 * d * mc.ffn_dim
        total_b += mc.n_layers * ((attn_w + ffn_w) * es + kv_bytes) + V * d * es + heads * V * 4.0 + rows * d * es
        total_f += mc.n_layers * (2.0 * rows * attn_w + ffn_f + 4.0 * keys * q) + 2.0 * heads * V * d
    return dict(bytes=total_b, flops=total_f)


# ------------------------------------------------------------------------ all
def prepare(case, seed):
    return {"attn": _attn_prepare, "sample": _sample_prepare, "select": _select_prepare, "gemm": _gemm_prepare,
            "rollout": _rollout_prepare}[case["kind"]](case, seed)


def run(state):
    if hasattr(state, "ro"):
        return _rollout_run(state)
    if hasattr(state, "w"):
        return _gemm_run(state)
    return {"attn": _attn_run, "sample": _sample_run, "select": _select_run}[state.case["kind"]](state)


def work(case):
    return {"attn": _attn_work, "sample": _sample_work, "select": _select_work, "gemm": _gemm_work,
            "rollout": _rollout_work}[case["kind"]](case)


def exact(case, seed):
    f = {"attn": _attn_exact, "sample": _sample_exact, "gemm": _gemm_exact, "rollout": _rollout_exact}.get(case["kind"])
    return f(case, seed) if f else None


def tolerance(case):
    if case["kind"] == "select":
        return "exact"   # ids, flags and counts
    if case["kind"] == "sample":
        return {"rel": 1e-5, "max": 1e-3}   # tokens are the same; fp32 sums over the vocabulary
    if case["kind"] == "attn":
        return {"rel": 1e-2, "max": 0.1}    # bf16 probabilities and results
    if case["kind"] == "gemm":
        # bf16 operands with fp32 sums; the SwiGLU result is rounded to bf16
        return {"rel": 1e-2, "max": 0.05} if PROJ[case["proj"]][2] == 3 else {"rel": 1e-5, "max": 1e-3}
    if case["model"] == "tiny":
        return {"rel": 1e-4, "max": 1e-2, "differ": 0.01}
    return {"rel": 0.03, "max": 0.9, "differ": 0.01}   # bf16 layers; a near tie may route to another expert
