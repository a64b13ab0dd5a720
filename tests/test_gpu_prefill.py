"""Prefill attention (causal, over the prompt's pages) through two decoder
layers against a plain float64 decoder with the same weights: the last
position's logits depend on every position's attention in the first layer."""
import math
from types import SimpleNamespace

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda"


def _reference(mc, w, tokens, low=lambda y: y):
    """low: what the operands of the projections and of attention are rounded by."""
    b, t = tokens.shape
    hq, hkv, hd = mc.n_q_heads, mc.n_kv_heads, mc.head_dim

    def norm(x):
        return x / torch.sqrt((x * x).mean(-1, keepdim=True) + mc.rms_eps)

    inv = mc.rope_theta ** (-2.0 * torch.arange(hd // 2, device=DEV, dtype=torch.float64) / hd)
    ang = torch.arange(t, device=DEV, dtype=torch.float64)[:, None] * inv
    cos, sin = ang.cos()[:, None], ang.sin()[:, None]

    def rope(y):
        a, c = y[..., :hd // 2], y[..., hd // 2:]
        return torch.cat([a * cos - c * sin, c * cos + a * sin], -1)

    mask = torch.full((t, t), -math.inf, dtype=torch.float64, device=DEV).triu(1)
    x = w[0].double()[tokens]
    for l in range(mc.n_layers):
        wq, wk, wv, wo, wg, wu, wd = [z.double() for z in w[2 + 7 * l: 9 + 7 * l]]
        h = low(norm(x))
        q, k = low(rope((h @ wq.T).view(b, t, hq, hd))), low(rope((h @ wk.T).view(b, t, hkv, hd)))
        v = low((h @ wv.T).view(b, t, hkv, hd))
        o = torch.empty(b, t, hq, hd, dtype=torch.float64, device=DEV)
        for i in range(b):
            for head in range(hq):
                kh = head // (hq // hkv)
                s = q[i, :, head] @ k[i, :, kh].T / math.sqrt(hd) + mask
                o[i, :, head] = torch.softmax(s, -1) @ v[i, :, kh]
        x = x + o.view(b, t, hq * hd) @ wo.T
        h = norm(x)
        x = x + (torch.nn.functional.silu(h @ wg.T) * (h @ wu.T)) @ wd.T
    return norm(x)[:, -1] @ w[1].double().T


@pytest.mark.parametrize("hq,hkv,hd,length", [
    (12, 4, 64, 16),      # one page, three heads per kv head
    (6, 2, 128, 48),      # less than one 64-key stage
    (24, 8, 32, 80),      # a second stage of one page
    (16, 1, 64, 208),     # sixteen heads per kv head
    (4, 4, 128, 320),     # one head per kv head
    (8, 1, 128, 64),      # exactly one stage
    (8, 2, 128, 4176),    # more stages than lanes hold page ids
])
def test_prefill_logits(hq, hkv, hd, length):
    print(f"prefill hq={hq} hkv={hkv} hd={hd} len={length}", flush=True)
    from paper_2605_30859_amd import binding as B
    B.load_library()
    mc = SimpleNamespace(n_layers=2, d_model=256, n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, ffn_dim=256, vocab=512,
                         n_experts=0, top_k=0, expert_ffn=0, rope_theta=1e4, rms_eps=1e-6, dtype="bf16", weight_seed=0)
    rc = SimpleNamespace(n_prompts=2, prompt_len=length, m=4, k=2, cap=8, L=1, m_up=None, kv_pool_gb=0.0,
                         sample_seed=1, temperature=1.0)
    g = torch.Generator(device=DEV).manual_seed(hq * 1000 + length)
    d, q, kv = 256, hq * hd, hkv * hd

    def mk(fan, *shape):
        return torch.empty(*shape, device=DEV).uniform_(-1, 1, generator=g).mul_(math.sqrt(3.0 / fan)).bfloat16()

    w = [mk(1, 512, d), mk(d, 512, d)]
    for _ in range(2):
        # queries and keys three times wider: scores of a few units, not near 0
        w += [mk(d / 3, q, d), mk(d / 3, kv, d), mk(d, kv, d), mk(q, d, q), mk(d, 256, d), mk(d, 256, d), mk(256, d, 256)]
    ro = B.Rollout(mc, rc, weights=w, flags=B.FLAG_PERMUTE_PAGES, page_perm_seed=3)
    prompts = torch.randint(0, 512, (2, length), device=DEV, generator=g, dtype=torch.int32)
    ro.debug_fill_kv(0xff)      # nothing that the prefill has not written is used
    ro.darts_prefill(prompts.view(-1), torch.full((8,), 100, dtype=torch.int32, device=DEV))
    got = ro.debug_logits(2).double()
    ro.close()
    ref = _reference(mc, w, prompts.long())
    err = float((got - ref).abs().max() / ref.abs().max())
    print(f"  max error over max|z|: {err:.2e}", flush=True)
    assert err <= 2e-2          # the project's bound for bf16 logits


@pytest.mark.parametrize("experts,prompts", [(8, 130), (40, 28)])
def test_moe_large_batch_lists_match_small_batches(experts, prompts):
    """The routed pairs of a prefill above 16384 pairs are counted and placed by
    several blocks, those of its halves by one.  With top-k equal to the number
    of experts no routing can differ, so the same prompts give the same logits
    within the bound for bf16 logits (GEMM plans depend on the batch)."""
    print(f"moe lists E={experts} prompts={prompts}", flush=True)
    from paper_2605_30859_amd import binding as B
    B.load_library()
    assert prompts // 2 * 16 * experts <= 16384 < prompts * 16 * experts
    g = torch.Generator(device=DEV).manual_seed(experts)
    d, q, kv, fe = 256, 256, 128, 256

    def mk(fan, *shape):
        return torch.empty(*shape, device=DEV).uniform_(-1, 1, generator=g).mul_(math.sqrt(3.0 / fan)).bfloat16()

    w = [mk(1, 512, d), mk(d, 512, d), mk(d, q, d), mk(d, kv, d), mk(d, kv, d), mk(q, d, q), mk(d, experts, d),
         mk(d, experts, fe, d), mk(d, experts, fe, d), mk(fe, experts, d, fe)]
    mc = SimpleNamespace(n_layers=1, d_model=d, n_q_heads=4, n_kv_heads=2, head_dim=64, ffn_dim=0, vocab=512,
                         n_experts=experts, top_k=experts, expert_ffn=fe, rope_theta=1e4, rms_eps=1e-6, dtype="bf16",
                         weight_seed=0)
    tokens = torch.randint(0, 512, (prompts, 16), device=DEV, generator=g, dtype=torch.int32)

    def logits(part):
        rc = SimpleNamespace(n_prompts=part.shape[0], prompt_len=16, m=2, k=2, cap=8, L=1, m_up=None, kv_pool_gb=0.0,
                             sample_seed=1, temperature=1.0)
        ro = B.Rollout(mc, rc, weights=w)
        ro.darts_prefill(part.contiguous().view(-1),
                         torch.full((2 * part.shape[0],), 100, dtype=torch.int32, device=DEV))
        out = ro.debug_logits(part.shape[0]).double()
        ro.close()
        return out

    whole = logits(tokens)
    halves = torch.cat([logits(tokens[:prompts // 2]), logits(tokens[prompts // 2:])])
    err = float((whole - halves).abs().max() / halves.abs().max())
    print(f"  max difference over max|z|: {err:.2e}", flush=True)
    assert err <= 2e-2


def _scored_model(hq, hkv, hd, seed):
    """Two layers over 256 dims whose first one scores a key by dim 1 of its
    token's embedding: dim 0 is 1 in every token and feeds the queries' slowest
    rotation pair, dim 1 feeds the keys'.  Dim 2 is 0 in every token."""
    d, q, kv = 256, hq * hd, hkv * hd
    mc = SimpleNamespace(n_layers=2, d_model=d, n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, ffn_dim=256, vocab=512,
                         n_experts=0, top_k=0, expert_ffn=0, rope_theta=1e4, rms_eps=1e-6, dtype="bf16", weight_seed=0)
    g = torch.Generator(device=DEV).manual_seed(seed)

    def mk(fan, *shape):
        return torch.empty(*shape, device=DEV).uniform_(-1, 1, generator=g).mul_(math.sqrt(3.0 / fan)).bfloat16()

    w = [mk(1, 512, d), mk(d, 512, d)]
    for _ in range(2):
        w += [mk(d, q, d), mk(d, kv, d), mk(d, kv, d), mk(q, d, q), mk(d, 256, d), mk(d, 256, d), mk(256, d, 256)]
    w[0][:, 0], w[0][:, 1:3] = 1.0, 0.0
    slow = hd // 2 - 1
    for x in (w[2], w[3]):                    # wq, wk of the first layer
        x.view(-1, hd, d)[:, slow] = 0.0
        x.view(-1, hd, d)[:, hd - 1] = 0.0
    w[2].view(hq, hd, d)[:, slow, 0] = 24.0
    w[3].view(hkv, hd, d)[:, slow, 1] = 24.0
    return mc, w


def _prefill_logits(mc, w, prompts):
    from paper_2605_30859_amd import binding as B
    B.load_library()
    n, length = prompts.shape
    rc = SimpleNamespace(n_prompts=n, prompt_len=length, m=4, k=2, cap=8, L=1, m_up=None, kv_pool_gb=0.0,
                         sample_seed=1, temperature=1.0)
    ro = B.Rollout(mc, rc, weights=w)
    ro.darts_prefill(prompts.int().contiguous().view(-1), torch.full((4 * n,), 100, dtype=torch.int32, device=DEV))
    out = ro.debug_logits(n).double()
    ro.close()
    return out


@pytest.mark.parametrize("hq,hkv,hd", [(4, 2, 64), (8, 2, 32), (2, 1, 128)])
@pytest.mark.parametrize("order", ["rising", "falling", "saw"])
def test_prefill_scores_that_move_the_maximum(hq, hkv, hd, order):
    """Scores spread over hundreds of units, so that the running maximum moves far
    in every stage of 64 keys, never again after the first keys, or in every
    other stage."""
    print(f"prefill maximum hd={hd} {order}", flush=True)
    mc, w = _scored_model(hq, hkv, hd, hd)
    w[0][:, 1] = torch.arange(512, device=DEV) / 128.0
    ids = torch.arange(512, device=DEV)
    if order == "falling":
        ids = ids.flip(0)
    elif order == "saw":
        ids = ids.view(8, 64)[[1, 0, 3, 2, 5, 4, 7, 6]].reshape(-1)
    prompts = torch.stack([ids, ids.roll(7)])
    got = _prefill_logits(mc, w, prompts)
    ref = _reference(mc, w, prompts, low=lambda y: y.bfloat16().double())
    err = float((got - ref).abs().max() / ref.abs().max())
    print(f"  max error over max|z|: {err:.2e}", flush=True)
    assert err <= 2e-2          # the project's bound for bf16 logits


@pytest.mark.parametrize("hq,hd", [(4, 64), (2, 128)])
def test_prefill_attention_error(hq, hd):
    """The last position's attention alone: no FFN, identity output projection and
    LM head.  What is left of the error against float64 (with rounded q, k, v) are
    two roundings of the result to bf16 and that of the weights, of which the
    largest is 1 and exact.  A rounding of log-uniform values has the relative
    rms ulp / sqrt(12) * sqrt((1 - 1/4) / (2 ln 2)), ulp = 2^-7; 16384 results make
    the rms of their errors known within 0.6%, and 1% is allowed."""
    print(f"prefill attention error hd={hd}", flush=True)
    d, n, length = 256, 64, 2048
    rnd = 2.0 ** -7 / math.sqrt(12.0) * math.sqrt(0.75 / (2.0 * math.log(2.0)))
    g = torch.Generator(device=DEV).manual_seed(length + hd)
    mc = SimpleNamespace(n_layers=1, d_model=d, n_q_heads=hq, n_kv_heads=1, head_dim=hd, ffn_dim=256, vocab=512,
                         n_experts=0, top_k=0, expert_ffn=0, rope_theta=1e4, rms_eps=1e-6, dtype="bf16", weight_seed=0)

    def mk(scale, *shape):
        return torch.empty(*shape, device=DEV).uniform_(-1, 1, generator=g).mul_(scale * math.sqrt(3.0)).bfloat16()

    eye = torch.eye(d, device=DEV)
    off = torch.zeros(256, d, device=DEV)
    w = [mk(0.125, 512, d), torch.cat([eye, off]).bfloat16(), mk(math.sqrt(3.0 / d), d, d),
         mk(math.sqrt(3.0 / d), hd, d), mk(4.0, hd, d), eye.bfloat16(), off.bfloat16(), off.bfloat16(), off.bfloat16()]
    prompts = torch.randint(0, 512, (n, length), device=DEV, generator=g)
    got = _prefill_logits(mc, w, prompts)[:, :d]

    low = lambda y: y.bfloat16().double()  # noqa: E731
    h = w[0].double()[prompts]
    h = low(h / torch.sqrt((h * h).mean(-1, keepdim=True) + mc.rms_eps))
    ang = torch.arange(length, device=DEV, dtype=torch.float64)[:, None, None] * (
        mc.rope_theta ** (-2.0 * torch.arange(hd // 2, device=DEV, dtype=torch.float64) / hd))

    def rope(y, a):
        y, z = y[..., :hd // 2], y[..., hd // 2:]
        return low(torch.cat([y * a.cos() - z * a.sin(), z * a.cos() + y * a.sin()], -1))

    q = rope((h[:, -1] @ w[2].double().T).view(n, hq, hd), ang[-1])
    k = rope((h @ w[3].double().T).view(n, length, 1, hd), ang)[:, :, 0]
    v = low(h @ w[4].double().T)
    p = torch.softmax((q[:, :, None] * k[:, None]).sum(-1) / math.sqrt(hd), -1)
    o = (p[..., None] * v[:, None]).sum(2)
    out = w[0].double()[prompts[:, -1]] + o.reshape(n, d)
    rest = p.scatter(-1, p.argmax(-1, keepdim=True), 0.0)
    weights = (rest[..., None] * (v[:, None] - o[:, :, None])).square().sum(2).reshape(n, d)
    size = out.square().mean(-1, keepdim=True).sqrt()
    err = float((got - out / size).norm() / math.sqrt(n * d))
    due = rnd * math.sqrt(float(((2.0 * out.square() + weights) / size.square()).mean()))
    print(f"  rms error {err:.3e}, due {due:.3e}", flush=True)
    assert err <= 1.01 * due


@pytest.mark.parametrize("hq,hkv,hd", [(4, 2, 64), (2, 1, 128)])
@pytest.mark.parametrize("value", ["-inf", "inf", "nan"])
def test_prefill_infinities_and_nan(hq, hkv, hd, value):
    """A token whose keys overflow: a score of -infinity is a weight of 0, as in
    float64, where it is merely very low; infinity and NaN make NaN of what
    attends to it, and of no other prompt."""
    print(f"prefill hd={hd} {value}", flush=True)
    mc, w = _scored_model(hq, hkv, hd, 100 + hd)
    odd = 300
    prompts = torch.randint(0, odd, (2, 208), device=DEV, generator=torch.Generator(device=DEV).manual_seed(hd))
    plain = _prefill_logits(mc, w, prompts)
    if value == "nan":
        w[0][odd, 2] = float("nan")
    else:
        w[0][odd, 2] = 8.0
        w[3].view(hkv, hd, 256)[:, hd // 2 - 1, 2] = -3e38 if value == "-inf" else 3e38
    hit = prompts.clone()
    hit[0, [1, 2, 63, 64, 100]] = odd
    got = _prefill_logits(mc, w, hit)
    assert bool((got[1] == plain[1]).all())
    if value == "-inf":
        ref = _reference(mc, w, hit)
        err = float((got - ref).abs().max() / ref.abs().max())
        print(f"  max error over max|z|: {err:.2e}", flush=True)
        assert err <= 2e-2
    else:
        assert bool(got[0].isnan().all())


def _moe_prefill(w, d, experts, tokens):
    mc = SimpleNamespace(n_layers=1, d_model=d, n_q_heads=2, n_kv_heads=1, head_dim=128, ffn_dim=0, vocab=512,
                         n_experts=experts, top_k=experts, expert_ffn=256, rope_theta=1e4, rms_eps=1e-6, dtype="bf16",
                         weight_seed=0)
    return _prefill_logits(mc, w, tokens)


def _moe_weights(d, experts, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)

    def mk(fan, *shape):
        return torch.empty(*shape, device=DEV).uniform_(-1, 1, generator=g).mul_(math.sqrt(3.0 / fan)).bfloat16()

    return [mk(1, 512, d), mk(d, 512, d), mk(d, 256, d), mk(d, 128, d), mk(d, 128, d), mk(256, d, 256),
            mk(d, experts, d), mk(d, experts, 256, d), mk(d, experts, 256, d), mk(256, experts, d, 256)], g


@pytest.mark.parametrize("prompts", [7, 8, 17])
def test_moe_large_tiles_partly_full(prompts):
    """256-row expert tiles with 112, 128 and 272 rows per expert (every expert
    takes every row) against the same prompts in batches of the smaller tiles."""
    print(f"moe partly full tiles, {16 * prompts} rows per expert", flush=True)
    w, g = _moe_weights(256, 8, prompts)
    tokens = torch.randint(0, 512, (prompts, 16), device=DEV, generator=g, dtype=torch.int32)
    whole = _moe_prefill(w, 256, 8, tokens)
    parts = torch.cat([_moe_prefill(w, 256, 8, t) for t in tokens.split(4)])
    err = float((whole - parts).abs().max() / parts.abs().max())
    print(f"  max difference over max|z|: {err:.2e}", flush=True)
    assert err <= 2e-2          # the project's bound for bf16 logits


def test_moe_rows_gathered_beyond_4_gib():
    """A prefill whose expert rows are gathered from 4.3 GB, beyond the 32-bit
    offsets of the 256-row tiles (the 128-row ring takes it), against its halves."""
    print("moe gather beyond 4 GiB", flush=True)
    w, g = _moe_weights(5120, 2, 5)
    tokens = torch.randint(0, 512, (3280, 128), device=DEV, generator=g, dtype=torch.int32)
    assert tokens.numel() * 5120 * 2 >= 2 ** 32 > tokens.numel() * 5120
    whole = _moe_prefill(w, 5120, 2, tokens)
    halves = torch.cat([_moe_prefill(w, 5120, 2, t) for t in tokens.split(1640)])
    err = float((whole - halves).abs().max() / halves.abs().max())
    print(f"  max difference over max|z|: {err:.2e}", flush=True)
    assert err <= 2e-2          # the project's bound for bf16 logits
