"""Prefill attention (causal, over the prompt's pages) through two decoder
layers against a plain float64 decoder with the same weights: the last
position's logits depend on every position's attention in the first layer."""
import math
from types import SimpleNamespace

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda"


def _reference(mc, w, tokens):
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
        h = norm(x)
        q, k = rope((h @ wq.T).view(b, t, hq, hd)), rope((h @ wk.T).view(b, t, hkv, hd))
        v = (h @ wv.T).view(b, t, hkv, hd)
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
