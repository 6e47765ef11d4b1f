"""SnapKV scoring and selection over many chunks, with budgets on the edges of the digit search.

Sequences over many 256-key chunks (just below, on and above their edges), four and
eight combinations of query heads and 32-query blocks, both head sizes, kept counts
from one position over the window to half the sequence.  Votes against float64 with plain torch
operations from the same bf16 caches: a vote is a sum of probabilities exp2(s - c) with s
an fp32 sum of d_h products (|s| up to about 20, off by up to 20 * d_h^0.5 * 6e-8 = 1.4e-5
relative after exp2).  Positions, Keys and Values must be those that the returned
votes select.
"""
from __future__ import annotations

import math

import pytest

pytestmark = pytest.mark.gpu


class Cfg:
    def __init__(self, heads, kv_heads, head_dim):
        self.n_layers, self.d_model, self.n_heads, self.n_kv_heads, self.head_dim = 2, 128, heads, kv_heads, head_dim
        self.d_ff, self.vocab, self.rope_theta, self.rms_eps, self.dtype = 64, 128, 1.0e4, 1.0e-5, "bf16"


@pytest.mark.parametrize("heads, kv_heads, dh, lens, w, kernel, average", [
    (32, 8, 128, [2047 + 64, 2048 + 64, 2049 + 64, 300], 64, 7, False),
    (16, 4, 128, [4400, 33, 256 + 16], 16, 5, True),
    (8, 8, 64, [4096 + 32, 2080], 32, 7, False),
    (8, 1, 64, [2600, 90], 32, 13, True),
])
def test_scores_and_selection(heads, kv_heads, dh, lens, w, kernel, average):
    import torch
    import paper_2608_08684_amd as rk
    m = Cfg(heads, kv_heads, dh)
    L, grp, n = m.n_layers, heads // kv_heads, len(lens)
    one = torch.zeros(128, device="cuda")
    weights = {k: one for k in ("tok_emb", "lm_head", "final_norm")}
    weights.update({k: [one] * L for k in ("w_qkv", "w_o", "w_gate_up", "w_down", "attn_norm", "mlp_norm")})
    model = rk.Model(m, weights)   # the selection reads the shape only
    offs = [0]
    for t in lens:
        offs.append(offs[-1] + t)
    R = offs[-1]
    g = torch.Generator(device="cuda").manual_seed(9)
    kv = torch.empty(L, R, 2 * kv_heads * dh, dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    q = torch.empty(L, n * w, heads * dh, dtype=torch.bfloat16, device="cuda").normal_(0, 2.5 / math.sqrt(dh), generator=g)
    batch = rk.Batch(torch.zeros(R, dtype=torch.int32, device="cuda"), offs)
    state = torch.zeros(model.snapkv_state_size(R, n, w), dtype=torch.uint8, device="cuda")
    kvb = kv.numel() * 2
    state[:kvb].copy_(kv.view(torch.uint8).reshape(-1))
    q0 = (kvb + 255) // 256 * 256
    state[q0:q0 + q.numel() * 2].copy_(q.view(torch.uint8).reshape(-1))
    budgets = [[min(t, w + 1 + (i + 3) * (l + 7)) if l else t // 2 for l in range(L)] for i, t in enumerate(lens)]
    total, lay = rk.snapkv_layout(batch, L, budgets)
    pos = torch.empty(kv_heads * total, dtype=torch.int32, device="cuda")
    ko, vo = (torch.empty(kv_heads * total, dh, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    sc = torch.empty(L, kv_heads, R - n * w, device="cuda")
    ws = torch.full((model.snapkv_workspace_size(R, n, w),), 0xFF, dtype=torch.uint8, device="cuda")
    model.snapkv_compress(batch, budgets, state, pos, ko, vo, ws, obs_window=w, pool_kernel=kernel,
                          pooling=rk.RK_POOL_AVG if average else rk.RK_POOL_MAX, scores=sc)
    torch.cuda.synchronize()
    r, worst = kernel // 2, 0.0
    for l in range(L):
        for i, T in enumerate(lens):
            for h in range(kv_heads):
                k = kv[l, offs[i]:offs[i + 1], h * dh:(h + 1) * dh]
                qq = q[l, i * w:(i + 1) * w].view(w, heads, dh)[:, h * grp:(h + 1) * grp].double()
                s = (qq.reshape(-1, dh) @ k.double().t()).view(w, grp, T) * math.log(2.0)
                hide = torch.arange(T, device="cuda")[None] > torch.arange(T - w, T, device="cuda")[:, None]
                p = torch.softmax(s.masked_fill(hide[:, None], -math.inf), -1).sum((0, 1))[:T - w]
                pad = torch.full((r,), 0.0 if average else -math.inf, dtype=torch.float64, device="cuda")
                win = torch.cat([pad, p, pad]).unfold(0, kernel, 1)
                want = win.sum(1) / kernel if average else win.max(1).values
                got = sc[l, h, offs[i] - i * w:offs[i + 1] - (i + 1) * w]
                worst = max(worst, ((got - want).abs() / want).max().item())
                keep = int(lay[i * L + l + 1] - lay[i * L + l])
                e = int(lay[i * L + l]) * kv_heads + h * keep
                top = torch.sort(got, descending=True, stable=True).indices[:keep - w]
                sel = torch.cat([top.sort().values, torch.arange(T - w, T, device="cuda")])
                assert torch.equal(pos[e:e + keep].long(), sel), (l, i, h)
                assert torch.equal(ko[e:e + keep], k[sel])
                v = kv[l, offs[i]:offs[i + 1], (kv_heads + h) * dh:(kv_heads + h + 1) * dh]
                assert torch.equal(vo[e:e + keep], v[sel])
    print(f"votes off by {worst:.2e} at most")
    assert worst < 3e-5


@pytest.mark.parametrize("heads, kv_heads, dh, lens, w, layers", [
    (8, 8, 64, [4096 + 32, 700], 32, 8),        # 17 and 3 chunks: 1280 workgroups of one, so two per workgroup
    (8, 2, 128, [8192 + 256 + 1, 513], 32, 16),   # a chunk of one key; 1184
])
def test_votes_of_chunk_pairs(heads, kv_heads, dh, lens, w, layers):
    """Two chunks per workgroup (all layers in one call) and one (a model of a single layer) vote bitwise the same."""
    import torch
    import paper_2608_08684_amd as rk
    n, R = len(lens), sum(lens)
    offs = [sum(lens[:i]) for i in range(n + 1)]
    g = torch.Generator(device="cuda").manual_seed(5)
    kv = torch.empty(layers, R, 2 * kv_heads * dh, dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    q = torch.empty(layers, n * w, heads * dh, dtype=torch.bfloat16, device="cuda").normal_(
        0, 2.5 / math.sqrt(dh), generator=g)
    batch = rk.Batch(torch.zeros(R, dtype=torch.int32, device="cuda"), offs)

    def votes(kv, q):
        m = Cfg(heads, kv_heads, dh)
        m.n_layers = L = kv.shape[0]
        one = torch.zeros(128, device="cuda")
        weights = {k: one for k in ("tok_emb", "lm_head", "final_norm")}
        weights.update({k: [one] * L for k in ("w_qkv", "w_o", "w_gate_up", "w_down", "attn_norm", "mlp_norm")})
        model = rk.Model(m, weights)
        state = torch.zeros(model.snapkv_state_size(R, n, w), dtype=torch.uint8, device="cuda")
        kvb = kv.numel() * 2
        state[:kvb].copy_(kv.contiguous().view(torch.uint8).reshape(-1))
        q0 = (kvb + 255) // 256 * 256
        state[q0:q0 + q.numel() * 2].copy_(q.contiguous().view(torch.uint8).reshape(-1))
        budgets = [[w + 1] * L] * n
        total, _ = rk.snapkv_layout(batch, L, budgets)
        pos = torch.empty(kv_heads * total, dtype=torch.int32, device="cuda")
        ko, vo = (torch.empty(kv_heads * total, dh, dtype=torch.bfloat16, device="cuda") for _ in range(2))
        sc = torch.empty(L, kv_heads, R - n * w, device="cuda")
        ws = torch.full((model.snapkv_workspace_size(R, n, w),), 0xFF, dtype=torch.uint8, device="cuda")
        model.snapkv_compress(batch, budgets, state, pos, ko, vo, ws, obs_window=w, pool_kernel=1,
                              pooling=rk.RK_POOL_MAX, scores=sc)
        torch.cuda.synchronize()
        return sc

    both = votes(kv, q)
    for l in range(layers):
        assert torch.equal(both[l], votes(kv[l:l + 1], q[l:l + 1])[0]), l
