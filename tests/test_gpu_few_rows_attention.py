"""Attention of few window rows behind a cached prefix: a sequence's result does not depend on its neighbours.

A sequence whose window rows times the query heads per KV head fit one 32-column block takes the few-row kernel,
whatever the other windows of the batch are: alone (retained positions read in place) and beside a second sequence with
a 40-row window (which takes the general kernel, behind gathered caches) its logits are bitwise the same.
"""
from __future__ import annotations

import pytest

pytestmark = pytest.mark.gpu


class Cfg:
    def __init__(self, heads, kv_heads, head_dim):
        self.n_layers, self.n_heads, self.n_kv_heads, self.head_dim = 2, heads, kv_heads, head_dim
        self.d_model, self.d_ff, self.vocab = 256, 256, 512
        self.rope_theta, self.rms_eps, self.dtype = 1.0e4, 1.0e-5, "bf16"


def make_model(m):
    import torch
    import paper_2608_08684_amd as rk
    g = torch.Generator(device="cuda").manual_seed(3)
    mat = lambda r, c: torch.empty(r, c, device="cuda", dtype=torch.bfloat16).normal_(0, c ** -0.5, generator=g)
    one = torch.ones(m.d_model, device="cuda")
    H, Hkv, dh, L = m.n_heads, m.n_kv_heads, m.head_dim, m.n_layers
    w = {"tok_emb": mat(m.vocab, 256), "lm_head": mat(m.vocab, 256), "final_norm": one, "attn_norm": [one] * L,
         "mlp_norm": [one] * L, "w_qkv": [mat((H + 2 * Hkv) * dh, 256) for _ in range(L)],
         "w_o": [mat(256, H * dh) for _ in range(L)], "w_gate_up": [mat(512, 256) for _ in range(L)],
         "w_down": [mat(256, 256) for _ in range(L)]}
    return rk.Model(m, w), g


@pytest.mark.parametrize("heads, kv_heads, dh, P, W, keep", [
    (8, 2, 128, 33, 1, [1, 0]),            # one key kept; the whole prefix
    (8, 2, 128, 300, 8, [31, 32]),         # all 32 columns used
    (8, 2, 128, 257, 5, [33, 257]),        # every position kept
    (4, 4, 64, 129, 32, [127, 128]),       # no query groups, 32 rows
    (4, 1, 64, 700, 3, [129, 0]),
    (8, 1, 128, 5000, 2, [4097, 4096]),    # more and as many positions as the block's table holds
])
def test_few_rows(heads, kv_heads, dh, P, W, keep):
    import torch
    import paper_2608_08684_amd as rk
    m = Cfg(heads, kv_heads, dh)
    model, g = make_model(m)
    tok = torch.randint(0, m.vocab, (2 * P + W + 40,), device="cuda", generator=g, dtype=torch.int32)
    stride = max(1, kv_heads * sum(keep))
    pos = torch.stack([torch.cat([torch.stack([torch.randperm(P, device="cuda", generator=g)[:k].sort().values
                                               for _ in range(kv_heads)]).reshape(-1) for k in keep if k])
                       for _ in range(2)]).to(torch.int32).contiguous()
    assert pos.shape[1] == stride
    offs = [0, kv_heads * keep[0]]

    def logits(lens):
        n, o = len(lens), [0]
        for t in lens:
            o.append(o[-1] + t)
        batch = rk.Batch(tok, o)
        state = torch.full((model.window_state_size(o[-1]),), 0xFF, dtype=torch.uint8, device="cuda")
        ws = torch.full((model.workspace_size(o[-1], 1, rk.RK_FLAG_CACHED_WINDOW | rk.RK_FLAG_UNFUSED_KL),), 0xFF,
                        dtype=torch.uint8, device="cuda")
        model.window_reference(batch, P, state, ws)
        rows = o[-1] - n * P
        d = torch.empty(n, device="cuda")
        kl = torch.empty(rows, device="cuda")
        lg = torch.empty(rows, m.vocab, device="cuda")
        model.policy_damage(batch, P, pos, offs, stride, keep, state, d, ws, kl_pos=kl, logits_out=lg)
        torch.cuda.synchronize()
        return lg[:W], kl[:W]

    a, _ = logits([P + W])
    b, _ = logits([P + W, P + 40])
    assert torch.equal(a, b)


@pytest.mark.parametrize("heads, kv_heads, dh, P, windows", [
    (4, 2, 64, 70, [16, 40, 3, 17]),      # two query heads per KV head: at most 16 rows take the few-row kernel
    (4, 1, 128, 129, [8, 171, 1, 9]),
    (8, 2, 128, 65, [33, 8, 4]),
])
def test_profile_does_not_depend_on_the_other_sequences(heads, kv_heads, dh, P, windows):
    """A cached-window profile over logits in memory (each row's KL is one workgroup's): all sequences in one batch and
    each in a batch of its own are bitwise the same."""
    import torch
    import paper_2608_08684_amd as rk
    m = Cfg(heads, kv_heads, dh)
    model, g = make_model(m)
    offs = [0]
    for t in windows:
        offs.append(offs[-1] + P + t)
    batch = rk.Batch(torch.randint(0, m.vocab, (offs[-1],), device="cuda", generator=g, dtype=torch.int32), offs)
    flags = rk.RK_FLAG_CACHED_WINDOW | rk.RK_FLAG_UNFUSED_KL

    def profile(max_rows):
        ws = torch.full((model.workspace_size(max_rows, 2, flags | rk.RK_WS_CLEAN_STATE),), 0xFF, dtype=torch.uint8,
                        device="cuda")
        s = torch.empty(1, 2, device="cuda")
        d = torch.empty(1, len(windows), 2, device="cuda")
        model.sensitivity_profile(batch, [0, 1], [0.1], s, ws, max_rows, 2, d_out=d, window_start=P, flags=flags)
        torch.cuda.synchronize()
        return d

    assert torch.equal(profile(batch.rows), profile(P + max(windows)))
