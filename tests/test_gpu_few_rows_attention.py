"""Attention of few window rows behind a cached prefix: a sequence's result does not depend on its neighbours.

A sequence whose window rows times the query heads per KV head fit one 32-column block takes the few-row kernel,
whatever the other windows of the batch are: alone (retained positions read in place) and beside a second sequence with
a 40-row window (which takes the general kernel, behind gathered caches) its logits are bitwise the same.  The logits
are also compared with float64, and short windows behind perturbed prefix Values with the oracle.
"""
from __future__ import annotations

import numpy as np
import pytest

import fixtures as F
from oracle import model as OM
from oracle import profile as OPR

from gpu_helpers import f32_weights, log, make_batch
from test_gpu_parity import assert_kl_close
from test_gpu_window import WindowRunner

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
    return rk.Model(m, w), g, w


FEW = [
    (8, 2, 128, 33, 1, [1, 0]),            # one key kept; the whole prefix
    (8, 2, 128, 300, 8, [31, 32]),         # all 32 columns used
    (8, 2, 128, 257, 5, [33, 257]),        # every position kept
    (4, 4, 64, 129, 32, [127, 128]),       # no query groups, 32 rows
    (4, 1, 64, 700, 3, [129, 0]),
    (8, 1, 128, 5000, 2, [4097, 4096]),    # more and as many positions as the block's table holds
]


@pytest.mark.parametrize("heads, kv_heads, dh, P, W, keep", FEW)
def test_few_rows(heads, kv_heads, dh, P, W, keep):
    import torch
    import paper_2608_08684_amd as rk
    m = Cfg(heads, kv_heads, dh)
    model, g, _ = make_model(m)
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
    model, g, _ = make_model(m)
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


@pytest.mark.parametrize("heads, kv_heads, dh, P, W, keep", FEW)
def test_few_rows_against_float64(heads, kv_heads, dh, P, W, keep):
    """Two sequences' window logits over the retained positions, from the library's own bf16 caches.

    The first and last retained position and one at the end of a 32-key block have 64-fold Values, and so have all
    positions that are not retained: a lost key, or one too many, is far outside the bound.  Bound: 13 tensors are
    rounded to bf16 on the way (x, q|k|v, attention, x, SwiGLU and the softmax weights of two layers, the final
    norm), 2^-9 / sqrt(3) of their size each: 4.1e-3 in 2-norm where they add up as independent, and three times that.
    """
    import torch
    import paper_2608_08684_amd as rk
    m = Cfg(heads, kv_heads, dh)
    model, g, w = make_model(m)
    n, L, grp, V64 = 2, m.n_layers, heads // kv_heads, torch.float64
    tok = torch.randint(0, m.vocab, (n * (P + W),), device="cuda", generator=g, dtype=torch.int32)
    batch = rk.Batch(tok, [0, P + W, 2 * (P + W)])
    state = torch.full((model.window_state_size(batch.rows),), 0xFF, dtype=torch.uint8, device="cuda")
    ws = torch.full((model.workspace_size(batch.rows, 1, rk.RK_FLAG_CACHED_WINDOW | rk.RK_FLAG_UNFUSED_KL),), 0xFF,
                    dtype=torch.uint8, device="cuda")
    model.window_reference(batch, P, state, ws)
    kv = state[:L * n * P * 2 * kv_heads * dh * 2].view(torch.bfloat16).view(L, n, P, 2, kv_heads, dh)
    sel = [[[torch.randperm(P, device="cuda", generator=g)[:k].sort().values if k else torch.arange(P, device="cuda")
             for _ in range(kv_heads)] for k in keep] for _ in range(n)]
    for i in range(n):
        for l in range(L):
            for h, s in enumerate(sel[i][l]):
                gain = torch.full((P,), 64.0, device="cuda")
                gain[s] = 1.0
                gain[s[[0, -1, max(0, (len(s) - 1) // 32 * 32 - 1)]]] = 64.0
                kv[l, i, :, 1, h] *= gain[:, None].bfloat16()
    pos = torch.stack([torch.cat([torch.cat(sel[i][l]) for l in range(L) if keep[l]]) for i in range(n)])
    pos = pos.to(torch.int32).contiguous()
    d, kl = torch.empty(n, device="cuda"), torch.empty(n * W, device="cuda")
    lg = torch.empty(n * W, m.vocab, device="cuda")
    model.policy_damage(batch, P, pos, [0, kv_heads * keep[0]], pos.shape[1], keep, state, d, ws, kl_pos=kl,
                        logits_out=lg)
    torch.cuda.synchronize()

    half = dh // 2
    freq = m.rope_theta ** (-torch.arange(half, dtype=V64, device="cuda") * 2 / dh)

    def rope(x):   # rows P .. P + W - 1 of [W, heads, dh]
        a = torch.arange(P, P + W, dtype=V64, device="cuda")[:, None, None] * freq
        lo, hi = x[..., :half], x[..., half:]
        return torch.cat([lo * a.cos() - hi * a.sin(), hi * a.cos() + lo * a.sin()], -1)

    norm = lambda h: h * torch.rsqrt(h.square().mean(-1, keepdim=True) + m.rms_eps)
    W64 = lambda name, l: w[name][l].double()
    want = []
    for i in range(n):
        h = w["tok_emb"].double()[tok[i * (P + W) + P:(i + 1) * (P + W)].long()]
        for l in range(L):
            x = (norm(h) @ W64("w_qkv", l).t()).view(W, heads + 2 * kv_heads, dh)
            q, k, v = rope(x[:, :heads]), rope(x[:, heads:heads + kv_heads]), x[:, heads + kv_heads:]
            out = []
            for hq in range(heads):
                hk = hq // grp
                K = torch.cat([kv[l, i, sel[i][l][hk], 0, hk].double(), k[:, hk]])
                Vv = torch.cat([kv[l, i, sel[i][l][hk], 1, hk].double(), v[:, hk]])
                s = q[:, hq] @ K.t() / dh ** 0.5
                s[:, -W:].masked_fill_(torch.ones(W, W, device="cuda").triu(1).bool(), -torch.inf)
                out.append(torch.softmax(s, -1) @ Vv)
            h = h + torch.cat(out, -1) @ W64("w_o", l).t()
            gate, up = (norm(h) @ W64("w_gate_up", l).t()).split(m.d_ff, -1)
            h = h + (torch.nn.functional.silu(gate) * up) @ W64("w_down", l).t()
        want.append(norm(h) @ w["lm_head"].double().t())
    want = torch.cat(want)
    err = ((lg - want).norm() / want.norm()).item()
    log(f"few rows against float64: {heads}/{kv_heads} x {dh}, P {P}, keep {keep}: {err:.2e}")
    assert err < 1.25e-2


@pytest.mark.parametrize("heads, kv_heads, dh, P, windows", [
    (4, 2, 64, 70, [16, 3, 9]),       # two query heads per KV head: at most 16 rows
    (2, 2, 64, 95, [32, 17]),         # one: at most 32
    (4, 1, 128, 129, [8, 1, 5]),
    (4, 1, 128, 65, [8, 33, 2]),      # the second one takes the general kernel
])
def test_perturbed_prefix_values(heads, kv_heads, dh, P, windows):
    """Short ragged windows behind perturbed prefix Values: rk_profile_layer against the oracle (tolerances as in the
    other cached-window tests), rk_sensitivity_profile with several joined passes bitwise as one at a time."""
    import paper_2608_08684_amd as rk
    cfg = F.small_model(n_layers=3, d_model=256, n_heads=heads, n_kv_heads=kv_heads, head_dim=dh, d_ff=384, vocab=640,
                        rope_theta=1.0e4, dtype="bf16")
    lens = [P + t for t in windows]
    W = F.make_weights(cfg)
    run = WindowRunner(cfg, W)
    m = OM.Model(cfg, f32_weights(cfg, W), np.float64)
    toks = F.make_tokens(F.make_workload("w", cfg, lens, seed_id=19))
    batch = make_batch(toks)
    state = run.window_state(batch, P)
    ref = [OPR.window_clean_state(m, t, P) for t in toks]
    woff = np.concatenate([[0], np.cumsum(windows)])
    p = OPR.PerturbParams(0.2, window_start=P, protect_head=2, protect_tail=3)
    for l in range(cfg.n_layers):
        d, _, lg = run.window_layer(batch, state, l, p.alpha, P, want_logits=True, protect_head=2, protect_tail=3)
        want = []
        for k in range(len(toks)):
            err = np.abs(lg[woff[k]:woff[k + 1]] - OM.logits(m, OPR.window_perturbed_final(m, ref[k], k, l, p))).max()
            log(f"short windows {heads}/{kv_heads} x {dh} layer {l} seq {k}: logits max abs err {err:.3e}")
            assert err <= 2e-2
            want.append(OPR.window_profile_layer(m, ref[k], k, l, p)[0])
        assert_kl_close(d, want, f"layer {l} window d")
    layers, flags = list(range(cfg.n_layers)), rk.RK_FLAG_CACHED_WINDOW | rk.RK_FLAG_UNFUSED_KL
    args = dict(max_group=6, window_start=P, protect_head=2, protect_tail=3, flags=flags)
    _, one = run.profile(batch, layers, [0.2, 0.1], max_rows=batch.rows, **args)
    for joined in (2, 3, 4):
        _, d = run.profile(batch, layers, [0.2, 0.1], max_rows=joined * batch.rows, **args)
        np.testing.assert_array_equal(d, one)
