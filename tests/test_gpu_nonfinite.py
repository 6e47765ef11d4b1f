"""fp32 attention with a non-finite row: the rows before it do not see it.

A token whose embedding is NaN makes its own row's Keys and Values NaN.  Causal attention
passes them to that row and to later rows of its sequence only, so the rows before it,
also those whose query block holds it, keep bit for bit the values they have with an
ordinary token in its place.
"""
from __future__ import annotations

import pytest

pytestmark = pytest.mark.gpu


class Shape:
    n_layers, d_model, d_ff, vocab, rope_theta, rms_eps, dtype = 2, 256, 64, 128, 1.0e4, 1.0e-5, "f32"

    def __init__(self, heads, kv_heads, head_dim):
        self.n_heads, self.n_kv_heads, self.head_dim = heads, kv_heads, head_dim


@pytest.mark.parametrize("heads, kv_heads, dh", [(8, 4, 32), (4, 2, 64), (4, 1, 128)])
@pytest.mark.parametrize("T, at", [(70, 50), (33, 32), (32, 31), (200, 97), (5, 0)])
def test_rows_before_a_nan_row(heads, kv_heads, dh, T, at):
    import torch
    import paper_2608_08684_amd as rk
    m = Shape(heads, kv_heads, dh)
    d, bad = m.d_model, m.vocab - 1
    g = torch.Generator(device="cuda").manual_seed(5)
    mat = lambda r, c: torch.empty(r, c, device="cuda").normal_(0, c ** -0.5, generator=g)
    one = torch.ones(d, device="cuda")
    w = {"tok_emb": mat(m.vocab, d), "lm_head": mat(m.vocab, d), "final_norm": one, "attn_norm": [one] * 2,
         "mlp_norm": [one] * 2, "w_qkv": [mat((heads + 2 * kv_heads) * dh, d)] * 2, "w_o": [mat(d, heads * dh)] * 2,
         "w_gate_up": [mat(2 * m.d_ff, d)] * 2, "w_down": [mat(d, m.d_ff)] * 2}
    w["tok_emb"][bad] = float("nan")
    model = rk.Model(m, w)
    other = 41   # a second sequence, untouched
    tok = torch.randint(0, bad, (T + other,), device="cuda", generator=g, dtype=torch.int32)

    def block_output(tokens):
        batch = rk.Batch(tokens, [0, T, T + other])
        state = torch.full((model.clean_state_size(batch.rows),), 0xFF, dtype=torch.uint8, device="cuda")
        ws = torch.full((model.workspace_size(batch.rows, 1, 0),), 0xFF, dtype=torch.uint8, device="cuda")
        model.reference_forward(batch, state, ws)
        torch.cuda.synchronize()
        return state[:2 * batch.rows * d * 4].view(torch.float32).view(2, batch.rows, d)[1].clone()

    want = block_output(tok)
    tok[at] = bad
    got = block_output(tok)
    assert torch.isfinite(want).all()
    assert torch.isnan(got[at:T]).all()
    assert torch.equal(got[:at], want[:at])
    assert torch.equal(got[T:], want[T:])
