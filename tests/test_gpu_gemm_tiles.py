"""The projection GEMMs at the edges of their tiles, through one decoder block.

rk_reference_forward of a two-layer model leaves the input of block 1, which is
the output of block 0: the four projections with their epilogues (rotary,
residual, SwiGLU).  Reference: the same block in float64 with plain torch
operations, from the same bf16 weights.

Tolerance: the block rounds x, q|k|v, the attention output, the second x and the
feed-forward activations to bf16 (relative 2^-9 each, uniform, so rms 2^-9 /
sqrt(3) = 1.1e-3); five such roundings in a row give a relative 2-norm of about
sqrt(5) * 1.1e-3 = 2.5e-3 of the block's update, and a single element stays within
five standard deviations of a few times that.  A misplaced tile, row or k-step is
an error of the update's own size.  Weights have variance 1 / columns: a score s = q . k
/ sqrt(d_h) of two rounded rows is off by about sqrt(2) * 1.1e-3 |s|, which the softmax
passes on as a relative error of a weight, so |s| has to stay near 1 for it to count
as one of the roundings (at a fixed 0.05 the scores of d = 2048 have a standard
deviation of 5, and the update was off by 1.0e-2).
"""
from __future__ import annotations

import math

import pytest

pytestmark = pytest.mark.gpu


class Shape:
    def __init__(self, d, heads, kv_heads, head_dim, d_ff, vocab=128):
        self.n_layers, self.d_model, self.n_heads, self.n_kv_heads = 2, d, heads, kv_heads
        self.head_dim, self.d_ff, self.vocab = head_dim, d_ff, vocab
        self.rope_theta, self.rms_eps, self.dtype = 1.0e4, 1.0e-5, "bf16"


def block(m, w, h, lengths):
    """One decoder block in float64."""
    import torch
    f = lambda k: w[k][0].double()

    def norm(x, g):
        return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + m.rms_eps) * g

    qc, kc = m.n_heads * m.head_dim, m.n_kv_heads * m.head_dim
    y = norm(h, f("attn_norm")) @ f("w_qkv").t()
    half = m.head_dim // 2
    pos = torch.cat([torch.arange(t, device=h.device) for t in lengths]).double()
    freq = m.rope_theta ** (-torch.arange(half, device=h.device).double() * 2 / m.head_dim)
    c, s = torch.cos(pos[:, None, None] * freq), torch.sin(pos[:, None, None] * freq)

    def rope(x):
        x = x.view(x.shape[0], -1, m.head_dim)
        a, b = x[..., :half], x[..., half:]
        return torch.cat([a * c - b * s, b * c + a * s], -1)

    q, k, v = rope(y[:, :qc]), rope(y[:, qc:qc + kc]), y[:, qc + kc:].reshape(len(h), -1, m.head_dim)
    out, o, grp = torch.empty_like(q), 0, m.n_heads // m.n_kv_heads
    for t in lengths:
        mask = torch.ones(t, t, device=h.device, dtype=torch.bool).triu(1)
        for g in range(m.n_heads):
            sc = (q[o:o + t, g] @ k[o:o + t, g // grp].t()) / math.sqrt(m.head_dim)
            out[o:o + t, g] = torch.softmax(sc.masked_fill(mask, -math.inf), -1) @ v[o:o + t, g // grp]
        o += t
    h = h + out.reshape(len(h), -1) @ f("w_o").t()
    gu = norm(h, f("mlp_norm")) @ f("w_gate_up").t()
    return h + (torch.nn.functional.silu(gu[:, :m.d_ff]) * gu[:, m.d_ff:]) @ f("w_down").t()


def check_block(m, lengths, tol=7.5e-3, big=0.06):
    import torch
    import paper_2608_08684_amd as rk
    g = torch.Generator(device="cuda").manual_seed(5)
    dtype = torch.float32 if m.dtype == "f32" else torch.bfloat16
    mat = lambda r, c, s=None: torch.empty(r, c, device="cuda", dtype=dtype).normal_(
        0, s or c ** -0.5, generator=g)
    gain = lambda: 1.0 + 0.2 * torch.randn(m.d_model, device="cuda", generator=g)
    qkv, att = (m.n_heads + 2 * m.n_kv_heads) * m.head_dim, m.n_heads * m.head_dim
    L = range(m.n_layers)
    w = {"tok_emb": mat(m.vocab, m.d_model, 1.0), "lm_head": mat(m.vocab, m.d_model), "final_norm": gain(),
         "w_qkv": [mat(qkv, m.d_model) for _ in L], "w_o": [mat(m.d_model, att) for _ in L],
         "w_gate_up": [mat(2 * m.d_ff, m.d_model) for _ in L], "w_down": [mat(m.d_model, m.d_ff) for _ in L],
         "attn_norm": [gain() for _ in L], "mlp_norm": [gain() for _ in L]}
    offs = [0]
    for t in lengths:
        offs.append(offs[-1] + t)
    rows = offs[-1]
    tok = torch.randint(0, m.vocab, (rows,), device="cuda", generator=g, dtype=torch.int32)
    model, batch = rk.Model(m, w), rk.Batch(tok, offs)
    # the buffers' tails hold NaN: padding rows that reach a result show
    state = torch.full((model.clean_state_size(rows),), 0xFF, dtype=torch.uint8, device="cuda")
    ws = torch.full((model.workspace_size(rows, 1, 0),), 0xFF, dtype=torch.uint8, device="cuda")
    model.reference_forward(batch, state, ws)
    torch.cuda.synchronize()
    h = state[:m.n_layers * rows * m.d_model * 4].view(torch.float32).view(m.n_layers, rows, m.d_model)
    h0 = w["tok_emb"][tok.long()].double()
    assert torch.equal(h[0].double(), h0)
    want = block(m, w, h0, lengths) - h0
    got = h[1].double() - h0
    rel = ((got - want).norm() / want.norm()).item()
    worst = ((got - want).abs().max() / want.square().mean().sqrt()).item()
    print(f"rows {rows}: update off by {rel:.2e} (2-norm), {worst:.2e} of its rms at most")
    assert rel < tol and worst < big


# large M: the 8-wave tiles, with one, two, three and four k-steps and ragged last tile rows
@pytest.mark.parametrize("m, lengths", [
    (Shape(256, 4, 4, 64, 64), [512] * 63 + [300]),
    (Shape(256, 2, 2, 128, 128), [512] * 63 + [511]),
    (Shape(256, 4, 2, 64, 192), [512] * 64),
    (Shape(768, 12, 12, 64, 384), [512] * 22 + [257]),    # 192-wide residual tiles
    (Shape(512, 4, 1, 128, 320), [700] * 23 + [1]),
], ids=["k64", "k128", "k192", "n192", "k320"])
def test_large_tiles(m, lengths):
    check_block(m, lengths)


# few rows: the ring tiles, K from one k-step past the deepest ring, single rows and ragged tiles
@pytest.mark.parametrize("m, lengths", [
    (Shape(256, 4, 4, 64, 64), [1]),
    (Shape(256, 2, 2, 128, 192), [33, 1]),
    (Shape(384, 6, 2, 64, 320), [31, 33, 64]),
    (Shape(512, 4, 4, 128, 576), [200, 57]),
    (Shape(768, 12, 12, 64, 704), [509]),
    (Shape(1024, 8, 2, 128, 1088), [300, 1, 99]),
    (Shape(768, 12, 12, 64, 3072), [700, 1300]),
    (Shape(2048, 16, 8, 128, 640), [900, 101]),
    (Shape(128, 2, 1, 64, 8192), [17]),                    # long K, 16-wide tiles
    (Shape(512, 8, 2, 64, 8256), [32, 1]),
    (Shape(1024, 8, 2, 128, 1088), [17]),                  # 32-wide tiles with every epilogue
    (Shape(1024, 16, 4, 64, 2048), [64] * 17),             # a ring tile's last round partly filled
], ids=["1row", "34", "k320", "k576", "509", "400", "2000", "wide", "k8192", "k8256", "17", "1088"])
def test_few_rows(m, lengths):
    check_block(m, lengths)


def test_rows_do_not_depend_on_the_batch():
    """A sequence's block output is bitwise the same alone and among many rows (other tiles)."""
    import torch
    import paper_2608_08684_amd as rk
    m = Shape(768, 12, 4, 64, 1536)
    g = torch.Generator(device="cuda").manual_seed(6)
    mat = lambda r, c, s=0.05: torch.empty(r, c, device="cuda", dtype=torch.bfloat16).normal_(0, s, generator=g)
    one = torch.ones(m.d_model, device="cuda")
    w = {"tok_emb": mat(m.vocab, 768, 1.0), "lm_head": mat(m.vocab, 768), "final_norm": one}
    for k, shape in (("w_qkv", (1280, 768)), ("w_o", (768, 768)), ("w_gate_up", (3072, 768)), ("w_down", (768, 1536))):
        w[k] = [mat(*shape) for _ in range(2)]
    w["attn_norm"] = w["mlp_norm"] = [one, one]
    model = rk.Model(m, w)
    tok = torch.randint(0, m.vocab, (40,), device="cuda", generator=g, dtype=torch.int32)
    got = []
    for copies in (1, 4, 16, 60):
        batch = rk.Batch(tok.repeat(copies), [40 * i for i in range(copies + 1)])
        state = torch.empty(model.clean_state_size(batch.rows), dtype=torch.uint8, device="cuda")
        ws = torch.empty(model.workspace_size(batch.rows, 1, 0), dtype=torch.uint8, device="cuda")
        model.reference_forward(batch, state, ws)
        h = state[:2 * batch.rows * 768 * 4].view(torch.float32).view(2, batch.rows, 768)
        got.append(h[1, -40:].clone())
    for x in got[1:]:
        assert torch.equal(x, got[0])


@pytest.mark.parametrize("d, vocab, windows", [
    (1024, 16384, [8] * 5),      # 64x128 tiles for both sets of rows, 32x64 for one sequence alone
    (256, 16384, [9, 1, 30]),    # 64x64
    (128, 65536, [25] * 8),      # an 8-wave tile, in a launch for each set
])
def test_two_sets_of_logits(d, vocab, windows):
    """Clean and pass logits of one launch: with every cache whole they are the same rows, so the KL is exactly 0, and
    a sequence's logits are bitwise those that it has alone."""
    import torch
    import paper_2608_08684_amd as rk
    m = Shape(d, 4, 1, 64, 192, vocab=vocab)
    g = torch.Generator(device="cuda").manual_seed(8)
    mat = lambda r, c: torch.empty(r, c, device="cuda", dtype=torch.bfloat16).normal_(0, c ** -0.5, generator=g)
    one = torch.ones(d, device="cuda")
    w = {"tok_emb": mat(vocab, d), "lm_head": mat(vocab, d), "final_norm": one, "attn_norm": [one] * 2,
         "mlp_norm": [one] * 2, "w_qkv": [mat(384, d) for _ in range(2)], "w_o": [mat(d, 256) for _ in range(2)],
         "w_gate_up": [mat(384, d) for _ in range(2)], "w_down": [mat(d, 192) for _ in range(2)]}
    model, P = rk.Model(m, w), 33
    toks = [torch.randint(0, vocab, (P + t,), device="cuda", generator=g, dtype=torch.int32) for t in windows]
    none = torch.zeros(1, dtype=torch.int32, device="cuda")

    def logits(toks):
        offs = [0]
        for t in toks:
            offs.append(offs[-1] + len(t))
        batch, n = rk.Batch(torch.cat(toks), offs), len(toks)
        flags = rk.RK_FLAG_CACHED_WINDOW | rk.RK_FLAG_UNFUSED_KL
        state = torch.full((model.window_state_size(offs[-1]),), 0xFF, dtype=torch.uint8, device="cuda")
        ws = torch.full((model.workspace_size(offs[-1], 1, flags),), 0xFF, dtype=torch.uint8, device="cuda")
        model.window_reference(batch, P, state, ws)
        rows = offs[-1] - n * P
        out, kl = torch.empty(n, device="cuda"), torch.full((rows,), -1.0, device="cuda")
        lg = torch.empty(rows, vocab, device="cuda")
        model.policy_damage(batch, P, none, [0, 0], 1, [0, 0], state, out, ws, kl_pos=kl, logits_out=lg)
        torch.cuda.synchronize()
        assert torch.equal(kl, torch.zeros_like(kl))
        return lg

    both, r = logits(toks), 0
    for t in toks:
        assert torch.equal(both[r:r + len(t) - P], logits([t]))
        r += len(t) - P


# fp32: the same block on the fp32 tiles and the fp32 attention, head dims 32, 64 and 128, one row to several
# 32-query blocks, many and few tiles.  fp32 sums of up to 1000 terms in chunks of 32: about sqrt(64) * 6e-8 = 5e-7
# relative per product of the block, a few of them in a row
@pytest.mark.parametrize("m, lengths", [
    (Shape(128, 4, 2, 32, 64), [1, 31, 32, 33, 1]),
    (Shape(256, 4, 4, 64, 192), [256, 129, 3]),
    (Shape(384, 4, 1, 128, 320), [100, 161]),
    (Shape(512, 16, 4, 32, 1024), [900, 1200, 77]),
    (Shape(1024, 16, 16, 64, 704), [1500, 333]),
], ids=["hd32", "hd64", "hd128", "hd32-many", "hd64-many"])
def test_fp32_block(m, lengths):
    m.dtype = "f32"
    check_block(m, lengths, tol=2e-6, big=2e-5)


# the clean log-sum-exp: 128- and 256-wide column blocks, ragged rows, and a vocabulary whose pairs do not fit the
# scratch of a narrow model at once (several launches).  Logits are fp32 sums of d bf16 products (|x| |w| near 1 each, so
# off by about 1e-6); log-sum-exp passes that on and rounds once to fp32 (|lse| up to 12: 5e-7)
@pytest.mark.parametrize("d, vocab, lengths", [(256, 384, [1]), (256, 512, [300, 7]), (128, 128128, [513]),
                                               (128, 81920, [40, 1000])])
def test_clean_log_sum_exp(d, vocab, lengths):
    import torch
    import paper_2608_08684_amd as rk
    m = Shape(d, 2, 1, 64, 64, vocab=vocab)
    g = torch.Generator(device="cuda").manual_seed(7)
    mat = lambda r, c: torch.empty(r, c, device="cuda", dtype=torch.bfloat16).normal_(0, c ** -0.5, generator=g)
    one = torch.ones(d, device="cuda")
    w = {"tok_emb": mat(vocab, d), "lm_head": mat(vocab, d), "final_norm": one, "attn_norm": [one] * 2,
         "mlp_norm": [one] * 2, "w_qkv": [mat(256, d)] * 2, "w_o": [mat(d, 128)] * 2, "w_gate_up": [mat(128, d)] * 2,
         "w_down": [mat(d, 64)] * 2}
    offs = [0]
    for t in lengths:
        offs.append(offs[-1] + t)
    rows = offs[-1]
    model = rk.Model(m, w)
    batch = rk.Batch(torch.randint(0, vocab, (rows,), device="cuda", generator=g, dtype=torch.int32), offs)
    state = torch.full((model.clean_state_size(rows),), 0xFF, dtype=torch.uint8, device="cuda")
    ws = torch.full((model.workspace_size(rows, 1, 0),), 0xFF, dtype=torch.uint8, device="cuda")
    model.reference_forward(batch, state, ws)
    up = lambda n: (n + 255) // 256 * 256
    x0 = up(2 * rows * d * 4)
    l0 = x0 + up(up(rows) * d * 2)
    x = state[x0:x0 + rows * d * 2].view(torch.bfloat16).view(rows, d).double()
    lse = state[l0:l0 + rows * 4].view(torch.float32).double()
    want = torch.logsumexp(x @ w["lm_head"].double().t(), dim=1)
    err = (lse - want).abs().max().item()
    print(f"d {d} vocab {vocab} rows {rows}: log-sum-exp off by {err:.2e}")
    assert err < 1e-5


# Logits far from zero (up to +-1032, exact in fp32: signed sums of powers of two and of multiples of 1/16, from
# embeddings of +-1 through blocks whose output weights are zero).  e^(x - max) of such logits is formed from the exact
# difference, so the log-sum-exp is off by its rounding to fp32 and by the rounding of the terms (exp2 1 ulp, 256 terms per
# column block: a few 1e-7), whatever the size of the maximum; scaled before the subtraction, the maximum alone would put
# it off by up to 4e-5
def test_clean_log_sum_exp_of_large_logits():
    import numpy as np
    import torch
    import paper_2608_08684_amd as rk
    d, vocab, rows = 256, 512, 300
    m = Shape(d, 2, 1, 64, 64, vocab=vocab)
    g = torch.Generator(device="cuda").manual_seed(11)
    mat = lambda r, c: torch.empty(r, c, device="cuda", dtype=torch.bfloat16).normal_(0, c ** -0.5, generator=g)
    zero = lambda r, c: torch.zeros(r, c, device="cuda", dtype=torch.bfloat16)
    one = torch.ones(d, device="cuda")
    gain = torch.cat([2.0 ** torch.arange(9, 1, -1), torch.randint(0, 128, (d - 8,)) / 16.0]).float().cuda()
    sign = lambda *shape: (torch.randint(0, 2, shape, device="cuda", generator=g) * 2 - 1).to(torch.bfloat16)
    head = zero(vocab, d)
    head[:, :8] = 1.0
    head[torch.arange(vocab), 8 + torch.arange(vocab) % (d - 8)] = 1.0
    w = {"tok_emb": sign(vocab, d), "lm_head": head, "final_norm": gain, "attn_norm": [one] * 2, "mlp_norm": [one] * 2,
         "w_qkv": [mat(256, d)] * 2, "w_o": [zero(d, 128)] * 2, "w_gate_up": [mat(128, d)] * 2, "w_down": [zero(d, 64)] * 2}
    model = rk.Model(m, w)
    tok = torch.randperm(vocab, device="cuda", generator=g)[:rows].to(torch.int32)
    batch = rk.Batch(tok, [0, rows])
    state = torch.full((model.clean_state_size(rows),), 0xFF, dtype=torch.uint8, device="cuda")
    ws = torch.full((model.workspace_size(rows, 1, 0),), 0xFF, dtype=torch.uint8, device="cuda")
    model.reference_forward(batch, state, ws)
    up = lambda n: (n + 255) // 256 * 256
    x0 = up(2 * rows * d * 4)
    l0 = x0 + up(up(rows) * d * 2)
    x = state[x0:x0 + rows * d * 2].view(torch.bfloat16).view(rows, d).double()
    assert torch.equal(x, w["tok_emb"][tok.long()].double() * gain.double())
    lse = state[l0:l0 + rows * 4].view(torch.float32).double().cpu().numpy()
    want = torch.logsumexp(x @ head.double().t(), dim=1).cpu().numpy()
    err = np.abs(lse - want)
    assert np.abs(want).max() > 500
    print(f"log-sum-exp up to {np.abs(want).max():.0f}: off by {err.max():.2e}")
    assert (err <= 0.5 * np.spacing(np.abs(want).astype(np.float32)) + 2e-6).all()
