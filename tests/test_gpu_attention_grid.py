"""Very many short queries: more workgroups of k_attn_f32 than a launch takes (2^32 threads in x), which
k_attn_valu's three-dimensional grid does take."""
import pytest
import torch

from paper_2607_04461_amd import flashbon as F

pytestmark = pytest.mark.gpu


def test_many_single_queries():
    batch, heads, dh, tk = 65535, 257, 8, 3      # 2^24 + 65279 (batch row, head) pairs of one query
    D = heads * dh
    g = torch.Generator(device="cuda").manual_seed(3)
    q = torch.randn(batch, D, generator=g, device="cuda")
    k, v = torch.randn(tk, D, generator=g, device="cuda"), torch.randn(tk, D, generator=g, device="cuda")
    out = torch.zeros(batch, D, device="cuda")
    F.flashbon_op_attention(F.FP32, batch, heads, dh, 1, tk, q, D, D, k, v, 0, D, None, 0, out, D, D)
    torch.cuda.synchronize()
    for h in range(0, heads, 16):                # 16 heads of 8 are 128 columns
        c = slice(h * dh, (h + 1) * dh)
        s = (q[:, None, c].double() * k[None, :, c].double()).sum(-1) * dh ** -0.5
        ref = (torch.softmax(s, 1)[:, :, None] * v[None, :, c].double()).sum(1)
        assert float((out[:, c].double() - ref).norm() / ref.norm()) <= 4 * (dh + tk) ** 0.5 * 2.0 ** -24
