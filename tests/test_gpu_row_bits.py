"""The bits of a row (of a layer) and of a candidate (of a pool) do not depend on how many rows or candidates share
the launch: every kernel that a rule on the row count may choose sums in one order."""
import dataclasses

import pytest
import torch

from paper_2607_04461_amd import flashbon as F
from paper_2607_04461_amd import synth
from paper_2607_04461_amd.pool import DraftPool

pytestmark = pytest.mark.gpu

CODE = {"bf16": F.BF16, "fp32": F.FP32}
ACT = {"bf16": torch.bfloat16, "fp32": torch.float32}
TILES = {"bf16": ["narrow", "128x128", "256x256"], "fp32": ["f32:64x64", "f32:32x32", "f32:dot", "f32:valu"]}


def _operands(dtype, M, N, K):
    g = torch.Generator(device="cuda").manual_seed(M + 3 * N + 7 * K)
    randn = lambda *s: torch.randn(s, generator=g, device="cuda")  # noqa: E731
    return (randn(M, K).to(ACT[dtype]), (0.05 * randn(N, K)).to(ACT[dtype]), randn(N), randn(N), randn(M, N))


def _layer(dtype, a, w, bias, gate, h, epi):
    """The layer on all rows of a; epi: an epilogue, or "plain" for a residual without bias and gate."""
    M, N, K = a.shape[0], w.shape[0], a.shape[1]
    if epi in ("residual", "plain"):
        out = torch.empty(M, N, device="cuda")
        full = epi == "residual"
        F.flashbon_op_linear_residual(CODE[dtype], M, N, K, a, w, bias if full else None, gate if full else None, h, out)
    else:
        code = {"store": F.EPI_STORE, "gelu": F.EPI_GELU, "store_f32": F.EPI_STORE_F32}[epi]
        out = torch.empty(M, N, device="cuda", dtype=torch.float32 if epi == "store_f32" else ACT[dtype])
        F.flashbon_op_linear(CODE[dtype], M, N, K, a, w, bias, code, out)
    torch.cuda.synchronize()
    return out


# rows and columns beside the tiles; one K tile, halves of one, tails of 8 and 24, and more tiles than the rings hold
@pytest.mark.parametrize("M,N,K", [(1, 4, 64), (33, 68, 96), (40, 24, 72), (65, 200, 8), (130, 72, 704), (64, 64, 1048),
                                   (70, 136, 1536)])
@pytest.mark.parametrize("dtype", list(TILES))
@pytest.mark.parametrize("epi", ["store", "gelu", "store_f32", "residual", "plain"])
def test_tiles(dtype, M, N, K, epi, monkeypatch):
    ops = _operands(dtype, M, N, K)
    outs = []
    for tile in TILES[dtype]:
        monkeypatch.setenv("FLASHBON_LINEAR_TILE", tile)
        outs.append(_layer(dtype, *ops, epi))
    for tile, o in zip(TILES[dtype], outs):
        assert torch.equal(o, outs[0]), tile


# the rows alone, as a few tiles and among enough rows for the largest tiles
@pytest.mark.parametrize("N,K", [(64, 256), (256, 704), (1536, 1536)])
@pytest.mark.parametrize("dtype", list(TILES))
@pytest.mark.parametrize("epi", ["store", "residual"])
def test_rows(dtype, N, K, epi, monkeypatch):
    monkeypatch.delenv("FLASHBON_LINEAR_TILE", raising=False)
    a, w, bias, gate, h = _operands(dtype, 9000, N, K)
    plans, outs = set(), []
    for M in (3, 40, 500, 9000):
        plans.add(F.flashbon_op_linear_plan(CODE[dtype], M, N, K, F.EPI_STORE)[1])
        outs.append(_layer(dtype, a[:M], w, bias, gate, h[:M], epi)[:3])
    assert len(plans) > 1 or (dtype == "fp32" and N < 1536)
    for o in outs[1:]:
        assert torch.equal(o, outs[0])


# layers of few tiles whose operands start off 16 bytes: half a K tile and a tail, columns in fours
@pytest.mark.parametrize("M,N,K", [(33, 68, 96), (40, 24, 72), (20, 36, 256)])
@pytest.mark.parametrize("dtype", list(TILES))
def test_operands_off_16_bytes(dtype, M, N, K, monkeypatch):
    monkeypatch.delenv("FLASHBON_LINEAR_TILE", raising=False)
    a, w, bias, gate, h = _operands(dtype, M, N, K)
    skip = 8 // a.element_size()
    off = [torch.cat([x.new_zeros(skip), x.flatten()])[skip:].view(x.shape) for x in (a, w)]
    assert all(x.data_ptr() % 16 == 8 for x in off)
    for epi in ("store", "residual"):
        assert torch.equal(_layer(dtype, *off, bias, gate, h, epi), _layer(dtype, a, w, bias, gate, h, epi))


# one candidate alone and in pools of 2 and 7: the head (and with small widths every layer) changes its kernel, and
# 2 heads of 1369 tokens would each be split differently between the waves of a workgroup
@pytest.mark.parametrize("dtype,hidden,heads", [("bf16", 128, 1), ("bf16", 128, 2), ("bf16", 64, 4), ("fp32", 256, 2),
                                                ("fp32", 64, 4)])
@pytest.mark.parametrize("rope", [False, True])
def test_pools(dtype, hidden, heads, rope):
    shape = synth.ModelShape(num_blocks=2, hidden=hidden, heads=heads, mlp_hidden=192, freq_dim=32, text_dim=32,
                             qk_norm_rope=rope)
    flat = synth.make_weights(shape, 17)[0]
    z0 = synth.make_latents(7, shape.latent_channels, 74, 74)
    outs = []
    for n in (1, 2, 7):
        wl = dataclasses.replace(synth.WORKLOADS["tiny"], name="pool", shape=shape, n=n, n_cond=1, latent_h=74, latent_w=74,
                                 dtype=dtype)
        pool = DraftPool(wl, weights=flat)
        pool.reset(z0[:n])
        for k in range(2):
            pool.draft_step(k, [0, 0], [0, 0])
        torch.cuda.synchronize()
        outs.append((pool.latents[0].clone(), pool.cache.view(2, 3, n, -1)[:, :2, 0].clone()))
        pool.close()
    for z, cache in outs[1:]:
        assert torch.equal(z, outs[0][0]) and torch.equal(cache, outs[0][1])
