"""Layers whose K ranges one workgroup takes in turn (a split that would bring less than a quarter more workgroups)
against the split launch with its reduction: the same number of ranges and the same bits."""
import pytest
import torch

from paper_2607_04461_amd import flashbon as F

pytestmark = pytest.mark.gpu


# tiles of 128 x 128, 160 x 128 and 128 x 256 with ragged rows and columns; 2 ranges of 16 and of 25 and 24 K tiles
@pytest.mark.parametrize("M,N,K", [(1601, 2056, 2048), (3000, 1536, 3136), (150, 27000, 2048)])
@pytest.mark.parametrize("epi", ["store", "gelu", "store_f32", "residual"])
def test_ranges_in_turn(M, N, K, epi, monkeypatch):
    g = torch.Generator(device="cuda").manual_seed(M)
    randn = lambda *s: torch.randn(s, generator=g, device="cuda")  # noqa: E731
    a, w, bias, gate, h = randn(M, K).bfloat16(), (0.02 * randn(N, K)).bfloat16(), randn(N), randn(N), randn(M, N)
    ws = torch.empty(48 << 20, dtype=torch.uint8, device="cuda")
    code = {"store": F.EPI_STORE, "gelu": F.EPI_GELU, "store_f32": F.EPI_STORE_F32, "residual": F.EPI_RESIDUAL}[epi]
    outs, cache = [], []
    for plan in (None, "128:256:3:2"):
        if plan:
            monkeypatch.setenv("FLASHBON_SPLITK", plan)
        else:
            monkeypatch.delenv("FLASHBON_SPLITK", raising=False)
        ws.fill_(0x7F)
        out = h.clone() if epi == "residual" else torch.empty(
            M, N, device="cuda", dtype=torch.float32 if epi == "store_f32" else torch.bfloat16)
        copy = torch.zeros(M, N, device="cuda") if epi == "residual" else None
        assert F.flashbon_op_linear_ws(F.BF16, M, N, K, a, w, bias, code, out, ws, gate=gate if copy is not None else None,
                                       cache_out=copy) == 2
        torch.cuda.synchronize()
        untouched = bool((ws == 0x7F).all())
        assert untouched == (plan is None)   # the split launch keeps its partial sums there
        outs.append(out)
        cache.append(copy)
    assert torch.equal(outs[0], outs[1])
    if epi == "residual":
        assert torch.equal(cache[0], outs[0]) and torch.equal(cache[1], outs[0])
        ref = h.double() + gate.double() * (a.double() @ w.double().T + bias.double())
        assert float((outs[0].double() - ref).norm() / ref.norm()) <= 2e-6
