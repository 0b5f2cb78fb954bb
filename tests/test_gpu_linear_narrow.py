"""Layers of few 32x64 tiles (k_linear_narrow) against the oracle at the edges of its tiles and K chunks, and
against the 128x128 tiles the dispatch takes for larger ones."""
import numpy as np
import pytest
import torch

from oracle import dit as odit
from paper_2607_04461_amd import flashbon as F
from paper_2607_04461_amd import synth
from tests._util import rel_l2

pytestmark = pytest.mark.gpu


def _run(M, N, K, epi):
    A = synth.round_to_bf16(synth.random_matrix((M, K), 501))
    W = synth.round_to_bf16(synth.random_matrix((N, K), 502, 0.05))
    bias, gate, h0 = synth.random_matrix((N,), 503), synth.random_matrix((N,), 504), synth.random_matrix((M, N), 505)
    dev = lambda x, t=torch.float32: torch.from_numpy(x).cuda().to(t)  # noqa: E731
    dA, dW, db = dev(A, torch.bfloat16), dev(W, torch.bfloat16), dev(bias)
    ref = odit.linear(A.astype(np.float64), W, bias)
    if epi == "residual":
        out, src, cache = torch.full((M, N), 3.0, device="cuda"), dev(h0), torch.full((M, N), 7.0, device="cuda")
        F.flashbon_op_linear_residual(F.BF16, M, N, K, dA, dW, db, dev(gate), src, out)
        inplace = dev(h0)
        F.flashbon_op_linear(F.BF16, M, N, K, dA, dW, db, F.EPI_RESIDUAL, inplace, dev(gate), cache)
        torch.cuda.synchronize()
        assert torch.equal(out, inplace) and torch.equal(cache, inplace) and torch.equal(src, dev(h0))
        ref, tol = h0 + gate * ref, 2e-6
    elif epi == "store_f32":
        out, tol = torch.empty((M, N), device="cuda"), 2e-6
        F.flashbon_op_linear(F.BF16, M, N, K, dA, dW, db, F.EPI_STORE_F32, out)
    else:   # one rounding to bf16
        out, tol = torch.empty((M, N), device="cuda", dtype=torch.bfloat16), 6e-3
        F.flashbon_op_linear(F.BF16, M, N, K, dA, dW, db, F.EPI_GELU if epi == "gelu" else F.EPI_STORE, out)
        ref = odit.gelu_tanh(ref) if epi == "gelu" else ref
    torch.cuda.synchronize()
    assert rel_l2(out.float().cpu().numpy().astype(np.float64), ref) <= tol


@pytest.mark.parametrize("M,N,K", [(1, 4, 32), (31, 60, 64), (33, 68, 96), (32, 64, 512), (64, 128, 1088), (130, 260, 160),
                                   (7, 8, 1536)])
@pytest.mark.parametrize("epi", ["store", "gelu", "store_f32", "residual"])
def test_narrow(M, N, K, epi, monkeypatch):
    """One row and column quad; rows and columns beside the tile; fewer and more K chunks than waves, half chunks."""
    monkeypatch.delenv("FLASHBON_LINEAR_TILE", raising=False)
    assert F.flashbon_op_linear_plan(F.BF16, M, N, K, 0)[1].startswith("k_linear_narrow")
    _run(M, N, K, epi)


@pytest.mark.parametrize("M,N,K", [(40, 24, 72), (9, 12, 8)])
def test_narrow_forced_on_k_tails(M, N, K, monkeypatch):
    monkeypatch.setenv("FLASHBON_LINEAR_TILE", "narrow")
    _run(M, N, K, "store_f32")
