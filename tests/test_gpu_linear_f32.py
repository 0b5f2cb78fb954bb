"""fp32 linear layers: every kernel of the fp32 dispatch against a 64-bit product, at the edges of its tiles."""
import numpy as np
import pytest
import torch

from oracle import dit as odit
from paper_2607_04461_amd import flashbon as F
from paper_2607_04461_amd import synth
from tests._util import rel_l2

pytestmark = pytest.mark.gpu

# Error of K products summed in fp32 against 64 bits: each addition rounds by at most 2^-24 of the running
# sum, whose size grows as a random walk, so about sqrt(K) 2^-24 of the result; 4 of these plus the epilogue's
# few roundings bound every order of summation (measured: 0.2 to 1 of sqrt(K) 2^-24).
def _tol(K):
    return (4.0 * np.sqrt(K) + 8.0) * 2.0 ** -24


def _dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, np.float32)).cuda()


def _run(M, N, K, epi, offset=0):
    """One layer; every buffer `offset` floats past a 256-byte boundary."""
    def place(x):
        buf = torch.zeros(x.size + 64, device="cuda")
        v = buf[offset:offset + x.size].view(x.shape)
        v.copy_(_dev(x))
        return v

    A, W = synth.random_matrix((M, K), 301), synth.random_matrix((N, K), 302, 0.05)
    bias, gate = synth.random_matrix((N,), 303), synth.random_matrix((N,), 304)
    h0, c0 = synth.random_matrix((M, N), 305), synth.random_matrix((M, N), 306)
    dA, dW, db = place(A), place(W), place(bias)
    ref = odit.linear(A.astype(np.float64), W, bias)
    if epi == "residual":
        out, cache = place(h0), place(c0)
        F.flashbon_op_linear(F.FP32, M, N, K, dA, dW, db, F.EPI_RESIDUAL, out, place(gate), cache)
        torch.cuda.synchronize()
        assert torch.equal(cache, out)
        ref = h0 + gate * ref
    else:
        out = place(h0)
        F.flashbon_op_linear(F.FP32, M, N, K, dA, dW, db, F.EPI_GELU if epi == "gelu" else F.EPI_STORE, out)
        ref = odit.gelu_tanh(ref) if epi == "gelu" else ref
    torch.cuda.synchronize()
    assert rel_l2(out.cpu().numpy().astype(np.float64), ref) <= _tol(K)
    return out


# one row and column quad, K below a tile, K tails of 8, 16 and 24, edges on and beside the tiles of 16, 32 and 64
SHAPES = [(1, 4, 8), (3, 12, 24), (32, 32, 32), (33, 36, 40), (64, 64, 64), (65, 68, 72), (100, 64, 64),
          (31, 132, 96), (130, 260, 200), (257, 64, 1536)]


@pytest.mark.parametrize("tile", ["valu", "dot", "32x32", "64x64"])
@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("epi", ["store", "gelu", "residual"])
def test_each_kernel(tile, M, N, K, epi, monkeypatch):
    monkeypatch.setenv("FLASHBON_LINEAR_TILE", "f32:" + tile)
    _run(M, N, K, epi)


@pytest.mark.parametrize("M,N,K", [(33, 36, 40), (130, 260, 200)])
@pytest.mark.parametrize("epi", ["store", "residual"])
def test_buffers_off_16_bytes(M, N, K, epi, monkeypatch):
    """Buffers on 4-byte boundaries take the vector-ALU kernel, whatever the size."""
    monkeypatch.delenv("FLASHBON_LINEAR_TILE", raising=False)
    off = _run(M, N, K, epi, offset=1)
    monkeypatch.setenv("FLASHBON_LINEAR_TILE", "f32:valu")
    assert torch.equal(off, _run(M, N, K, epi))


@pytest.mark.parametrize("K", [8960, 65536])
def test_long_sums(K, monkeypatch):
    monkeypatch.delenv("FLASHBON_LINEAR_TILE", raising=False)
    _run(70, 72, K, "store")
