"""fp32 matrix-core attention (fp32 operands, and bf16 ones of head dims below 128) against the oracle, at the
edges of its key and query tiles, for every number of slabs a key tile is split into."""
import numpy as np
import pytest
import torch

from oracle import dit as odit
from paper_2607_04461_amd import flashbon as F
from paper_2607_04461_amd import synth
from tests._util import rel_l2

pytestmark = pytest.mark.gpu

# fp32: scores of dh products, sums over tk keys, a few exponentials, each within some 2^-24; random-walk growth
# leaves sqrt(dh + tk) of them (measured: 1e-7 at tk = 16 to 1.5e-6 at 4096).  bf16 operands: probabilities
# stay fp32, so the output's rounding (2^-9 at most, 1.7e-3 on average) is what is left.
def _tol(dtype, dh, tk):
    return 3e-3 if dtype == "bf16" else 4.0 * np.sqrt(dh + tk) * 2.0 ** -24


def _case(dtype, batch, heads, dh, tq, tk, cross, seed=401, gap=0, offset=0):
    """Device views of q, k, v and out with `gap` extra elements a row and `offset` before the first, the kv
    index, and the oracle's result."""
    act = torch.bfloat16 if dtype == "bf16" else torch.float32
    n_kv = 2 if cross else batch
    D = heads * dh

    def place(rows, x=None):
        buf = torch.zeros(offset + rows * (D + gap) + 64, device="cuda", dtype=act)
        v = torch.as_strided(buf, (rows, D), (D + gap, 1), offset)
        if x is not None:
            v.copy_(torch.from_numpy(x))
        return v

    q, k, v = (synth.random_matrix((r, D), seed + i) for i, r in enumerate((batch * tq, n_kv * tk, n_kv * tk)))
    if dtype == "bf16":
        q, k, v = (synth.round_to_bf16(x) for x in (q, k, v))
    index = np.array([(3 * b + 1) % n_kv for b in range(batch)], np.int32) if cross else None
    ref = np.concatenate([odit.multi_head_attention(q[b * tq:(b + 1) * tq].astype(np.float64),
                                                    k[c * tk:(c + 1) * tk].astype(np.float64),
                                                    v[c * tk:(c + 1) * tk].astype(np.float64), heads)
                          for b, c in enumerate(range(batch) if index is None else index)])
    return place(batch * tq, q), place(n_kv * tk, k), place(n_kv * tk, v), place(batch * tq), index, n_kv, ref


def _run(dtype, batch, heads, dh, tq, tk, cross, **kw):
    q, k, v, out, index, n_kv, ref = _case(dtype, batch, heads, dh, tq, tk, cross, **kw)
    rs = q.stride(0)
    idx = None if index is None else torch.from_numpy(index).cuda()
    F.flashbon_op_attention(F.BF16 if dtype == "bf16" else F.FP32, batch, heads, dh, tq, tk, q, tq * rs, rs, k, v,
                            tk * rs, rs, idx, n_kv, out, tq * rs, rs)
    torch.cuda.synchronize()
    assert rel_l2(out.float().cpu().numpy().astype(np.float64), ref) <= _tol(dtype, dh, tk)
    return out.clone()


@pytest.mark.parametrize("slabs", ["1", "2", "4", "valu"])
@pytest.mark.parametrize("dtype,dh", [("fp32", 8), ("fp32", 16), ("fp32", 32), ("fp32", 64), ("fp32", 128),
                                      ("bf16", 8), ("bf16", 16), ("bf16", 32), ("bf16", 64)])
@pytest.mark.parametrize("tq,tk,cross", [(1, 1, False), (31, 7, True), (33, 33, False), (64, 65, True), (129, 128, True),
                                         (40, 257, True)])
def test_each_split(slabs, dtype, dh, tq, tk, cross, monkeypatch):
    """One key, keys and queries beside the tiles of 32, 64 and 128 (of 16 and 64 for the vector-ALU kernel that takes
    the calls this one does not), slabs wholly past the last key."""
    monkeypatch.setenv("FLASHBON_ATTN_F32", slabs)
    _run(dtype, 3, 3, dh, tq, tk, cross)


@pytest.mark.parametrize("dtype,gap,offset", [("fp32", 4, 0), ("fp32", 1, 0), ("fp32", 0, 1), ("bf16", 8, 0), ("bf16", 2, 0),
                                              ("bf16", 0, 3)])
def test_strides_and_addresses(dtype, gap, offset, monkeypatch):
    """Rows further apart than a row is long; strides and addresses off 16 bytes take the vector-ALU kernel."""
    monkeypatch.delenv("FLASHBON_ATTN_F32", raising=False)
    out = _run(dtype, 2, 3, 32, 50, 70, True, gap=gap, offset=offset)
    if gap % 4 or offset:
        monkeypatch.setenv("FLASHBON_ATTN_F32", "valu")
        assert torch.equal(out, _run(dtype, 2, 3, 32, 50, 70, True, gap=gap, offset=offset))


@pytest.mark.parametrize("dtype,dh", [("fp32", 8), ("fp32", 64), ("fp32", 128), ("bf16", 16), ("bf16", 64)])
@pytest.mark.parametrize("tq,tk", [(1, 1), (65, 47), (64, 16), (70, 33)])
def test_misaligned_rows(dtype, dh, tq, tk, monkeypatch):
    """The dispatch's own choice for rows that start off 16 bytes: the vector-ALU kernel at every head dim."""
    monkeypatch.delenv("FLASHBON_ATTN_F32", raising=False)
    out = _run(dtype, 2, 3, dh, tq, tk, True, gap=2, offset=2)
    monkeypatch.setenv("FLASHBON_ATTN_F32", "valu")
    assert torch.equal(out, _run(dtype, 2, 3, dh, tq, tk, True, gap=2, offset=2))


@pytest.mark.parametrize("slabs", ["1", "2", "4"])
def test_large_scores(slabs, monkeypatch):
    """Scores of a few hundred: the running maximum moves far and often, and most probabilities underflow."""
    monkeypatch.setenv("FLASHBON_ATTN_F32", slabs)
    q, k, v, out, _, _, _ = _case("fp32", 1, 2, 64, 200, 200, False, seed=431)
    q.mul_(30.0)
    F.flashbon_op_attention(F.FP32, 1, 2, 64, 200, 200, q, 0, q.stride(0), k, v, 0, k.stride(0), None, 1, out, 0, out.stride(0))
    torch.cuda.synchronize()
    ref = odit.multi_head_attention(*(x.cpu().numpy().astype(np.float64) for x in (q, k, v)), 2)
    # a score of size s is off by s 2^-24 or so, and the probabilities by that factor: s <= 30 * 40
    assert rel_l2(out.cpu().numpy().astype(np.float64), ref) <= 1200 * 2.0 ** -22
