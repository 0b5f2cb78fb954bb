"""One full-quality step of one block, at widths that choose the kernels' wider variants, against the oracle: rows of
the q/k normalisation beside its register bounds, timestep features of several passes, and a patch embedding whose
workgroups take several blocks of tokens, the last of them short."""
import dataclasses
import functools

import numpy as np
import pytest
import torch

from oracle import dit as odit
from paper_2607_04461_amd import synth
from paper_2607_04461_amd.pool import DraftPool
from tests._util import TOL_V, rel_l2

pytestmark = pytest.mark.gpu


def _workload(shape, n, h, w):
    return dataclasses.replace(synth.WORKLOADS["tiny"], name="wide", shape=shape, n=n, latent_h=h, latent_w=w, text_len=5)


def _step_velocity(wl, flat, dtype, z0, **kw):
    pool = DraftPool(dataclasses.replace(wl, dtype=dtype), weights=flat)
    pool.reset(z0)
    pool.refine_step(1, **kw)
    torch.cuda.synchronize()
    dt = np.float64(pool.schedule[2]) - np.float64(pool.schedule[1])
    v = (pool.latents.cpu().numpy().astype(np.float64) - z0) / dt
    pool.close()
    return v


def _oracle_velocity(wl, W, z0):
    sched = wl.schedule()
    text = synth.make_text(wl.n_cond, wl.text_len, wl.shape.text_dim)
    zn = odit.refine_step(W, wl.shape, z0, sched[1], sched[2], odit.prepare_text(W, wl.shape, text), wl.cond_index())
    return (zn - z0) / (np.float64(sched[2]) - np.float64(sched[1]))


@functools.lru_cache(maxsize=1)
def _normalised(hidden, heads):
    shape = synth.ModelShape(num_blocks=1, hidden=hidden, heads=heads, mlp_hidden=64, freq_dim=32, text_dim=32,
                             qk_norm_rope=True)
    wl = _workload(shape, 1, 6, 6)
    flat, W = synth.make_weights(shape, 41)
    z0 = synth.make_latents(wl.n, shape.latent_channels, wl.latent_h, wl.latent_w)
    return wl, flat, z0, _oracle_velocity(wl, W, z0)


# a lane holds up to 8, 24, 48 or 96 elements of a row: rows at and just past 512, 1536 and 3072
@pytest.mark.parametrize("hidden,heads", [(512, 4), (520, 65), (1544, 193), (3072, 24), (3080, 385)])
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_qk_norm_rows(hidden, heads, dtype):
    wl, flat, z0, v = _normalised(hidden, heads)
    assert rel_l2(_step_velocity(wl, flat, dtype, z0), v) <= TOL_V[dtype]


# 1024 features a pass: at it, a little past it, and two whole passes and a little
@pytest.mark.parametrize("freq_dim", [1024, 1032, 2056])
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_timestep_features(freq_dim, dtype):
    shape = synth.ModelShape(num_blocks=1, hidden=64, heads=4, mlp_hidden=64, freq_dim=freq_dim, text_dim=32)
    wl = _workload(shape, 1, 6, 6)
    flat, W = synth.make_weights(shape, 42)
    W["t_w2"] *= 20      # modulations of some tenths, so that a few features show in the velocity
    W["mod_w"] *= 5
    W["head_mod_w"] *= 5
    z0 = synth.make_latents(wl.n, shape.latent_channels, wl.latent_h, wl.latent_w)
    assert rel_l2(_step_velocity(wl, flat, dtype, z0), _oracle_velocity(wl, W, z0)) <= TOL_V[dtype]


# two blocks of 16 tokens a workgroup: 409 blocks of 6534 tokens (patches of 2 and 4), 502 of 8029 (of 1); the last
# workgroup has one block of the 409, and the last block 6 or 13 tokens
@pytest.mark.parametrize("channels,patch,hidden,heads,n,h,w", [(16, 2, 1536, 12, 6, 66, 66), (4, 4, 1536, 12, 3, 132, 264),
                                                               (8, 1, 1280, 10, 7, 31, 37)])
def test_embedding(channels, patch, hidden, heads, n, h, w):
    shape = synth.ModelShape(num_blocks=1, hidden=hidden, heads=heads, mlp_hidden=64, freq_dim=32, text_dim=32,
                             latent_channels=channels, patch=patch)
    wl = _workload(shape, n, h, w)
    flat, W = synth.make_weights(shape, 43)
    z0 = synth.make_latents(n, channels, h, w)
    dump = torch.zeros((2, n, wl.tokens, hidden), device="cuda")
    _step_velocity(wl, flat, "bf16", z0, hidden_dump=dump)
    tok = synth.round_to_bf16(z0).reshape(n, channels, h // patch, patch, w // patch, patch).transpose(0, 2, 4, 1, 3, 5)
    ref = tok.reshape(n, wl.tokens, -1).astype(np.float64) @ synth.round_to_bf16(W["pe_w"]).astype(np.float64).T + W["pe_b"]
    # sums of at most 64 products in fp32
    assert rel_l2(dump[0].cpu().numpy(), ref) <= 8 * 2.0 ** -24
