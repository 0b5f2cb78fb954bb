"""The head projection with its latent update (and preview) against the oracle's step, for the patch sizes and
channel counts whose columns meet the edges of its 32-row x 64-column tiles."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import dit as odit
from paper_2607_04461_amd import flashbon as fb
from paper_2607_04461_amd import synth
from paper_2607_04461_amd.pool import DraftPool
from tests._util import TOL_V, rel_l2

pytestmark = pytest.mark.gpu


# (channels, patch): C p^2 columns = 64, 8 (narrower than a tile), 72 and 128 (a second, partial or whole column
# tile); the hidden widths 72 and 1088 end inside a K chunk of 64 and give the waves unequal shares; the last three
# have more than one 32x64 tile per CU and take 128x128 tiles
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("channels,patch,hidden,heads,h,w", [
    (16, 2, 64, 4, 10, 6), (2, 2, 72, 9, 14, 22), (18, 2, 64, 4, 6, 6), (32, 2, 1088, 17, 10, 14), (8, 1, 64, 4, 5, 7),
    (8, 3, 64, 4, 9, 12), (4, 4, 128, 4, 8, 20), (16, 2, 128, 1, 106, 106), (32, 2, 192, 6, 60, 98), (8, 3, 128, 2, 108, 117)])
def test_head_update_and_preview(dtype, channels, patch, hidden, heads, h, w):
    shape = synth.ModelShape(num_blocks=1, hidden=hidden, heads=heads, mlp_hidden=64, freq_dim=32, text_dim=32,
                             latent_channels=channels, patch=patch)
    wl = dataclasses.replace(synth.WORKLOADS["tiny"], name="head", shape=shape, n=3, latent_h=h, latent_w=w, dtype=dtype)
    flat, W = synth.make_weights(shape, 77)
    z0 = synth.make_latents(wl.n, channels, h, w)
    text = synth.make_text(wl.n_cond, wl.text_len, shape.text_dim)
    sched = wl.schedule()
    zn = odit.refine_step(W, shape, z0, sched[1], sched[2], odit.prepare_text(W, shape, text), wl.cond_index())
    v = (zn - z0) / (np.float64(sched[2]) - np.float64(sched[1]))
    pool = DraftPool(wl, weights=flat)
    pool.reset(z0)
    prev = torch.full_like(pool.latents, 7.0)
    fb.flashbon_refine_step(pool.model, pool.latents, sched[1], sched[2], pool.text, pool.cond_index, pool.text_kv,
                            pool.text_kv_valid, preview=prev)
    torch.cuda.synchronize()
    got = pool.latents.cpu().numpy().astype(np.float64)
    assert rel_l2((got - z0) / (np.float64(sched[2]) - np.float64(sched[1])), v) <= TOL_V[dtype]
    assert rel_l2((z0 - prev.cpu().numpy()) / np.float64(sched[1]), v) <= TOL_V[dtype]
    pool.close()
