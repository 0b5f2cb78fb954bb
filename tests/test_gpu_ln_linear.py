"""adaLN made inside the layer that reads it (small layers) against the two launches it replaces, which a step takes
while the NORM site is timed: hidden states of every block, latents and cache."""
import dataclasses

import pytest
import torch

from paper_2607_04461_amd import flashbon as fb
from paper_2607_04461_amd import synth
from paper_2607_04461_amd.pool import DraftPool

pytestmark = pytest.mark.gpu


# rows beside the tiles of 16 and 32; widths that end inside a K chunk of 64 (bf16: 32 and 96 past one), the widest
# that fused rows take (512), one that is never fused (1024) and, for fp32, the widest and narrowest sums (64 and 8);
# guided steps have a second set of rows and the head's fp32 output
@pytest.mark.parametrize("dtype,hidden,heads", [("bf16", 64, 4), ("bf16", 96, 3), ("bf16", 256, 2), ("bf16", 288, 9), ("bf16", 512, 4), ("bf16", 1024, 8), ("fp32", 64, 4),
                                                ("fp32", 8, 1), ("fp32", 40, 5)])
@pytest.mark.parametrize("n,h,w,guidance", [(1, 2, 2, None), (3, 6, 22, None), (2, 10, 14, 3.0)])
def test_fused_equals_two_launches(dtype, hidden, heads, n, h, w, guidance):
    shape = synth.ModelShape(num_blocks=2, hidden=hidden, heads=heads, mlp_hidden=96, freq_dim=32, text_dim=32)
    wl = dataclasses.replace(synth.WORKLOADS["tiny"], name="ln", shape=shape, n=n, latent_h=h, latent_w=w, dtype=dtype)
    flat, _ = synth.make_weights(shape, 91)
    rows = n * (2 if guidance else 1)
    outs = []
    for sites in ([], ["norm"]):
        pool = DraftPool(wl, weights=flat, guidance=guidance)
        pool.reset()
        fb.flashbon_set_timing(pool.model, sites)
        dump = torch.zeros((3, rows, wl.tokens, hidden), device="cuda")
        prev = torch.zeros_like(pool.latents)
        pool.draft_step(0, hidden_dump=dump, preview=prev)
        torch.cuda.synchronize()
        launches = fb.flashbon_read_timing(pool.model, "norm")[1]
        assert launches == (7 if sites else 0)   # three a block and the head's
        outs.append([x.clone() for x in (dump, prev, pool.latents)])
        pool.close()
    # the fused rows are summed and rounded as the separate launch's
    assert all(torch.equal(a, b) for a, b in zip(*outs))
