"""Timing sites records events and nothing else: a step gives the same bits with no site timed, with the NORM site
timed (small layers then make adaLN in a launch of its own) and, for a refinement, in the allocation-free step."""
import dataclasses

import pytest
import torch

from paper_2607_04461_amd import flashbon as fb
from paper_2607_04461_amd import synth
from paper_2607_04461_amd.pool import DraftPool

pytestmark = pytest.mark.gpu


# hidden widths on both sides of the fused rows' 256 (4 and 8 pieces a lane, whole and partial ones) and the fp32
# rows' 64; 544, 1024 and 1040 are wider than rows that are fused
@pytest.mark.parametrize("dtype,hidden,heads", [("bf16", 64, 4), ("bf16", 96, 3), ("bf16", 256, 2), ("bf16", 288, 9),
                                                ("bf16", 512, 4), ("bf16", 544, 17), ("bf16", 1024, 8), ("bf16", 1040, 65), ("fp32", 8, 1), ("fp32", 40, 5),
                                                ("fp32", 64, 4)])
@pytest.mark.parametrize("guidance", [None, 3.0])
def test_same_bits(dtype, hidden, heads, guidance):
    shape = synth.ModelShape(num_blocks=2, hidden=hidden, heads=heads, mlp_hidden=96, freq_dim=32, text_dim=32)
    wl = dataclasses.replace(synth.WORKLOADS["tiny"], name="timing", shape=shape, n=3, latent_h=6, latent_w=22, dtype=dtype)
    pool = DraftPool(wl, weights=synth.make_weights(shape, 91)[0], guidance=guidance)
    rows = wl.n * (2 if guidance else 1)
    drafts, refined = [], []
    for sites in ([], ["norm"], fb.SITES):
        fb.flashbon_set_timing(pool.model, sites)
        pool.reset()
        pool.cache.zero_()
        dump = torch.zeros((3, rows, wl.tokens, hidden), device="cuda")
        pool.draft_step(0, hidden_dump=dump)
        pool.draft_step(1)
        drafts.append((dump, pool.latents.clone(), pool.cache.clone()))
        z = drafts[0][1].clone()
        pool.refine_step(2, latents=z)
        refined.append(z)
    z = drafts[0][1].clone()
    fb.flashbon_refine_step_noalloc(pool.model, z, pool.schedule[2], pool.schedule[3], pool.text, pool.cond_index,
                                    pool.text_kv, pool.text_kv_valid, pool.trace, cfg=pool._cfg(wl.n))
    refined.append(z)
    torch.cuda.synchronize()
    for d in drafts[1:]:
        assert all(torch.equal(a, b) for a, b in zip(d, drafts[0]))
    assert all(torch.equal(z, refined[0]) for z in refined[1:])
    pool.close()
