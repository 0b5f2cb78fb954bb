"""Latents and cache of bf16 steps against recorded digests of their bytes.  Tilings, fused launches and splits are
chosen for speed and keep them; a change that is meant to round otherwise (or another compiler) records them anew."""
import dataclasses
import hashlib

import pytest
import torch

from paper_2607_04461_amd import synth
from paper_2607_04461_amd.pool import DraftPool

pytestmark = pytest.mark.gpu


def _digest(*tensors):
    h = hashlib.sha256()
    for t in tensors:
        h.update(t.contiguous().cpu().numpy().tobytes())
    return h.hexdigest()[:16]


def small_draft():
    """A small ragged pool over computed and proxied steps, q/k norm and rotary positions."""
    wl = dataclasses.replace(synth.WORKLOADS["mid_rope"], dtype="bf16")
    shape = wl.shape
    pool = DraftPool(wl, weights=synth.make_weights(shape, 5)[0])
    pool.reset()
    pool.cache.zero_()
    for k in range(5):
        pool.draft_step(k, [0] * shape.num_blocks, [k % 2] * shape.num_blocks)
    return _digest(pool.latents, pool.cache)


def test_small_draft():
    assert small_draft() == "cef9235cb4c7a7b4"


def guided_refine():
    """Two token rows of 1560 tokens at the 1.3B layer shapes: the MLP down-projection's K ranges are taken in turn."""
    shape = dataclasses.replace(synth.WORKLOADS["wan1.3b_step"].shape, num_blocks=1, qk_norm_rope=True)
    wl = dataclasses.replace(synth.WORKLOADS["wan1.3b_step"], shape=shape, text_len=64)
    pool = DraftPool(wl, weights=synth.make_weights(shape, 6)[0], guidance=5.0)
    pool.reset()
    for k in range(2):
        pool.refine_step(25 + k)
    return _digest(pool.latents)


def test_guided_refine():
    assert guided_refine() == "4371aea17c72dbbe"
