"""Kernels and branches at the sizes where they can go wrong: edges of tiles, remainders, the smallest and largest of a range."""
import numpy as np
import pytest
import torch

from helpers import cfg_kw, np_weights, to_np
from paper_2509_18085_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.fixture(scope="module")
def sp():
    from paper_2509_18085_amd import spiffy
    return spiffy


@pytest.mark.parametrize("V,K,B", [(1003, 5, 7), (130, 8, 33), (2049, 1, 1)])
def test_topk_slices_of_the_last_chunk(sp, V, K, B):
    """A chunk of 128 tokens is recomputed by eight workgroups: last chunks of 107, 2 and 1 tokens end inside a slice and inside
    a group of four rows."""
    from test_gpu_parity import check_head_topk
    cfg = synth.CONFIGS["c1"].scaled(dtype="bf16", d=192, V=V, B=B, G=3)
    st = synth.random_states(cfg.G, cfg.B, cfg.V, 0.2, 0.9, 3)
    st[1, :] = cfg.mask_id
    check_head_topk(sp, cfg, st, synth.hidden_states(cfg), synth.head_weights(cfg), 6.0, K, (0, 1))
