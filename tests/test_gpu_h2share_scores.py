"""Anchor decode where its score codes cross a wavefront's LDS buffer: its capacity (the blocks of one wavefront's
partials, fewer for wide groups), odd block counts, wavefront ranges longer than it, and the split pass of many items."""
import numpy as np
import pytest
import torch

import synth
from paper_2608_06849_amd import aoh_decode, aoh_decode_anchor, aoh_decode_workspace_bytes
from tests.helpers import bits
from tests.test_gpu_h2share import DEV, _bf, _check_selection, _decode_setup, _fill

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,L,lens,hq,hkv,d,mask,top_k", [
    (4, 30000, [30000, 29999, 29985, 17], 32, 2, 64, [0, 0], 100),        # 16 heads: 6 blocks a buffer, ranges beyond it
    (2, 8000, [8000, 7777], 7, 1, 128, [0], 64),                          # 7 heads: 32 blocks
    (2, 5000, [4993, 33], 4, 4, 128, [0, 1, 0, 0], 40),                   # 1 head: 226 blocks
    (130, 300, [(37 * i) % 300 + 1 for i in range(130)], 8, 2, 64, [0, 1], 20),  # whole items per wavefront
    (5, 4200, [1023, 1024, 1025, 4096, 4097], 2, 1, 64, [0], 50),         # runs of 1 and 4 positions of the selection
    (66, 700, [(53 * i) % 700 + 1 for i in range(66)], 32, 2, 128, [0, 0], 30),  # 16 heads: 14 blocks
])
def test_anchor_score_buffer(B, L, lens, hq, hkv, d, mask, top_k):
    k, v, full, ring = _decode_setup(B, L, hq, hkv, d, mask, 4, 64, B + hq)
    _fill(k, v, mask, lens, full, ring, 4, 64)
    q = _bf(synth.gaussian((B, hq, d), B + hq, "h2-q"))
    lens_t = torch.tensor(lens, dtype=torch.int32, device=DEV)
    out_a, idx = aoh_decode_anchor(q.to(DEV), full, ring, mask, lens_t, 4, 64, top_k)
    ws = torch.empty(aoh_decode_workspace_bytes(B, hq, d, full.block_table.shape[1], 68) // 4 + 4,
                     dtype=torch.float32, device=DEV)
    out_d = aoh_decode(q.to(DEV), full, ring, mask, lens_t, 4, 64, workspace=ws)
    torch.cuda.synchronize()
    assert np.array_equal(bits(out_a), bits(out_d)), "anchor output differs from aoh_decode"
    _check_selection(idx.cpu().numpy(), q, k, lens, mask, top_k, f"anchor {B, L, hq, hkv, d, top_k}")
