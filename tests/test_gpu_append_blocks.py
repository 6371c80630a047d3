"""Bulk appends whose chunks fill whole pages and ring blocks, or not: prompts in pieces at odd positions, sinks and
windows that are and are not multiples of a block, bit-exact against the oracle's cache placement model."""
import numpy as np
import pytest
import torch

from paper_2608_06849_amd import aoh_kv_append
from tests.test_gpu_decode import DEV, Run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("n_sink,window", [(64, 256), (16, 48), (32, 40), (5, 37), (0, 16), (0, 15), (7, 1), (20, 300)])
@pytest.mark.parametrize("pieces", [[700], [16, 16, 300], [13, 500, 1, 90], [1, 15, 64, 257, 33]])
def test_append_in_pieces(dtype, D, n_sink, window, pieces):
    total = sum(pieces)
    run = Run(2, 4, 4, D, [0, 1, 1, 0], n_sink, window, [total, total], 1, dtype, seed=total + window)
    at = 0
    for n in pieces:
        aoh_kv_append(run.k_seq[:, at:at + n].to(DEV), run.v_seq[:, at:at + n].to(DEV), run.mask, run.lens, run.full,
                      run.ring, n_sink, window)
        run.lens += n
        at += n
    torch.cuda.synchronize()
    run.check_caches()


def test_append_of_sequences_at_different_positions():
    # one call, start positions of every alignment, caches with room for some of them only
    B, D, n = 17, 128, 100
    run = Run(B, 4, 2, D, [0, 1], 16, 64, [16 + n] * B, 1, torch.bfloat16, seed=5)
    for b in range(B):
        f, r = run._views(b)
        if b:
            aoh_kv_append(run.k_seq[b:b + 1, :b].to(DEV), run.v_seq[b:b + 1, :b].to(DEV), run.mask, run.lens[b:b + 1],
                          f, r, 16, 64)
        run.lens[b] += b
    k = torch.stack([run.k_seq[b, b:b + n] for b in range(B)]).to(DEV)
    v = torch.stack([run.v_seq[b, b:b + n] for b in range(B)]).to(DEV)
    aoh_kv_append(k, v, run.mask, run.lens, run.full, run.ring, 16, 64)
    run.lens += n
    torch.cuda.synchronize()
    run.check_caches()
    assert np.array_equal(run.lens.cpu().numpy(), np.arange(B) + n)
