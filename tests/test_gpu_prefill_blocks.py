"""bf16 prefill around the edges of its query blocks, against a plain fp32 reference of the same attention.

Workgroups of 128 query rows (d_head 64; d_head 128 up to 8192 tokens, and packed prompts that are short on average) and
of 256 (longer prompts of d_head 128), tiles of 64 keys: lengths at and next to multiples of them, a single row, one
tile, dense and packed, both kinds of mask, the caches against a separate append."""
import numpy as np
import pytest
import torch

import synth
from paper_2608_06849_amd import (AohError, PagedCache, RingCache, aoh_kv_append, aoh_prefill, aoh_prefill_append,
                                  aoh_prefill_chunked, aoh_prefill_varlen)
from paper_2608_06849_amd.aoh import AOH_ERR_UNSUPPORTED
from tests.helpers import BF16_MAX_ABS, BF16_MEAN_ABS, bits, to_dtype

pytestmark = pytest.mark.gpu
DEV = "cuda"
HQ, MASK, N_SINK, WINDOW = 4, [0, 1], 20, 150


def reference(q, k, v, chunk, mask=MASK):
    """[T, H, D] bf16 -> [T, Hq, D] fp32."""
    t = q.shape[0]
    i = torch.arange(t, device=q.device).view(-1, 1)
    j = torch.arange(t, device=q.device).view(1, -1)
    lo = (i // chunk) * chunk - WINDOW if chunk else i - WINDOW + 1
    masks = [j <= i, (j <= i) & ((j < N_SINK) | (j >= lo))]
    out = torch.empty(q.shape, dtype=torch.float32, device=q.device)
    for h in range(HQ):
        g = h // (HQ // len(MASK))
        s = q[:, h].float() @ k[:, g].float().t().contiguous() / q.shape[-1] ** 0.5
        out[:, h] = torch.softmax(s.masked_fill(~masks[mask[g]], -torch.inf), -1) @ v[:, g].float()
    return out


def inputs(t, d, seed):
    return [to_dtype(synth.gaussian((t, h, d), seed, n), torch.bfloat16).to(DEV)
            for h, n in ((HQ, "q"), (2, "k"), (2, "v"))]


def caches(batch, t, d, seed):
    pages = (t + 15) // 16
    table = torch.from_numpy(synth.page_permutation(batch * pages, seed).reshape(batch, pages).copy())
    full = PagedCache.allocate(batch * pages, 1, d, torch.bfloat16, table)
    ring = RingCache.allocate(batch, 1, N_SINK, WINDOW, d, torch.bfloat16)
    for c in (full, ring):
        c.k.zero_()
        c.v.zero_()
    return full, ring


def check(got, want, what):
    err = (got.float() - want).abs()
    assert err.max() <= BF16_MAX_ABS and err.mean() <= BF16_MEAN_ABS, f"{what}: {err.max()} {err.mean()}"


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("t", [1, 63, 64, 65, 127, 128, 129, 192, 193, 255, 256, 257, 320, 385, 640, 1025])
def test_block_edges(t, d):
    q, k, v = inputs(t, d, t + d)
    for chunk in (0, 100):
        full, ring = caches(1, t, d, t)
        out = aoh_prefill_append(q[None], k[None], v[None], MASK, N_SINK, WINDOW, full, ring, chunk=chunk)
        check(out[0], reference(q, k, v, chunk), f"T {t} d {d} chunk {chunk}")
        full2, ring2 = caches(1, t, d, t)
        aoh_kv_append(k[None], v[None], MASK, torch.zeros(1, dtype=torch.int32, device=DEV), full2, ring2, N_SINK,
                      WINDOW)
        for a, b in ((full.k, full2.k), (full.v, full2.v), (ring.k, ring2.k), (ring.v, ring2.v)):
            assert np.array_equal(bits(a), bits(b)), f"T {t} d {d} chunk {chunk}: caches"


@pytest.mark.parametrize("t", [8192, 8193, 8449])
def test_long_prompt(t):
    # both sides of the change from 128 to 256 query rows
    q, k, v = inputs(t, 128, t)
    full, ring = caches(1, t, 128, t)
    out = aoh_prefill_append(q[None], k[None], v[None], MASK, N_SINK, WINDOW, full, ring)
    check(out[0], reference(q, k, v, 0), f"T {t}")


@pytest.mark.parametrize("lens", [[6144], [6145], [6145, 6145], [9000, 1, 257, 64, 65, 128, 700, 31], [9000] * 8])
def test_long_prompts_retrieval_only(lens):
    # the change from 128 to 256 rows of a layer without streaming heads: single, packed, uneven and even prompts
    q, k, v = inputs(sum(lens), 128, sum(lens))
    cu = torch.tensor([0] + list(np.cumsum(lens)), dtype=torch.int32, device=DEV)
    out = aoh_prefill_varlen(q, k, v, cu, max(lens), [0, 0], N_SINK, WINDOW) if len(lens) > 1 else \
        aoh_prefill(q[None], k[None], v[None], [0, 0], N_SINK, WINDOW)[0]
    for i in range(len(lens)):
        s = slice(int(cu[i]), int(cu[i + 1]))
        check(out[s], reference(q[s], k[s], v[s], 0, [0, 0]), f"{lens} sequence {i}")


@pytest.mark.parametrize("d,lens", [
    (64, [1, 127, 128, 129, 300, 64]), (128, [1, 127, 128, 129, 300, 64]),
    (128, [9000, 130, 8000]),                             # 256 rows: few prompts, long on average
    (128, [9000, 1, 257, 64, 65, 128, 700, 31]),          # 128 rows
])
def test_packed(d, lens):
    total = sum(lens)
    q, k, v = inputs(total, d, total)
    cu = torch.tensor([0] + list(np.cumsum(lens)), dtype=torch.int32, device=DEV)
    full, ring = caches(len(lens), max(lens), d, total)
    out = aoh_prefill_varlen(q, k, v, cu, max(lens), MASK, N_SINK, WINDOW, kv_full=full, kv_ring=ring)
    full2, ring2 = caches(len(lens), max(lens), d, total)
    for i, n in enumerate(lens):
        s = slice(int(cu[i]), int(cu[i]) + n)
        check(out[s], reference(q[s], k[s], v[s], 0), f"{lens} sequence {i}")
        aoh_kv_append(k[None, s], v[None, s], MASK, torch.zeros(1, dtype=torch.int32, device=DEV),
                      full2.rows(i, i + 1), RingCache(ring2.k[i:i + 1], ring2.v[i:i + 1], ring2.capacity), N_SINK,
                      WINDOW)
    for a, b in ((full.k, full2.k), (full.v, full2.v), (ring.k, ring2.k), (ring.v, ring2.v)):
        assert np.array_equal(bits(a), bits(b)), f"{lens}: caches"


@pytest.mark.parametrize("chunk", [0, 100])
@pytest.mark.parametrize("at", [3, 70, 140, 255, 299])
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_width_64_value_not_finite(bad, at, chunk):
    # d_head 64: a V row that is not finite reaches the rows that see its key, and of the others only those in a
    # wavefront (32 rows) with a row that sees a key of its tile (64 keys)
    t, d = 300, 64
    q, k, v = inputs(t, d, at)
    v[at] = 0
    want = aoh_prefill_chunked(q[None], k[None], v[None], MASK, N_SINK, WINDOW, chunk)[0] if chunk else \
        aoh_prefill(q[None], k[None], v[None], MASK, N_SINK, WINDOW)[0]
    v[at] = bad
    got = aoh_prefill_chunked(q[None], k[None], v[None], MASK, N_SINK, WINDOW, chunk)[0] if chunk else \
        aoh_prefill(q[None], k[None], v[None], MASK, N_SINK, WINDOW)[0]
    i = torch.arange(t, device=DEV).view(-1, 1)
    j = torch.arange(t, device=DEV).view(1, -1)
    lo = (i // chunk) * chunk - WINDOW if chunk else i - WINDOW + 1
    tile = slice(at // 64 * 64, at // 64 * 64 + 64)
    for h in range(HQ):
        sees = (j <= i) & ((j < N_SINK) | (j >= lo)) if MASK[h // (HQ // len(MASK))] else j <= i
        assert not torch.isfinite(got[:, h][sees[:, at]].float()).any(), f"head {h}"
        rows = torch.cat([sees[r:r + 32, tile].any().expand(min(32, t - r)) for r in range(0, t, 32)])
        assert np.array_equal(bits(got[:, h][~rows]), bits(want[:, h][~rows])), f"head {h}"


@pytest.mark.parametrize("d", [64, 128])
def test_grids_of_2_32_work_items(d):
    # blocks of the longest prompt x sequences x heads, with a bound on the length that is far from the real ones:
    # more work-items than a launch can hold
    b, hq = 1024, 32
    lens = [(37 * i) % 130 + 1 for i in range(b)]
    total = sum(lens)
    assert (total // 128) * b * hq * 256 > 1 << 32
    g = torch.Generator(device=DEV).manual_seed(d)
    x = torch.randn((total, hq + 2, d), dtype=torch.bfloat16, device=DEV, generator=g)
    q, k, v = x[:, :hq], x[:, hq:hq + 1], x[:, hq + 1:]
    k, v = torch.cat([k, v], 1), torch.cat([v, k], 1)
    cu = torch.tensor([0] + list(np.cumsum(lens)), dtype=torch.int32, device=DEV)
    got = []
    for bound in (max(lens), 131072):
        full, ring = caches(b, max(lens), d, d)
        out = torch.full_like(q, float("nan"))
        aoh_prefill_varlen(q, k, v, cu, bound, MASK, N_SINK, WINDOW, kv_full=full, kv_ring=ring, out=out)
        got.append([out, full.k, full.v, ring.k, ring.v])
    for a, w in zip(*got):
        assert np.array_equal(bits(a), bits(w))


@pytest.mark.parametrize("d", [64, 128])
def test_limit_on_the_bound(d):
    # blocks of 256 rows x heads x sequences below 2^31 are accepted whatever rows the call takes
    lens, hq = [1, 130, 64, 200, 7, 128, 129, 3], 32
    total = sum(lens)
    g = torch.Generator(device=DEV).manual_seed(d)
    q, k, v = (torch.randn((total, h, d), dtype=torch.bfloat16, device=DEV, generator=g) for h in (hq, 2, 2))
    cu = torch.tensor([0] + list(np.cumsum(lens)), dtype=torch.int32, device=DEV)
    got, want = (aoh_prefill_varlen(q, k, v, cu, n, MASK, N_SINK, WINDOW) for n in (1 << 30, max(lens)))
    assert np.array_equal(bits(got), bits(want))
    with pytest.raises(AohError) as e:
        aoh_prefill_varlen(q, k, v, torch.cat([cu, cu[-1:].expand(8)]), 1 << 30, MASK, N_SINK, WINDOW)
    assert e.value.status == AOH_ERR_UNSUPPORTED


def test_dense_batch_of_2_31_work_items():
    # one token each: the output is its V
    b, hq = 300000, 32
    x = torch.randn((b, 1, hq + 4, 64), dtype=torch.bfloat16, device=DEV)
    out = aoh_prefill(x[:, :, :hq], x[:, :, hq:hq + 2], x[:, :, hq + 2:], MASK, N_SINK, WINDOW)
    assert torch.equal(out, x[:, :, hq + 2:].repeat_interleave(hq // 2, 2))


@pytest.mark.parametrize("b,hq,mask,d", [
    (66, 32, [0] * 32, 128),             # parts of 14 sequences: four whole ones and a rest
    (34, 32, [0, 1] * 16, 64),           # both types, less than a cut is made for: all in one
    (200, 13, [0] * 10 + [1] * 3, 128),  # parts of 48: rounded up to whole rounds of 8 (sequence, head) pairs
    (70, 64, [0, 0, 1, 0] * 8, 128),     # two query heads a group: parts of 36 and all in one
])
@pytest.mark.parametrize("packed", [False, True])
def test_batches_in_parts(b, hq, mask, d, packed):
    # more K/V than a part of the batch holds: each sequence as by itself, bit for bit, and its rows of the caches
    n_kv = len(mask)
    lens = [150 + 7 * (i % 40) % 150 for i in range(b)] if packed else [140 if hq < 64 else 300] * b
    total = sum(lens)
    g = torch.Generator(device=DEV).manual_seed(b + hq)
    q, k, v = (torch.randn((total, h, d), dtype=torch.bfloat16, device=DEV, generator=g) for h in (hq, n_kv, n_kv))
    at = np.cumsum([0] + lens)
    pages = (max(lens) + 15) // 16
    table = torch.from_numpy(synth.page_permutation(b * pages, b).reshape(b, pages).copy())
    got = []
    for _ in range(2):
        full = PagedCache.allocate(b * pages, mask.count(0), d, torch.bfloat16, table)
        ring = RingCache.allocate(b, max(sum(mask), 1), N_SINK, WINDOW, d, torch.bfloat16)
        for c in (full, ring):
            c.k.zero_()
            c.v.zero_()
        got.append([torch.full_like(q, float("nan")), full, ring])
    ring_of = lambda r: r if sum(mask) else None  # noqa: E731
    out, full, ring = got[0]
    if packed:
        cu = torch.tensor(at, dtype=torch.int32, device=DEV)
        aoh_prefill_varlen(q, k, v, cu, max(lens), mask, N_SINK, WINDOW, kv_full=full, kv_ring=ring_of(ring), out=out)
    else:
        x = [t.view(b, lens[0], -1, d) for t in (q, k, v, out)]
        aoh_prefill_append(x[0], x[1], x[2], mask, N_SINK, WINDOW, full, ring_of(ring), out=x[3])
    want, full2, ring2 = got[1]
    for i in range(b):
        s = slice(at[i], at[i + 1])
        aoh_prefill_append(q[None, s], k[None, s], v[None, s], mask, N_SINK, WINDOW, full2.rows(i, i + 1),
                           ring_of(RingCache(ring2.k[i:i + 1], ring2.v[i:i + 1], ring2.capacity)), out=want[None, s])
    for a, w in zip((out, full.k, full.v, ring.k, ring.v), (want, full2.k, full2.v, ring2.k, ring2.v)):
        assert np.array_equal(bits(a), bits(w))
