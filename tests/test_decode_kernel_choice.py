"""Which split pass a bf16 decode step takes (no GPU: the host's rule on batch, heads, width and capacities).

The rows of the GPU tests of many items are checked for the kernel that they are meant for, and the lines of the rule on
both sides.  Workspaces of batches over 64 sequences are sized for fixed splits, so the kernel for many items is left out
where its slots do not fit."""
import pytest

from paper_2608_06849_amd import aoh as A
from tests import test_gpu_decode_many as many

FIXED, WORK_SPACE, MANY = range(3)


def kernel(batch, hq, hkv, d, max_pages, ring_capacity):
    return A.lib().aoh_internal_decode_kernel(batch, hq, hkv, d, max_pages, ring_capacity)


@pytest.mark.parametrize("row", many.CASES, ids=lambda r: "-".join(str(x) for x in r[:4]))
def test_rows_of_the_gpu_tests(row):
    b, hq, hkv, d, mask, n_sink, window, prompt = row
    pages = (max(prompt) + 2 + 15) // 16 if 0 in mask else 1
    want = FIXED if b > 1024 or (b, hq, hkv) in many.SMALL_WORKSPACE else MANY
    assert kernel(b, hq, hkv, d, pages, n_sink + window) == want


@pytest.mark.parametrize("hq,hkv,d,items", [
    (16, 16, 128, 384), (16, 8, 128, 192), (24, 8, 128, 192), (32, 8, 128, 128), (28, 4, 128, 128),
    (16, 16, 64, 512), (16, 8, 64, 384), (32, 8, 64, 256), (14, 2, 64, 256 + 2),
])
def test_lines_between_the_work_space_kernels(hq, hkv, d, items):
    # items = (sequence, KV head) pairs; 14 / 2 heads reach 256 only with more sequences than the other kernel takes
    for pages in (33, 512, 8192):
        assert kernel(items // hkv, hq, hkv, d, pages, 384) == MANY
        if items // hkv <= 65:
            assert kernel(min(64, items // hkv - 1), hq, hkv, d, pages, 384) == WORK_SPACE
    short = 128 if d == 128 else 256
    if short // hkv <= 64:
        assert kernel(short // hkv, hq, hkv, d, 32, 384) == MANY
        assert kernel(short // hkv - 1, hq, hkv, d, 32, 384) == WORK_SPACE


def test_larger_batches():
    assert kernel(65, 4, 1, 128, 30, 384) == FIXED and kernel(65, 4, 1, 128, 31, 384) == MANY  # 481 tokens
    assert kernel(1024, 8, 2, 64, 64, 384) == MANY and kernel(1025, 8, 2, 64, 64, 384) == FIXED
