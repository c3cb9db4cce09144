"""The forward kernels' q-tile heights and head dims against the fp64 oracle where a run crosses the
64-tile windows of its descriptors, ends on an odd step, or has a single step."""
import numpy as np
import pytest

from _harness import Case

pytestmark = pytest.mark.gpu

CASES = [
    # N, P, layout, shard, hq, hkv, d, bm, bn, document lengths (repeated to fill N)
    (8320, 1, "contiguous", 0, 2, 1, 64, 64, 64, [8320]),       # runs of up to 130 tiles, odd and even
    (8320, 1, "contiguous", 0, 1, 1, 64, 64, 64, [8320]),       # the same over four key streams
    (8320, 1, "contiguous", 0, 1, 1, 64, 128, 64, [8320]),
    (16640, 2, "contiguous", 1, 1, 1, 64, 128, 128, [16640]),   # 65 tiles per chunk
    (8320, 1, "contiguous", 0, 1, 1, 128, 64, 64, [8320]),
    (4096, 2, "zigzag", 1, 6, 3, 128, 64, 128, [1, 130, 7]),
    (4096, 2, "zigzag", 0, 6, 3, 64, 64, 128, [1, 130, 7]),
    (64, 1, "contiguous", 0, 1, 1, 64, 64, 64, [1, 62]),        # one tile, one step
    (128, 2, "contiguous", 1, 1, 1, 128, 64, 64, [128]),
    # q-tiles x heads on either side of where the key streams per workgroup change: four, two, one
    (2048, 1, "contiguous", 0, 8, 8, 64, 64, 64, [900, 3, 70]),     # 256
    (2048, 1, "contiguous", 0, 9, 3, 64, 64, 128, [900, 3, 70]),    # 288
    (2048, 1, "contiguous", 0, 17, 17, 64, 64, 64, [900, 3, 70]),   # 544
    (2048, 1, "contiguous", 0, 16, 8, 64, 128, 64, [2048]),         # 256: two, and 272: one
    (2048, 1, "contiguous", 0, 17, 17, 64, 128, 128, [2048]),
    (2048, 1, "contiguous", 0, 12, 4, 128, 128, 128, [5, 1200]),    # 192: two, and 208: one
    (2048, 1, "contiguous", 0, 13, 13, 128, 128, 64, [5, 1200]),
    (4096, 2, "zigzag", 1, 4, 4, 128, 64, 64, [4096]),              # 128 x 2 chunks
]


@pytest.mark.parametrize("split", [-1, 0, 3])
@pytest.mark.parametrize("case", CASES)
def test_forward_shapes(case, split):
    # O is bf16 and P enters its product as bf16: a relative error of 2^-8 of each, 2^-7 together;
    # LSE is fp32 (its scores are fp32 sums of exact bf16 products)
    N, P, layout, shard, hq, hkv, d, bm, bn, docs = case
    lengths = []
    while sum(lengths) < N:
        lengths.append(docs[len(lengths) % len(docs)])
    lengths[-1] -= sum(lengths) - N
    cu = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    c = Case(cu, N, P, layout, shard, hq, hkv, d, bm, bn, seed=4)
    got, ref = c.run_executor(max_run_tiles=split), c.run_oracle()
    for key, tol in (("o", 2.0 ** -7), ("lse", 1e-5)):
        for form in ("", "_fused", "_staged"):
            err = np.linalg.norm(got[key + form] - ref[key]) / np.linalg.norm(ref[key])
            assert err <= tol, (case, split, key + form, err)
