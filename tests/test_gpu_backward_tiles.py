"""The dK/dV kernel's workgroup shapes (128, 64 or 32 keys, one, two or four streams of sub-tiles)
against the fp64 oracle at the grid sizes where the choice changes and where a stream runs out."""
import numpy as np
import pytest
import torch

from _harness import Case, compare_backward
from paper_2606_30460_amd.shard_attention import to_sharded

pytestmark = pytest.mark.gpu

CASES = [
    # N, hq, hkv, d, bm, bn, document lengths (repeated to fill N); key blocks of 32 in the call
    (2048, 8, 8, 128, 128, 128, [700]),     # 512: 32 keys per workgroup, four streams
    (2048, 9, 9, 128, 128, 128, [700]),     # 576: the same over runs; 64 keys, two streams in the tile-list call
    (2048, 16, 16, 128, 256, 64, [333]),    # 1024, 64-key tiles
    (4096, 18, 9, 128, 64, 128, [97, 5]),   # 1152: 128 keys, 64-row q-tiles, two query heads per K/V head
    (2048, 18, 18, 128, 64, 64, [2048]),    # 1152, 64-key tiles
    (2048, 8, 8, 64, 64, 64, [700]),        # head_dim 64: 512 and 576 blocks
    (2048, 18, 9, 64, 128, 64, [41]),
    (256, 3, 1, 128, 64, 128, [64]),        # runs of one 64-row q-tile per head: two sub-tiles, four streams
    (128, 1, 1, 64, 64, 64, [128]),
    # the dQ kernel's key streams: four at 256 q-tiles x heads (above), two at 288, 96 and 192, one at 208
    (2048, 9, 9, 64, 64, 64, [700, 9]),
    (2048, 6, 6, 64, 128, 64, [2048]),
    (2048, 12, 4, 128, 128, 128, [5, 1200]),
    (2048, 13, 13, 128, 128, 64, [5, 1200]),
]


def _case(N, hq, hkv, d, bm, bn, docs, seed=1):
    lengths = []
    while sum(lengths) < N:
        lengths.append(docs[len(lengths) % len(docs)])
    lengths[-1] -= sum(lengths) - N
    cu = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    return Case(cu, N, 1, "contiguous", 0, hq, hkv, d, bm, bn, seed=seed, backward=True)


@pytest.mark.parametrize("case", CASES)
def test_backward_workgroup_shapes(case):
    # bf16 gradients of the executor and fp32 accumulators of the tile-list call; the bar is what
    # bf16 P, dS and results give: 2^-8 of the largest element, against the oracle in 64 bits
    c = _case(*case)
    ref = c.run_oracle()
    for got in (c.run_executor(), c.run_tile_list()):
        rep = compare_backward(got, ref)
        assert max(rep.values()) <= 2.0 ** -7, (case, rep)
        for key in ("dk", "dv"):
            err = np.linalg.norm(got[key] - ref[key]) / np.linalg.norm(ref[key])
            assert err <= 2.0 ** -7, (case, key, err)


# runs of more than 64 tiles, so the kernels load a second and a third window of descriptors, and the dK/dV kernel
# starts over with the first at each query head of the group
LONG = [
    (8320, 1, 1, 64, 64, 64, [8320]),       # dK/dV 32 keys a workgroup; dQ four streams
    (4288, 6, 3, 64, 64, 64, [4288]),       # 32 keys, two heads a group; two streams
    (8320, 4, 2, 64, 64, 64, [8320]),       # the tile-list call 64 keys, the runs 32; one stream
    (4288, 12, 6, 64, 64, 64, [4288]),      # 64 keys
    (4288, 2, 1, 128, 64, 64, [4288]),      # head_dim 128: 32 keys; two streams
    (4288, 12, 6, 128, 64, 64, [4288]),     # 64 keys; one stream
    (8320, 2, 1, 128, 64, 128, [8320]),     # 128-key tiles, 32 keys
    (8320, 4, 4, 128, 64, 128, [8320]),     # 128 keys
]


@pytest.mark.parametrize("case", LONG)
def test_backward_descriptor_windows(case):
    test_backward_workgroup_shapes(case)


# several chunks and zigzag shards on both sides of the lines where the workgroups' keys (reachable 32-key blocks: 640
# for 128-key tiles, 768 for 64-key tiles, 512 in a chunk for the tile-list call) and the dQ streams change
CHUNKS = [
    # N, P, layout, shard, hq, hkv, d, bm, bn, document lengths
    (4096, 2, "zigzag", 1, 10, 5, 128, 128, 128, [4096]),       # 480 reachable, 80 q-tiles x heads
    (4096, 2, "zigzag", 0, 14, 7, 128, 128, 128, [900, 33]),    # 896
    (4096, 2, "contiguous", 1, 8, 8, 64, 64, 64, [2500, 7]),    # 1024, in a chunk 512; 256
    (4096, 4, "contiguous", 1, 10, 10, 64, 128, 64, [4096]),    # 640
    (6144, 3, "contiguous", 2, 4, 2, 128, 64, 64, [130, 3000]),     # 384; 128
    (6144, 3, "contiguous", 2, 6, 6, 128, 256, 128, [130, 3000]),   # 1152
]


@pytest.mark.parametrize("case", CHUNKS)
def test_backward_workgroup_shapes_of_chunks(case):
    # the bar of test_backward_workgroup_shapes
    N, P, layout, shard, hq, hkv, d, bm, bn, docs = case
    c = _case(N, hq, hkv, d, bm, bn, docs)
    c = Case(c.cu, N, P, layout, shard, hq, hkv, d, bm, bn, seed=2, backward=True)
    ref = c.run_oracle()
    for got in (c.run_executor(), c.run_tile_list()):
        rep = compare_backward(got, ref)
        assert max(rep.values()) <= 2.0 ** -7, (case, rep)
        for key in ("dk", "dv"):
            err = np.linalg.norm(got[key] - ref[key]) / np.linalg.norm(ref[key])
            assert err <= 2.0 ** -7, (case, key, err)


@pytest.mark.parametrize("d,bm,bn", [(64, 64, 64), (128, 128, 128)])
def test_many_empty_documents_in_a_wave(d, bm, bn):
    # repeated cu_seqlens entries are documents of no tokens: a hundred among one wave's 32 queries (inside
    # rows 64..95, and at the first row of 192..223), more boundaries than the kernels' 64-entry window holds
    cu = [0, 40] + [70] * 100 + [75, 128] + [192] * 100 + [200] + [200] * 70 + [256]
    c = Case(np.asarray(cu, dtype=np.int32), 256, 1, "contiguous", 0, 2, 1, d, bm, bn, seed=5, backward=True)
    got, ref = c.run_executor(), c.run_oracle()
    rep = compare_backward(got, ref)
    assert max(rep.values()) <= 2.0 ** -7, rep
    for form in ("", "_fused"):
        for key, tol in (("o", 2.0 ** -7), ("lse", 1e-5)):
            assert np.linalg.norm(got[key + form] - ref[key]) / np.linalg.norm(ref[key]) <= tol, key + form


@pytest.mark.parametrize("case", CASES[:7])
def test_dk_keeps_p_in_32_bits(case):
    # dS = P (dP - delta) from P in fp32: bf16 roundings (to nearest) leave the component of dK along the
    # exact one at 1 up to 0.003 / sqrt(elements) < 1e-5; a P cut to the 11 bits of fp16 loses
    # 2^-12 of it on average (2.4e-4).  (The executor's 128-key workgroups, CASES[3], do hold fp16.)
    c = _case(*case)
    ref = c.run_oracle()["dk"]
    outs = [c.run_tile_list()] + ([c.run_executor()] if case != CASES[3] else [])
    for got in outs:
        along = float(np.sum(got["dk"].astype(np.float64) * ref) / np.sum(np.square(ref, dtype=np.float64)))
        assert abs(along - 1.0) <= 2.0 ** -14, (case, along)


# the executor's choice by the lengths of its plan's runs (the descriptor's choice in brackets)
PLANS = [
    (2048, 16, 16, 128, 128, 128, [300]),   # 128 keys (128), P in fp32 up to 1024 blocks
    (2048, 15, 15, 128, 64, 128, [700]),    # 128 keys (128), 64-row q-tiles
    (2048, 14, 14, 128, 128, 128, [2048]),  # 64 keys (128)
    (2048, 36, 9, 128, 128, 128, [2048]),   # 32 keys (32), four query heads per K/V head
    (2048, 22, 11, 128, 64, 64, [2048]),    # 64 keys (32)
    (2048, 16, 16, 64, 64, 64, [2048]),     # 64 keys (64)
]


@pytest.mark.parametrize("case", PLANS)
def test_backward_by_plan(case):
    # the bars of test_backward_workgroup_shapes and test_dk_keeps_p_in_32_bits
    c = _case(*case)
    ref, got = c.run_oracle(), c.run_executor()
    rep = compare_backward(got, ref)
    assert max(rep.values()) <= 2.0 ** -7, (case, rep)
    along = float(np.sum(got["dk"].astype(np.float64) * ref["dk"]) / np.sum(np.square(ref["dk"], dtype=np.float64)))
    assert abs(along - 1.0) <= 2.0 ** -14, (case, along)


@pytest.mark.parametrize("case", [CASES[1], CASES[5]])
def test_backward_unaligned_outputs(case):
    # dK and dV 2 bytes (fp32 accumulators: 4 bytes) off a 16-byte boundary give the aligned bits
    from paper_2606_30460_amd import _lib as L
    c = _case(*case)
    s = L.shard_desc(c.N, 1, "contiguous", 0, c.bm, c.bn)
    desc = L.attn_desc(s, c.hq, c.hkv, c.d, c.d ** -0.5)
    dev = torch.device("cuda")
    q, k, v, d_o = (to_sharded(s, x.to(dev)).contiguous() for x in (c.q, c.k, c.v, c.do))
    ex = L.Executor(desc, backward=True)
    ex.plan(c.cu)
    o, lse = torch.empty_like(q), torch.empty(c.hq, c.N, dtype=torch.float32, device=dev)
    ex.forward(q, k, v, o, lse)
    got = {}
    for off in (0, 1):
        dq = torch.empty_like(q)
        dk, dv = (torch.zeros(k.numel() + off, dtype=k.dtype, device=dev)[off:].view(k.shape) for _ in range(2))
        ex.backward(q, k, v, d_o, o, lse, dq, dk, dv)
        delta = torch.empty_like(lse)
        L.attn_bwd_preprocess(o, d_o, c.N, c.hq, c.d, delta)
        doc_start = torch.empty(c.N, dtype=torch.int32, device=dev)
        L.doc_start(torch.from_numpy(c.cu).to(dev), c.N, doc_start)
        tiles = torch.from_numpy(L.plan(c.cu, s)["tiles"]).to(dev)
        dqa = torch.zeros(q.shape, dtype=torch.float32, device=dev)
        dka, dva = (torch.zeros(k.numel() + off, dtype=torch.float32, device=dev)[off:].view(k.shape) for _ in range(2))
        L.partial_attn_bwd(desc, q, k, v, d_o, lse, delta, doc_start, tiles, dqa, dka, dva)
        torch.cuda.synchronize()
        got[off] = [x.clone() for x in (dk, dv, dka, dva)]
    ex.close()
    for a, b in zip(got[0], got[1]):
        assert torch.equal(a, b)


def _lists(c):
    """Device inputs of a one-chunk case, its lists by k-tile and by q-tile, and a descriptor."""
    from paper_2606_30460_amd import _lib as L
    s = L.shard_desc(c.N, 1, "contiguous", 0, c.bm, c.bn)
    desc = L.attn_desc(s, c.hq, c.hkv, c.d, c.d ** -0.5)
    dev = torch.device("cuda")
    q, k, v, d_o = (to_sharded(s, x.to(dev)).contiguous() for x in (c.q, c.k, c.v, c.do))
    doc_start = torch.empty(c.N, dtype=torch.int32, device=dev)
    L.doc_start(torch.from_numpy(c.cu).to(dev), c.N, doc_start)
    tiles = L.plan(c.cu, s)["tiles"]
    lists = [[torch.from_numpy(np.ascontiguousarray(x)).to(dev) for x in L.plan_runs(s, tiles, m, 0)[:2]]
             for m in (L.MAJOR_K, L.MAJOR_Q_ALL)]
    return desc, q, k, v, d_o, doc_start, lists


@pytest.mark.parametrize("case", [(2048, 18, 18, 128, 128, 128, [700]), (2048, 36, 18, 64, 64, 64, [700, 31]),
                                  (2048, 16, 16, 128, 64, 64, [2048])])
def test_bits_do_not_depend_on_how_lists_are_cut(case):
    # the same runs in one call and in five: the same bits (the workgroup's shape follows from the descriptor)
    from paper_2606_30460_amd import _lib as L
    c = _case(*case)
    desc, q, k, v, d_o, doc_start, ((tk, rk), (ta, ra)) = _lists(c)
    lse = torch.full((c.hq, c.N), 6.0, device="cuda")
    delta = torch.randn(c.hq, c.N, generator=torch.Generator("cuda").manual_seed(3), device="cuda")
    got = []
    for pieces in (1, 5):
        for fp32 in (False, True):
            t = torch.float32 if fp32 else torch.bfloat16
            out = [torch.zeros(x.shape, dtype=t, device="cuda") for x in (q, k, v)]
            for i in range(pieces):
                cut = lambda r: r[len(r) * i // pieces:len(r) * (i + 1) // pieces].contiguous().reshape(-1)
                fn = L.partial_attn_bwd_runs if fp32 else L.attn_bwd_bf16
                fn(desc, q, k, v, d_o, lse, delta, doc_start, tk.reshape(-1), cut(rk), ta.reshape(-1), cut(ra), *out)
            got.append(out)
    for a, b in ((got[0], got[2]), (got[1], got[3])):
        for x, y in zip(a, b):
            assert torch.equal(x, y), (case, x.dtype)


@pytest.mark.parametrize("d", [64, 128])
def test_infinite_do_stays_infinite(d):
    # a run of three 64-row q-tiles over four streams of sub-tiles: two streams end past the run.  An
    # infinite dO in the last row gives infinities in dV of the k-tiles that lie wholly below it (every
    # P > 0 there), and no NaN
    c = _case(192, 1, 1, d, 64, 64, [192])
    c.do[191, 0, :] = float("inf")
    for got in (c.run_executor(), c.run_tile_list()):
        dv = got["dv"].reshape(-1, d)
        assert np.isposinf(dv[:128]).all(), (d, np.isnan(dv[:128]).sum())


def test_backward_q_rows_beyond_32_bit_offsets():
    # 2^20 query heads of 64: 32 Q rows are 4 GiB, so the dK/dV kernel's transfers take 64-bit addresses.
    # The heads repeat a block of 64 (16 K/V heads), so every block has to give the bits of the first, and the
    # first what a call over that block alone gives (other workgroup shapes: bf16 P, dS and results, 2^-7)
    from paper_2606_30460_amd import _lib as L
    N, D, hq, hkv, reps = 64, 64, 64, 16, 1 << 14
    dev = torch.device("cuda")
    g = torch.Generator(device="cuda").manual_seed(0)
    small = [torch.randn(N, h, D, generator=g, device=dev).to(torch.bfloat16) for h in (hq, hkv, hkv, hq)]
    lse_s = torch.full((hq, N), 4.0, device=dev)
    delta_s = torch.randn(hq, N, generator=g, device=dev)
    cu = np.asarray([0, N], dtype=np.int32)
    doc_start = torch.zeros(N, dtype=torch.int32, device=dev)
    got = {}
    for r in (1, reps):
        s = L.shard_desc(N, 1, "contiguous", 0, 64, 64)
        desc = L.attn_desc(s, hq * r, hkv * r, D, D ** -0.5)
        tiles = L.plan(cu, s)["tiles"]
        lists = [torch.from_numpy(np.ascontiguousarray(x).reshape(-1)).to(dev)
                 for m in (L.MAJOR_K, L.MAJOR_Q_ALL) for x in L.plan_runs(s, tiles, m, 0)[:2]]
        q, k, v, d_o = (x.repeat(1, r, 1) for x in small)
        lse, delta = lse_s.repeat(r, 1), delta_s.repeat(r, 1)
        for fp32 in (False, True):
            t = torch.float32 if fp32 else torch.bfloat16
            dq, dk, dv = (torch.zeros(x.shape, dtype=t, device=dev) for x in (q, k, v))
            if fp32:
                L.partial_attn_bwd(desc, q, k, v, d_o, lse, delta, doc_start, torch.from_numpy(tiles).to(dev), dq, dk, dv)
            else:
                L.attn_bwd_bf16(desc, q, k, v, d_o, lse, delta, doc_start, *lists, dq, dk, dv)
            for name, x, h in (("dq", dq, hq), ("dk", dk, hkv), ("dv", dv, hkv)):
                first = x[:, :h].contiguous()
                for i in range(0, r, 1024):     # (in pieces: the comparison's own buffers stay small)
                    part = x[:, i * h:min(r, i + 1024) * h].view(N, -1, h, D)
                    assert torch.equal(part, first.unsqueeze(1).expand_as(part)), (name, fp32, r, i)
                got[name, fp32, r] = first.float()
            del dq, dk, dv
        del q, k, v, d_o, lse, delta
    for name in ("dq", "dk", "dv"):
        for fp32 in (False, True):
            a, b = got[name, fp32, 1], got[name, fp32, reps]
            assert float((a - b).norm() / a.norm()) <= 2.0 ** -7, (name, fp32)
