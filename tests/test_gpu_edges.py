"""Edges of the kernels' tiles, batches and dispatch rules (GPU, against the oracle).

GEMM cases use small-integer operands, whose fp32 partial sums are exact in any
order, so every comparison is bit for bit; so are the chunk sums and the
permutation by their definition."""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_09200_amd import binding as occ
from gpu_common import DEV, bf16_bits

pytestmark = pytest.mark.gpu


def int_gemm(M, N, K, layout, variant=0, grid_cap=0, seed=0):
    """(result bits, oracle bits) of an integer GEMM; C starts as NaN."""
    g = torch.Generator().manual_seed(seed)
    A = torch.randint(-2, 3, (M, K), generator=g).to(torch.bfloat16)
    B = torch.randint(-2, 3, (K, N) if layout == "kn" else (N, K), generator=g).to(torch.bfloat16)
    C = torch.full((M, N), float("nan"), device=DEV, dtype=torch.bfloat16)
    f = occ.occ_gemm_ex if layout == "kn" else occ.occ_gemm_bt_ex
    f(A.to(DEV), B.to(DEV), C, variant=variant, grid_cap=grid_cap)
    torch.cuda.synchronize()
    return bf16_bits(C), oracle.gemm_bf16(A, B, M, N, K, b_layout=layout)


# 256x256 tile: one to five k-steps (the two-stage pipeline's fill and drain), a
# last k-step of one 8-wide chunk, one row or column more or less than a tile,
# and rows of C that are not 16-byte aligned (B N x K only)
@pytest.mark.parametrize("layout", ["kn", "nk"])
@pytest.mark.parametrize("M,N,K", [(256, 256, 8), (255, 248, 64), (257, 264, 72), (256, 512, 128), (1, 8, 136),
                                   (511, 136, 192), (300, 520, 264), (129, 257, 320), (64, 131, 200)])
def test_large_tile_edges(layout, M, N, K):
    if layout == "kn":
        N = (N + 7) // 8 * 8
    variant = 32 if layout == "kn" else 16
    for cap in (0, 1):  # one workgroup per tile, and one that walks all tiles
        got, ref = int_gemm(M, N, K, layout, variant, cap, seed=M + K)
        assert np.array_equal(got, ref), cap


# the collective reads each GEMM's output through the device counter while the
# next GEMM runs: every tile kernel's device-scope stores, wide and narrow rows
@pytest.mark.parametrize("layout,variant,M,N,K", [
    ("kn", 32, 520, 264, 128), ("nk", 16, 520, 264, 128), ("nk", 16, 264, 129, 72), ("kn", 35, 264, 200, 72),
    ("nk", 14, 264, 129, 72), ("kn", 39, 72, 136, 64), ("nk", 9, 72, 133, 64), ("kn", 37, 72, 136, 64),
    ("nk", 7, 72, 133, 64), ("kn", 43, 72, 136, 64), ("nk", 18, 72, 133, 64), ("kn", 33, 16, 264, 136), ("nk", 21, 8, 133, 136), ("nk", 34, 16, 100, 1024)])
def test_collective_reads_the_gemm_output(layout, variant, M, N, K):
    n = 4
    g = torch.Generator().manual_seed(M + N)
    A = torch.randint(-2, 3, (M, K), generator=g).to(torch.bfloat16)
    B = torch.randint(-2, 3, (K, N) if layout == "kn" else (N, K), generator=g).to(torch.bfloat16)
    peers = torch.randint(-4, 5, (2, M * N), generator=g).float()
    ref = oracle.gemm_bf16(A, B, M, N, K, b_layout=layout)
    C = torch.full((n, M, N), float("nan"), device=DEV, dtype=torch.bfloat16)
    out = torch.full((M * N,), float("nan"), device=DEV)
    occ.run_overlap(A.to(DEV), B.to(DEV), C, bufs=peers.to(DEV), out=out, n_iter=n, reps=1, warmup=0,
                    flags=occ.OCC_RUN_OVL, gemm_variant=variant, b_layout=layout, reduce_own=True, dep="counter")
    torch.cuda.synchronize()
    for i in range(n):
        assert np.array_equal(bf16_bits(C[i]), ref), i
    own = (ref.astype(np.uint32) << 16).view(np.float32).reshape(-1)
    assert np.array_equal(out.cpu().numpy(), own + peers[0].numpy() + peers[1].numpy())


def f32_at(values, offset):
    """A GPU copy of `values` starting `offset` elements past a 16-byte boundary."""
    buf = torch.full((values.numel() + 8,), float("nan"), device=DEV, dtype=values.dtype)
    assert buf.data_ptr() % 16 == 0
    v = buf[offset:offset + values.numel()]
    v.copy_(values)
    return v


# every exact term count and the batched ones, one to a few positions per lane,
# chunks and output each at its own offset from a 16-byte boundary
@pytest.mark.parametrize("terms", list(range(1, 18)) + [64])
@pytest.mark.parametrize("length", [1, 3, 6, 515, 4099, 262151])
def test_chunk_sum_terms_and_alignments(terms, length):
    if length > 5000 and terms > 17:
        length = 5003
    g = torch.Generator().manual_seed(terms * 1000 + length)
    x = torch.rand((terms, length), generator=g) * 2 - 1
    for shift in (0, 1, 3):
        bufs = [f32_at(x[c], (c + shift) % 4) if shift else x[c].to(DEV) for c in range(terms)]
        out = f32_at(torch.zeros(length), shift)
        occ.share_reduce(bufs, out, wgs=3 if length > 200000 else 0)
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy().view(np.uint32), oracle.chunk_sum_f32(x.numpy()).view(np.uint32)), shift


@pytest.mark.parametrize("peers", [0, 1, 2, 6, 15, 16, 63])
@pytest.mark.parametrize("length", [1, 7, 515, 66053])
def test_own_chunk_sum_terms_and_alignments(peers, length):
    g = torch.Generator().manual_seed(peers * 1000 + length)
    own = torch.randn(length, generator=g).to(torch.bfloat16)
    x = torch.rand((peers, length), generator=g) * 2 - 1
    want = own.float()
    for c in range(peers):
        want = want + x[c]
    for shift in (0, 1, 2):  # own at 16-, 2- and 4-byte alignment
        out = f32_at(torch.zeros(length), shift)
        occ.share_reduce_own(f32_at(own, shift), [f32_at(x[c], (c + shift) % 4) for c in range(peers)], out)
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy().view(np.uint32), want.numpy().view(np.uint32)), shift


# chunk sizes around 16 bytes and around a workgroup's round, source and
# destination at their own byte offsets; nothing outside the destination changes
@pytest.mark.parametrize("nchunks,chunk_bytes", [(1, 1), (5, 15), (3, 16), (7, 17), (512, 31), (33, 1000), (3, 16384),
                                                 (2, 16400), (5, 40001), (3, 300003), (300, 20480), (4, 1 << 20)])
def test_permute_alignments(nchunks, chunk_bytes):
    g = torch.Generator().manual_seed(chunk_bytes)
    src = torch.randint(0, 256, (nchunks * chunk_bytes,), generator=g, dtype=torch.uint8)
    perm = torch.randperm(nchunks, generator=g).to(torch.int32)
    want = oracle.permute_chunks(src.numpy(), perm.numpy(), chunk_bytes)
    for so, do in ((0, 0), (1, 0), (0, 3), (8, 15), (2, 2)):
        s = torch.zeros(src.numel() + 32, dtype=torch.uint8, device=DEV)
        s[so:so + src.numel()] = src.to(DEV)
        d = torch.full((src.numel() + 64,), 77, dtype=torch.uint8, device=DEV)
        view = d[16 + do:16 + do + src.numel()]
        occ.share_permute(s[so:so + src.numel()], view, perm, chunk_bytes, wgs=0 if do else 5)
        torch.cuda.synchronize()
        assert np.array_equal(view.cpu().numpy(), want), (so, do)
        assert (d[:16 + do] == 77).all() and (d[16 + do + src.numel():] == 77).all(), (so, do)


# register-pipelined tiles: one to several k-steps (fewer than, as many as and more
# than the stages), partial tiles, rows of C off 16 bytes (B N x K); 128x128 with
# its non-temporal B is covered by the shape rule below
@pytest.mark.parametrize("layout,variant", [("kn", v) for v in (35, 40, 41, 42, 43, 44)] + [("nk", v) for v in (10, 11, 12, 13, 14, 17, 18)])
@pytest.mark.parametrize("M,N,K", [(64, 64, 8), (65, 72, 64), (255, 136, 136), (257, 120, 256), (128, 264, 328),
                                   (40, 129, 520), (130, 67, 1032), (31, 33, 392)])
def test_register_pipelined_tile_edges(layout, variant, M, N, K):
    if layout == "kn":
        N = (N + 7) // 8 * 8
    for cap in (0, 1):
        got, ref = int_gemm(M, N, K, layout, variant, cap, seed=M + K)
        assert np.array_equal(got, ref), cap


def test_shape_rule_takes_every_tile_and_gives_the_same_bits():
    # one shape per tile of the automatic choice; all tiles sum over k in one order
    for (M, N, K), kn, nk in (((4096, 4096, 512), 32, 16), ((1792, 2816, 1024), 40, 10), ((2048, 2048, 512), 35, 14),
                              ((1024, 2048, 1024), 41, 11), ((1024, 1024, 1536), 42, 12), ((640, 512, 256), 39, 9),
                              ((512, 1024, 1536), 43, 17), ((512, 512, 1536), 44, 18),
                              # the 32-row tiles have no limit in K of their own
                              ((1024, 512, 512), 43, 17), ((512, 512, 512), 44, 18), ((64, 1024, 512), 44, 18),
                              ((64, 1024, 520), 44, 18), ((300, 696, 400), 44, 18)):
        assert occ.occ_gemm_plan_query(M, N, K)["kernel_id"] == kn, (M, N, K)
        assert occ.occ_gemm_bt_plan_query(M, N, K)["kernel_id"] == nk, (M, N, K)
        g = torch.Generator(device=DEV).manual_seed(M)
        A = torch.randn((M, K), generator=g, device=DEV).to(torch.bfloat16)
        Bt = torch.randn((N, K), generator=g, device=DEV).to(torch.bfloat16)
        B = Bt.t().contiguous()
        C = [torch.full((M, N), float("nan"), device=DEV, dtype=torch.bfloat16) for _ in range(3)]
        occ.occ_gemm(A, B, C[0])
        occ.occ_gemm_bt(A, Bt, C[1])
        occ.occ_gemm_ex(A, B, C[2], variant=37)
        torch.cuda.synchronize()
        assert torch.equal(C[0].view(torch.int16), C[2].view(torch.int16)), (M, N, K)
        assert torch.equal(C[1].view(torch.int16), C[2].view(torch.int16)), (M, N, K)
    # a pad beside which the tile does not fit, but the one by tile count does
    assert occ.occ_gemm_plan_query(512, 1024, 1536, 128 << 10)["kernel_id"] == 39


@pytest.mark.parametrize("layout,M,kernel", [("kn", 40, 35), ("nk", 40, 13), ("nk", 70, 14)])
def test_streamed_weight_takes_non_temporal_loads(layout, M, kernel):
    # B just above the last-level cache, one row of tiles: against the opt2 tile
    N, K = 16520, 8192
    q = occ.occ_gemm_plan_query if layout == "kn" else occ.occ_gemm_bt_plan_query
    assert q(M, N, K)["kernel_id"] == kernel
    g = torch.Generator(device=DEV).manual_seed(5)
    A = torch.randn((M, K), generator=g, device=DEV).to(torch.bfloat16)
    B = torch.randn((K, N) if layout == "kn" else (N, K), generator=g, device=DEV).to(torch.bfloat16)
    C = [torch.full((M, N), float("nan"), device=DEV, dtype=torch.bfloat16) for _ in range(2)]
    f = occ.occ_gemm_ex if layout == "kn" else occ.occ_gemm_bt_ex
    f(A, B, C[0])
    f(A, B, C[1], variant=37 if layout == "kn" else 7)
    torch.cuda.synchronize()
    assert torch.equal(C[0].view(torch.int16), C[1].view(torch.int16))


# skinny K x N: 32-, 64- and 128-column units at and around their limits, the same
# ones with a pad, K of less than a block per wave and ragged
@pytest.mark.parametrize("M,N,K", [(1, 8, 8), (5, 40, 72), (16, 2048, 200), (13, 2056, 136), (16, 2120, 1032),
                                   (7, 16384, 40), (16, 16392, 64)])
def test_skinny_kn_unit_widths(M, N, K):
    cus = occ.occ_gemm_plan_query(512, 512, 512)["num_cus"]
    plan = occ.occ_gemm_plan_query(M, N, K)
    want = 32 if -(-N // 32) <= cus // 4 else 64 if -(-N // 64) <= cus else 128
    assert plan["kernel_id"] == 33 and plan["tile_n"] == want and plan["tiles"] == -(-N // want)
    # a pad changes the residency, not the kernel: up to the last byte that fits
    for pad in (1, 16 << 10, plan["max_lds_per_wg"] - plan["tile_lds_bytes"]):
        p = occ.occ_gemm_plan_query(M, N, K, pad)
        assert p["feasible"] and p["tile_n"] == want and p["tile_lds_bytes"] == plan["tile_lds_bytes"], pad
    assert not occ.occ_gemm_plan_query(M, N, K, pad + 1)["feasible"]
    for cap in (0, 3):
        got, ref = int_gemm(M, N, K, "kn", 33, cap, seed=N + K)
        assert np.array_equal(got, ref), cap
    g = torch.Generator(device=DEV).manual_seed(N)
    A = torch.randn((M, K), generator=g, device=DEV).to(torch.bfloat16)
    B = torch.randn((K, N), generator=g, device=DEV).to(torch.bfloat16)
    C = [torch.full((M, N), float("nan"), device=DEV, dtype=torch.bfloat16) for _ in range(3)]
    occ.occ_gemm(A, B, C[0])
    occ.occ_gemm(A, B, C[1], lds_bytes=16 << 10)
    occ.occ_gemm(A, B, C[2], lds_bytes=pad)
    torch.cuda.synchronize()
    assert torch.equal(C[0].view(torch.int16), C[1].view(torch.int16))
    assert torch.equal(C[0].view(torch.int16), C[2].view(torch.int16))


def tile_by_count(M, N, cus):
    """LDS of the largest of 256x256, 128x128 and 64x64 that still gives a 256x256 tile
    per CU or a 128x128 one per two CUs: the pads it leaves room for are never refused."""
    if -(-M // 256) * -(-N // 256) >= cus:
        return 128 << 10
    return (96 << 10) if -(-M // 128) * -(-N // 128) >= cus // 2 else (32 << 10)


# one shape per tile of the automatic choice, and streamed weights
@pytest.mark.parametrize("layout", ["kn", "nk"])
@pytest.mark.parametrize("M,N,K", [(4096, 4096, 512), (1792, 2816, 1024), (2048, 2048, 512), (1024, 2048, 1024),
                                   (1024, 1024, 1536), (640, 512, 256), (512, 1024, 1536), (512, 512, 1536),
                                   (40, 16520, 8192), (70, 16520, 8192), (4104, 4104, 1024)])
def test_pad_keeps_the_tile_wherever_it_fits(layout, M, N, K):
    q = occ.occ_gemm_plan_query if layout == "kn" else occ.occ_gemm_bt_plan_query
    p0 = q(M, N, K)
    limit, tile = p0["max_lds_per_wg"], p0["tile_lds_bytes"]
    for pad in (1, 16, 1 << 10, 8 << 10, 16 << 10, 32 << 10, (32 << 10) + 16, 64 << 10, 96 << 10, 128 << 10,
                (128 << 10) + 16, limit - tile, limit - tile + 1, limit + 16):
        p = q(M, N, K, pad)
        if tile + pad <= limit:
            assert p["feasible"] and p["kernel_id"] == p0["kernel_id"], pad
            assert p["wg_per_cu"] <= p0["wg_per_cu"], pad
        else:
            assert p["feasible"] == (tile_by_count(M, N, p0["num_cus"]) + pad <= limit), pad
    # the pad that takes one resident workgroup away is one to offer wherever there are two
    if p0["wg_per_cu"] > 1:
        p = q(M, N, K, p0["lds_per_cu"] // p0["wg_per_cu"] + 1 - tile)
        assert p["kernel_id"] == p0["kernel_id"] and p["wg_per_cu"] == p0["wg_per_cu"] - 1
    g = torch.Generator(device=DEV).manual_seed(M)
    A = torch.randn((M, K), generator=g, device=DEV).to(torch.bfloat16)
    B = torch.randn((K, N) if layout == "kn" else (N, K), generator=g, device=DEV).to(torch.bfloat16)
    C = [torch.full((M, N), float("nan"), device=DEV, dtype=torch.bfloat16) for _ in range(2)]
    f = occ.occ_gemm if layout == "kn" else occ.occ_gemm_bt
    f(A, B, C[0])
    for pad in (16, limit - tile, min(limit - tile_by_count(M, N, p0["num_cus"]), 128 << 10)):
        f(A, B, C[1].fill_(float("nan")), lds_bytes=pad)
        torch.cuda.synchronize()
        assert torch.equal(C[0].view(torch.int16), C[1].view(torch.int16)), pad


# a rate is an upper bound at the default grid too, where a workgroup moves as
# little as one partial round or one position: the transfer takes at least
# bytes / rate (less 2 % for the two clocks), and not several times that (a
# workgroup's share is whole positions or rounds of 16 KiB; 30 us for the
# launches and the waits' granularity).  Results are those of the unpaced call.
PACED = [("permute", 16, 400 << 10), ("permute", 64, 100 << 10), ("permute", 8, 1 << 20), ("permute", 32, 500 << 10),
         ("permute", 16, (400 << 10) + 2), ("permute", 7, 16384 * 3 + 16), ("permute", 512, 1001)]
PACED += [("reduce", n, length) for n in (2, 3, 4, 5, 8, 16, 20) for length in (1 << 16, (1 << 18) + 3, 1 << 20)]
PACED += [("own", n, length) for n in (1, 2, 7) for length in (1 << 16, (1 << 18) + 64)]


@pytest.mark.parametrize("kind,n,size", PACED)
def test_paced_collective_keeps_the_rate_at_the_default_grid(kind, n, size):
    g = torch.Generator(device=DEV).manual_seed(size + n)
    A, B = (torch.ones((64, 64), device=DEV, dtype=torch.bfloat16) for _ in range(2))
    C = torch.empty((64, 64), device=DEV, dtype=torch.bfloat16)
    rate = 50.0 if kind == "permute" else 100.0
    if kind == "permute":
        src = torch.randint(0, 256, (n * size,), generator=g, device=DEV, dtype=torch.uint8)
        perm = torch.arange(n - 1, -1, -1, dtype=torch.int32)
        comm = dict(src=src, dst=torch.zeros_like(src), perm=perm, chunk_bytes=size)
        want, got, nbytes = src.view(n, size).flip(0).reshape(-1), comm["dst"], 2 * n * size
    else:
        x = torch.rand((n, size), generator=g, device=DEV)
        want, got = torch.empty(size, device=DEV), torch.zeros(size, device=DEV)
        comm = dict(bufs=x, out=got)
        nbytes = 4 * (n + 1) * size
        if kind == "own":
            A, B = torch.ones((8, 8), device=DEV, dtype=torch.bfloat16), torch.ones((8, size // 8), device=DEV, dtype=torch.bfloat16)
            C = torch.empty((3, 8, size // 8), device=DEV, dtype=torch.bfloat16)
            comm["reduce_own"] = True
            nbytes += 2 * size
            occ.share_reduce_own(torch.full((size,), 8.0, device=DEV, dtype=torch.bfloat16), x, want)
        else:
            occ.share_reduce(x, want)
    r = occ.run_overlap(A, B, C, n_iter=3, reps=3, warmup=1, comm_priority=0, comm_rate_gbs=rate,
                        flags=occ.OCC_RUN_ISO | occ.OCC_RUN_PACE_ALL, **comm)
    torch.cuda.synchronize()
    assert torch.equal(got.view(torch.uint8), want.view(torch.uint8))
    paced_us = nbytes / rate * 1e-3
    assert 0.98 * paced_us <= r["t_comm_ms"] * 1e3 <= 2.0 * paced_us + 30.0, (r["t_comm_ms"] * 1e3, paced_us)


def test_k_beyond_the_64x64_tile_is_refused_or_register_staged():
    # also for the shapes whose 32x32 tile could address twice that K
    for M, N in ((17, 64), (32, 8), (300, 200), (4096, 4096)):
        k = 1 << 24
        assert occ.occ_gemm_plan_query(M, N, k)["feasible"] and occ.occ_gemm_bt_plan_query(M, N, k)["kernel_id"] != 7
        for K in (k + 8, (1 << 25) + 8):
            with pytest.raises(occ.OccError) as e:
                occ.occ_gemm_plan_query(M, N, K)
            assert e.value.status == occ.OCC_EINVAL, (M, N, K)
            assert occ.occ_gemm_bt_plan_query(M, N, K)["kernel_id"] == 7, (M, N, K)


# Schedules in a row on the same buffers, as a program runs them: each pass has other
# operands, so a line of C left in some L2 by the pass before (or by the checks
# between them, which read C) would show in the sum.  One iteration per pass checks
# every output that is read; three check the last.  Every kernel with device-scope
# stores, wide and narrow rows, C of a few KiB and of several MiB, 1 to 8 terms.
@pytest.mark.parametrize("layout,variant,M,N,K,peers", [
    ("kn", 32, 2048, 2056, 64, 7), ("nk", 16, 2048, 2048, 72, 7), ("nk", 16, 264, 136, 64, 2), ("kn", 40, 1000, 1032, 64, 7),
    ("nk", 10, 520, 264, 128, 3), ("kn", 35, 1024, 1024, 64, 7), ("nk", 14, 264, 136, 72, 1), ("kn", 41, 264, 200, 72, 7),
    ("nk", 11, 1024, 1024, 64, 7), ("kn", 42, 200, 264, 136, 2), ("nk", 12, 1024, 1024, 128, 7), ("nk", 13, 64, 16384, 128, 7),
    ("kn", 43, 72, 136, 64, 7), ("nk", 17, 512, 1024, 136, 7), ("kn", 44, 512, 512, 200, 7), ("nk", 18, 72, 136, 64, 0),
    ("kn", 38, 512, 1024, 64, 7), ("nk", 25, 512, 1024, 64, 2), ("kn", 39, 512, 1024, 64, 7), ("nk", 9, 512, 1024, 64, 7),
    ("kn", 36, 72, 136, 64, 2), ("kn", 37, 512, 1024, 64, 7), ("nk", 6, 72, 136, 64, 2), ("nk", 7, 512, 1024, 64, 7),
    ("kn", 33, 16, 264, 136, 7), ("kn", 33, 16, 4096, 72, 7), ("kn", 33, 16, 28672, 64, 7), ("nk", 21, 8, 4096, 136, 7),
    ("nk", 34, 16, 4096, 1024, 7)])
def test_schedules_in_a_row_read_the_fresh_gemm_output(layout, variant, M, N, K, peers):
    g = torch.Generator(device=DEV).manual_seed(M + N + variant)
    ints = lambda lo, hi, *shape: torch.randint(lo, hi, shape, generator=g, device=DEV)
    B = ints(-2, 3, *((K, N) if layout == "kn" else (N, K))).to(torch.bfloat16)
    bufs = ints(-4, 5, peers, M * N).float()
    A = torch.empty((M, K), device=DEV, dtype=torch.bfloat16)
    C = torch.full((3, M, N), float("nan"), device=DEV, dtype=torch.bfloat16)
    out = torch.full((M * N,), float("nan"), device=DEV)
    ws = torch.zeros(occ.occ_overlap_workspace_bytes(3), dtype=torch.uint8, device=DEV)
    err = torch.zeros(1, dtype=torch.int32, device=DEV)
    comm = torch.cuda.Stream()
    for n in (1, 1, 3, 1):
        A.copy_(ints(-2, 3, M, K))
        # integer sums below 2^24: exact in fp32, rounded to bf16 once
        ref = (A.float() @ (B.float() if layout == "kn" else B.float().t())).to(torch.bfloat16)
        want = ref.float().reshape(-1) + bufs.sum(0)
        torch.cuda.synchronize()
        occ.occ_overlap_enqueue(A, B, C[:n], workspace=ws, comm_stream=comm, err=err, bufs=bufs, out=out, n_iter=n,
                                gemm_variant=variant, b_layout=layout, reduce_own=True)
        torch.cuda.synchronize()
        assert int(err.item()) == 0
        for i in range(n):
            assert torch.equal(C[i].view(torch.int16), ref.view(torch.int16)), (n, i)
        assert torch.equal(out, want), n
