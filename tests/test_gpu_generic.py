"""The generic kernel's loaders (16-byte reads of rows at any alignment, the turning loader of weights stored
K x N, element gathers where neither applies) and its groups of wavefronts that share a tile along k, at the sizes
where their edges lie."""
import numpy as np
import pytest

import oracle
from gpu_util import DT, DeviceConv, c_close, run_gemm, sample_rows
from paper_2104_09455_amd import binding as B
from paper_2104_09455_amd import workloads as wl

pytestmark = pytest.mark.gpu

# (M, N, K): rows shorter than 16 bytes, exactly 16 bytes, one element more; a k tile less / plus one; one, two and three
# columns (a group of four bytes is two fp16 or four int8 columns) and tile edges; few rows; the first k loops that groups
# share (five k tiles) with a whole and a cut last tile, and one whose last step leaves groups without a tile
EDGES = [(5, 9, 7), (9, 70, 4100), (33, 1, 8), (64, 2, 9), (17, 3, 15), (65, 4, 17), (31, 63, 63), (64, 64, 65), (70, 65, 127),
         (96, 130, 129), (66, 127, 257), (66, 127, 449), (40, 66, 513), (130, 70, 1025), (64, 200, 1100)]


@pytest.mark.parametrize("dtype", ["f16", "bf16", "i8"])
@pytest.mark.parametrize("layout", [B.B_NK, B.B_KN])
@pytest.mark.parametrize("shape", EDGES)
def test_edges_of_the_generic_loaders(shape, layout, dtype):
    M, N, K = shape
    A, Bm = wl.gemm_operands(M, N, K, dtype, seed=M * 131 + N * 17 + K, dist_a="normal", dist_b="normal")
    C_ref = oracle.gemm(A, Bm, dtype)
    for mode in (B.NONE, B.GLOBAL, B.THREAD):
        # (pads and an odd start move every row to another alignment)
        for pads in ((0, 0, 0, 0), (3, 1, 5, 1)):
            print("case", shape, layout, dtype, mode, pads, flush=True)
            r = run_gemm(A, Bm, dtype, mode, layout=layout, lda_pad=pads[0], ldb_pad=pads[1], ldc_pad=pads[2], misalign=pads[3],
                         use_beta=mode == B.GLOBAL)
            assert c_close(r.C, C_ref, dtype), (mode, pads)
            assert r.flag == 0, (mode, pads, r.report.worst_ratio)
            if mode != B.NONE:
                assert r.report.worst_ratio < 0.5


@pytest.mark.parametrize("dtype", ["f16", "i8"])
@pytest.mark.parametrize("mode", [B.GLOBAL, B.THREAD, B.TWOSIDED])
def test_faults_where_groups_share_a_tile_along_k(mode, dtype):
    """511-like odd sizes on the four-group tile: a fault in a group's running or finished partial accumulator, or in
    the added-up value, is seen, and C carries exactly that flip (int8)."""
    M, N, K = 75, 133, 1301
    dt = DT[dtype]
    A, Bm = wl.gemm_operands(M, N, K, dtype, seed=77, dist_a="normal", dist_b="normal")
    C_ref = oracle.gemm(A, Bm, dtype)
    assert B.abft_k_ways(M, N, K, dt, mode, False)[0] == 4
    ks = B.abft_tile_shape(M, N, K, dt, False)[2]
    parts = B.abft_k_parts(M, N, K, dt, mode, False)
    assert sorted(k for p in parts for k in p) == list(range(K))
    for t, k_after in enumerate([-1, -2, ks, 3 * ks, 4 * ks, (K - 1) // ks * ks]):
        i, j, bit = (13 * t + 5) % M, (29 * t + 60) % N, 30
        print("case", mode, dtype, k_after, i, j, flush=True)
        r = run_gemm(A, Bm, dtype, mode, layout=B.B_KN, inject=B.Fault(i, j, bit, k_after), want_report=False)
        assert r.flag == 1, k_after
        if dtype == "i8":
            if k_after == -2:
                bad = oracle.inject(A, Bm, C_ref, dtype, i, j, bit)
            else:
                bad = oracle.inject(A, Bm, C_ref, dtype, i, j, bit, k_after=k_after,
                                    k_set=parts[oracle.part_of(parts, (K if k_after < 0 else k_after) - 1)])
            assert np.array_equal(r.C, ((bad + 2 ** 31) % 2 ** 32) - 2 ** 31), k_after


# 64 x 64 and 128 x 128 tiles; k loops of whole 16-byte chunks that end inside a k tile (one chunk into it, one short of
# it), ragged rows and columns
ALIGNED = [(1900, 1100, 200, "G64"), (1900, 1100, 376, "G64"), (3000, 1000, 72, "G128"), (2997, 1003, 248, "G128")]


@pytest.mark.parametrize("dtype", ["f16", "bf16", "i8"])
@pytest.mark.parametrize("case", ALIGNED, ids=str)
def test_aligned_operands_take_the_general_path_s_results(case, dtype):
    """Aligned operands whose k loop is no whole number of k tiles have instances of the kernel of their own: bit for
    bit what the general ones store, and right."""
    M, N, K, kernel = case
    K = 2 * K if dtype == "i8" else K
    A, Bm = wl.gemm_operands(M, N, K, dtype, seed=M + K, dist_a="normal", dist_b="normal")
    rows = sample_rows(M, 400)
    C_ref = oracle.gemm(A[rows], Bm, dtype)
    for mode in (B.NONE, B.GLOBAL, B.THREAD, B.REPLICA, B.THREAD_HALF, B.TWOSIDED):
        print("case", case, dtype, mode, flush=True)
        assert {B.abft_kernel_name(M, N, K, DT[dtype], mode, al) for al in (True, False)} == {kernel}
        a = run_gemm(A, Bm, dtype, mode, use_beta=mode == B.GLOBAL)
        u = run_gemm(A, Bm, dtype, mode, misalign=1, use_beta=mode == B.GLOBAL)
        assert np.array_equal(a.C, u.C) and c_close(a.C[rows], C_ref, dtype), mode
        assert a.flag == 0 and u.flag == 0
        assert mode == B.NONE or (a.report.worst_ratio < 0.5 and a.report.tiles == u.report.tiles)


@pytest.mark.parametrize("dtype,conv,kernel", [
    ("f16", wl.Conv(8, 64, 63, 24, 48, 3, 3, 1, 1), "G128"), ("bf16", wl.Conv(20, 50, 44, 40, 150, 5, 5, 2, 2), "G64"),
    ("i8", wl.Conv(16, 28, 28, 96, 96, 3, 3, 1, 1), "G64")], ids=str)
def test_convolutions_of_whole_chunks(dtype, conv, kernel):
    """Channels that fill chunks but no k tiles: every scheme against the oracle."""
    d = DeviceConv(conv, dtype, seed=3)
    A = oracle.im2col(d.x, dtype, conv.KH, conv.KW, conv.stride, conv.pad)
    rows = sample_rows(d.M, 1500)
    C_ref = oracle.gemm(A[rows], d.Wm, dtype)
    for mode in (B.NONE, B.GLOBAL, B.THREAD, B.TWOSIDED):
        print("case", conv, dtype, mode, flush=True)
        assert B.abft_kernel_name(d.M, d.N, d.K, d.dt, mode, conv=True) == kernel
        flag, rep = d.run(mode)
        assert c_close(d.C(rows), C_ref, dtype) and flag == 0, mode
        assert mode == B.NONE or rep.worst_ratio < 0.5


# (M, N, K) on the 16 x 64 tile, the 64 x 64 tile alone and in four groups, the 128 x 128 tile: one k tile and less,
# a chunk's length, k loops that leave groups without a tile, and long ones
UNALIGNED = [(5, 70, 8), (16, 130, 63), (3, 300, 130), (9, 200, 2100), (70, 65, 16), (130, 66, 129), (66, 100, 257), (200, 300, 321),
             (511, 130, 1023), (2000, 1700, 77), (1900, 1701, 200)]


@pytest.mark.parametrize("dtype", ["f16", "bf16", "i8"])
@pytest.mark.parametrize("layout", [B.B_NK, B.B_KN], ids=["nk", "kn"])
@pytest.mark.parametrize("shape", UNALIGNED, ids=str)
def test_unaligned_operands_take_the_general_path_s_results(shape, layout, dtype):
    """Operands whose rows are contiguous have instances of the kernel with loaders of their own: bit for bit what the
    general one, which a planted fault goes through, stores everywhere but at the fault."""
    M, N, K = shape
    K = 2 * K if dtype == "i8" and K > 16 else K
    A, Bm = wl.gemm_operands(M, N, K, dtype, seed=M + N + K, dist_a="normal", dist_b="normal")
    rows = sample_rows(M, 300)
    C_ref = oracle.gemm(A[rows], Bm, dtype)
    i, j = M // 2, N - 1
    for mode in (B.NONE, B.GLOBAL, B.THREAD, B.REPLICA):
        print("case", shape, layout, dtype, mode, flush=True)
        for pads in (dict(misalign=1), dict(lda_pad=3, ldb_pad=1, ldc_pad=2)):
            r = run_gemm(A, Bm, dtype, mode, layout=layout, **pads)
            assert c_close(r.C[rows], C_ref, dtype) and r.flag == 0, mode
            assert mode == B.NONE or r.report.worst_ratio < 0.5
            bad = run_gemm(A, Bm, dtype, mode, layout=layout, inject=B.Fault(i, j, 30, -1), **pads)
            same = bad.C == r.C
            same[i, j] = True
            assert same.all() and bad.flag == (mode != B.NONE), mode


# the four-group tile in halves of 32 rows (at most 128 tiles of 64 x 64): rows that fill one half, both, a half and one row;
# the first grid that is no longer halved
HALVES = [(32, 64, 1100), (33, 65, 705), (64, 130, 1024), (97, 70, 4001), (1024, 512, 520), (1025, 512, 520)]


@pytest.mark.parametrize("dtype", ["f16", "i8"])
@pytest.mark.parametrize("layout", [B.B_NK, B.B_KN], ids=["nk", "kn"])
@pytest.mark.parametrize("shape", HALVES, ids=str)
def test_halved_tiles_keep_the_four_group_tile_s_results_and_comparisons(shape, layout, dtype):
    """Bit for bit what a planted fault's call, on whole tiles, stores everywhere but at the fault; as many comparisons."""
    M, N, K = shape
    A, Bm = wl.gemm_operands(M, N, K, dtype, seed=M + N, dist_a="normal", dist_b="normal")
    rows = sample_rows(M, 200)
    C_ref = oracle.gemm(A[rows], Bm, dtype)
    for mode in (B.NONE, B.THREAD, B.REPLICA):
        print("case", shape, layout, dtype, mode, flush=True)
        assert B.abft_kernel_name(M, N, K, DT[dtype], mode, False) == "G64K"
        r = run_gemm(A, Bm, dtype, mode, layout=layout, misalign=1)
        assert c_close(r.C[rows], C_ref, dtype) and r.flag == 0
        assert mode == B.NONE or (r.report.tiles == -(-M // 32) * -(-N // 32) and r.report.worst_ratio < 0.5)
        bad = run_gemm(A, Bm, dtype, mode, layout=layout, misalign=1, inject=B.Fault(M - 1, N - 1, 30, -2))
        same = bad.C == r.C
        same[M - 1, N - 1] = True
        assert same.all() and bad.flag == (mode != B.NONE)


# (M, N, K, pitch of A, of B, which operand's pitch is large): weights K x N of more than 2 GiB, whose k loops take several runs of
# 32-bit offsets (the last one cut) on every tile of the generic kernel; k loops far shorter than the k tile, on either side of the
# pitch where a k tile's offsets leave 31 bits; rows of A, of B whose tile does
WIDE = [("kn", 9, 70, 600, 600, 4_000_000), ("kn", 40, 66, 777, 777, 4_000_000), ("kn", 70, 130, 130, 130, 16_000_000),
        ("kn", 1500, 1400, 130, 131, 16_000_000), ("kn", 4, 9, 17, 17, 8_000_000), ("kn", 4, 9, 17, 17, 40_000_000),
        ("nk", 33, 40, 41, 35_000_000, 41), ("nk", 33, 40, 41, 41, 35_000_000), ("nk", 33, 40, 41, 30_000_000, 20_000_000)]


@pytest.mark.parametrize("dtype", ["f16", "i8"])
@pytest.mark.parametrize("case", WIDE, ids=str)
def test_pitches_beyond_32_bit_offsets(case, dtype):
    """Bit for bit what the operands without their pitches give; what lies between the rows is no number (int8: large)."""
    import torch
    from gpu_util import DEV, to_dev
    layout, M, N, K, lda, ldb = case
    A, Bm = wl.gemm_operands(M, N, K, dtype, seed=M + N, dist_a="normal", dist_b="normal")
    t, c_t, gap = (torch.int8, torch.int32, 77) if dtype == "i8" else (torch.float16, torch.float16, float("nan"))
    order, W = (B.B_NK, Bm.T) if layout == "nk" else (B.B_KN, Bm)

    def spread(x, pitch):
        rows, cols = x.shape
        buf = torch.full(((rows - 1) * pitch + cols,), gap, dtype=t, device=DEV)
        torch.as_strided(buf, (rows, cols), (pitch, 1)).copy_(to_dev(np.ascontiguousarray(x), dtype))
        return buf, pitch

    C_ref = oracle.gemm(A, Bm, dtype)
    flag = torch.zeros(1, dtype=torch.int32, device=DEV)
    stored = {}
    for a_pitch, b_pitch in ((K + 1, W.shape[1] + 1), (lda, ldb)):
        (dA, a_pitch), (dB, b_pitch) = spread(A, a_pitch), spread(W, b_pitch)
        for mode in (B.NONE, B.GLOBAL, B.THREAD):
            print("case", case, dtype, mode, a_pitch, b_pitch, flush=True)
            need = max(B.abft_workspace_bytes(M, N, K, DT[dtype], mode), 256)
            ws = torch.zeros(need, dtype=torch.uint8, device=DEV)
            C = torch.zeros((M, N), dtype=c_t, device=DEV)
            B.abft_gemm(M, N, K, dA, a_pitch, dB, b_pitch, order, C, N, DT[dtype], mode, workspace=ws, workspace_bytes=need, fault_flag=flag)
            torch.cuda.synchronize()
            assert int(flag.item()) == 0
            assert torch.equal(C, stored.setdefault(mode, C))
        del dA, dB
    got = stored[B.THREAD].cpu().numpy()
    assert c_close(got.astype(np.int64) if dtype == "i8" else got.astype(np.float64), C_ref, dtype)


# (M, N, K in bytes): one chunk, the whole k tile, between; one tile and one row or column more, many tiles more wide than high
# and more high than wide
SHALLOW = [(17, 1, 16), (64, 64, 128), (65, 63, 18), (33, 130, 58), (41, 157, 34), (129, 200, 112), (700, 70, 126), (70, 1500, 98), (488, 276, 106)]


@pytest.mark.parametrize("dtype", ["f16", "bf16", "i8"])
@pytest.mark.parametrize("shape", SHALLOW, ids=str)
def test_products_of_one_k_tile_straight_from_memory_are_those_of_the_tile_in_lds(shape, dtype):
    """Rows of 16 to 128 bytes, unprotected and thread-level, go without LDS; a planted fault's call does not: the same
    elements bit by bit, as many comparisons, and NaN in an input is flagged."""
    M, N, K = shape[0], shape[1], shape[2] // (1 if dtype == "i8" else 2)
    A, Bm = wl.gemm_operands(M, N, K, dtype, seed=M + N + K, dist_a="normal", dist_b="normal")
    C_ref = oracle.gemm(A, Bm, dtype)
    i, j = M - 1, N - 1
    for mode in (B.NONE, B.THREAD):
        for kw in (dict(misalign=1), dict(lda_pad=3, ldb_pad=1, ldc_pad=5, want_report=False)):
            assert B.abft_kernel_name(M, N, K, DT[dtype], mode, False) == "G64"
            print("case", shape, dtype, mode, kw, flush=True)
            r = run_gemm(A, Bm, dtype, mode, **kw)
            assert c_close(r.C, C_ref, dtype) and r.flag == 0
            bad = run_gemm(A, Bm, dtype, mode, inject=B.Fault(i, j, 30, -1), **kw)
            if r.report and mode != B.NONE:
                assert r.report.tiles == bad.report.tiles == -(-M // 32) * -(-N // 32) and r.report.worst_ratio == 0.0
            same = bad.C == r.C
            same[i, j] = True
            assert same.all() and bad.flag == (mode != B.NONE)
            if dtype != "i8":
                lost = A.copy()
                lost[i, K - 1] = np.float16("nan") if dtype == "f16" else 0x7fc0
                assert run_gemm(lost, Bm, dtype, mode, **kw).flag == (mode != B.NONE)
