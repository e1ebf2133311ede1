"""C's edges, activation and leading dimensions on the tiles whose lanes hold adjacent columns: two or four columns per lane
are stored at once wherever C's rows start, fewer where N cuts them; nothing outside C is written, and a fault lands in the
element it names."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import DEV, DT, c_close, c_to_host, to_dev
from paper_2104_09455_amd import binding as B
from paper_2104_09455_amd import workloads as wl

pytestmark = pytest.mark.gpu
# (M, N, K) on each tile: columns that end inside a wavefront tile and at its edge
CASES = {
    "F256W": (3585, 4097, 128), "F256N": (2049, 2240, 512), "F256S": (65571, 60, 512), "F128E": (1150, 2056, 512),
    "F128": (2300, 2190, 256), "F128T": (16400, 100, 128), "F64T": (3000, 390, 384), "R64": (131105, 130, 64),
}


@pytest.mark.parametrize("dtype", ["f16", "bf16", "i8"])
@pytest.mark.parametrize("name", sorted(CASES))
def test_edges_and_leading_dimensions(name, dtype):
    M, N, K = CASES[name]
    dt = DT[dtype]
    K = 2 * K if dtype == "i8" else K    # (the same bytes)
    A, Bm = wl.gemm_operands(M, N, K, dtype, seed=M + N, dist_a="int8" if dtype == "i8" else "normal",
                             dist_b="int8" if dtype == "i8" else "normal")
    dA, dB = to_dev(A, dtype), to_dev(np.ascontiguousarray(Bm.T), dtype)
    rows = np.unique(np.r_[0:40, 120:136, M // 2:M // 2 + 70, M - 70:M])
    C_ref = oracle.gemm(A[rows], Bm, dtype)
    t = {"f16": torch.float16, "bf16": torch.bfloat16, "i8": torch.int32}[dtype]
    flag = torch.zeros(1, dtype=torch.int32, device=DEV)
    seen = set()
    for mode in (B.NONE, B.THREAD):
        seen.add(B.abft_kernel_name(M, N, K, dt, mode))
        for pad, shift in ((0, 0), (1, 0), (2, 0), (4, 0), (8, 1), (8, 2), (8, 4)):
            print("case", name, dtype, mode, pad, shift, flush=True)
            ldc = -(-N // 8) * 8 + pad
            buf = torch.full((M * ldc + 16,), 77, dtype=t, device=DEV)
            C = buf[shift:shift + M * ldc].view(M, ldc)
            B.abft_gemm(M, N, K, dA, K, dB, K, B.B_NK, C, ldc, dt, mode, fault_flag=flag)
            torch.cuda.synchronize()
            got = C[torch.as_tensor(rows, device=DEV)][:, :N].contiguous()
            assert c_close(c_to_host(got, dtype), C_ref, dtype), (mode, pad, shift)
            assert bool((C[:, N:] == 77).all()) and bool((buf[:shift] == 77).all()) and bool((buf[shift + M * ldc:] == 77).all())
            assert int(flag.item()) == 0
            if pad == 0 and shift == 0:
                whole = C[:, :N].clone()
            assert C[:, :N].equal(whole)
    # a flipped top bit of a finished accumulator changes that element and no other
    for i, j in ((0, 1), (M - 1, N - 1), (M // 2, N // 3)):
        C = torch.zeros((M, N), dtype=t, device=DEV)
        B.abft_gemm(M, N, K, dA, K, dB, K, B.B_NK, C, N, dt, B.THREAD, fault_flag=flag, inject=B.Fault(i, j, 31, -1))
        torch.cuda.synchronize()
        assert [tuple(x) for x in (C != whole).nonzero().tolist()] == [(i, j)]
    print("tiles", name, seen, flush=True)
    assert name in seen or (dtype == "i8" and name == "R64")


@pytest.mark.parametrize("dtype", ["f16", "bf16", "i8"])
@pytest.mark.parametrize("name", sorted(CASES))
def test_columns_that_cut_a_lane_s_run(name, dtype):
    """One, two or three of the columns that a lane holds inside C, rows that end inside its rows, at any alignment of C's
    rows: what the larger product has there, bit for bit, and nothing written beside it."""
    M, N, K = CASES[name]
    N += 4 if name == "R64" else 0    # (more than 128 columns, also when cut)
    dt = DT[dtype]
    K = 2 * K if dtype == "i8" else K
    A, Bm = wl.gemm_operands(M, N, K, dtype, seed=M + N, dist_a="int8" if dtype == "i8" else "normal",
                             dist_b="int8" if dtype == "i8" else "normal")
    dA, dB = to_dev(A, dtype), to_dev(np.ascontiguousarray(Bm.T), dtype)
    t = {"f16": torch.float16, "bf16": torch.bfloat16, "i8": torch.int32}[dtype]
    flag = torch.zeros(1, dtype=torch.int32, device=DEV)
    seen = set()
    for mode in (B.NONE, B.THREAD):
        ref = torch.zeros((M, N), dtype=t, device=DEV)
        B.abft_gemm(M, N, K, dA, K, dB, K, B.B_NK, ref, N, dt, mode, fault_flag=flag)
        for cut, pad, shift in ((1, 0, 0), (2, 3, 1), (3, 0, 3), (3, 6, 2)):
            m, n = M - 5 * cut, N - cut
            ldc = n + pad
            print("case", name, dtype, mode, m, n, K, ldc, shift, flush=True)
            assert B.abft_kernel_name(m, n, K, dt, mode) == B.abft_kernel_name(M, N, K, dt, mode)
            seen.add(B.abft_kernel_name(m, n, K, dt, mode))
            buf = torch.full((m * ldc + 16,), 77, dtype=t, device=DEV)
            C = buf[shift:shift + m * ldc].view(m, ldc)
            B.abft_gemm(m, n, K, dA, K, dB, K, B.B_NK, C, ldc, dt, mode, fault_flag=flag)
            torch.cuda.synchronize()
            assert C[:, :n].equal(ref[:m, :n]), (mode, cut)
            assert bool((C[:, n:] == 77).all()) and bool((buf[:shift] == 77).all()) and bool((buf[shift + m * ldc:] == 77).all())
    assert int(flag.item()) == 0 and (name in seen or (dtype == "i8" and name == "R64"))


@pytest.mark.parametrize("shape", [(250, 4000, 256), (70, 3000, 256), (1, 1500, 512), (1900, 2500, 256), (2500, 1900, 256),
                                   (300, 1100, 257), (1100, 300, 257), (5, 1000, 131), (2100, 2200, 130), (2200, 2100, 130)], ids=str)
@pytest.mark.parametrize("layout", [B.B_NK, B.B_KN])
def test_every_tile_once_whatever_their_number(shape, layout):
    """Numbers of tiles that 8 does and does not divide, more tile columns than rows and the reverse: all of C is written,
    exactly (int8)."""
    M, N, K = shape
    A, Bm = wl.gemm_operands(M, N, K, "i8", seed=M + N, dist_a="int8", dist_b="int8")
    W = np.ascontiguousarray(Bm.T) if layout == B.B_NK else Bm
    dA, dB = to_dev(A, "i8"), to_dev(W, "i8")
    flag = torch.zeros(1, dtype=torch.int32, device=DEV)
    C_ref = oracle.gemm(A, Bm, "i8")
    for mode in (B.NONE, B.THREAD):
        print("case", shape, layout, mode, flush=True)
        C = torch.full((M, N), -7, dtype=torch.int32, device=DEV)
        B.abft_gemm(M, N, K, dA, K, dB, W.shape[1], layout, C, N, B.I8, mode, fault_flag=flag)
        torch.cuda.synchronize()
        assert np.array_equal(C.cpu().numpy(), C_ref) and int(flag.item()) == 0


CONVS = {
    "R64 one tap": wl.Conv(2700, 7, 7, 64, 64, 3, 3, 1, 1), "R64 taps": wl.Conv(36, 123, 121, 32, 64, 2, 2, 2, 0),
    "strips of pixels": wl.Conv(45, 54, 55, 64, 64, 3, 3, 1, 1), "strips of runs": wl.Conv(12, 215, 214, 3, 64, 7, 7, 2, 3),
}


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("name", sorted(CASES) + sorted(CONVS))
def test_relu_of_every_tile(name, dtype):
    """ReLU as C is stored: what is stored without it, and zeros for its negative values, bit for bit, with and without checks
    (the checks read the accumulators before; without them the activation is the first to).  A signalling NaN (the top exponent bit
    of a value between 1 and 1.5 flipped) stores 0, as any NaN."""
    dt = DT[dtype]
    t = {"f16": torch.float16, "bf16": torch.bfloat16}[dtype]
    if name in CASES:
        M, N, K = CASES[name]
        c, geo = None, B.Conv()
        x, w = wl.random_matrix((M, K), dtype, "normal", 5), wl.random_matrix((N, K), dtype, "normal", 6)
    else:
        c = CONVS[name]
        geo = B.Conv(c.batch, c.H, c.W, c.Cin, c.KH, c.KW, c.stride, c.pad)
        M, N, K = c.batch * c.OH * c.OW, c.Cout, c.KH * c.KW * c.Cin
        x, w = wl.random_matrix((c.batch * c.H * c.W, c.Cin), dtype, "normal", 5), wl.random_matrix((N, K), dtype, "normal", 6)
    dx, dw = to_dev(x, dtype), to_dev(w, dtype)
    plan = B.abft_plan_create([B.Layer(M, N, K, dt, B.B_NK, 0 if c is None else 1, geo, dw.data_ptr(), K)])
    flag = torch.zeros(1, dtype=torch.int32, device=DEV)

    def run(mode, act, fault=None):
        C = torch.full((M, N), 77, dtype=t, device=DEV)
        flag.zero_()
        B.abft_plan_set_mode(plan, 0, mode)
        B.abft_plan_set_activation(plan, 0, act)
        B.abft_plan_set_diagnostics(plan, 0, None, fault)
        B.abft_plan_run(plan, 0, dx, K, C, N, flag)
        torch.cuda.synchronize()
        return C, int(flag.item())

    for mode in (B.NONE, B.THREAD, B.GLOBAL):
        print("case", name, dtype, mode, flush=True)
        plain, f0 = run(mode, B.ACT_NONE)
        act, f1 = run(mode, B.ACT_RELU)
        assert f0 == 0 and f1 == 0 and bool((plain < 0).any())
        assert act.equal(torch.where(plain > 0, plain, torch.zeros_like(plain)))
        i, j = ((plain > 1.02) & (plain < 1.48)).nonzero()[7].tolist()
        bad, f = run(mode, B.ACT_RELU, B.Fault(i, j, 30, -1))
        assert f == (mode != B.NONE) and float(bad[i, j]) == 0
        bad[i, j] = act[i, j]
        assert bad.equal(act)
    # sums beyond the range of the output type, and (bf16) of the accumulators, of either sign
    dx[0] = 0
    dx[0, 0] = 60000.0 if dtype == "f16" else 3.0e38
    plain, _ = run(B.NONE, B.ACT_NONE)
    act, _ = run(B.NONE, B.ACT_RELU)
    assert bool((plain == float("inf")).any()) and bool((plain == -float("inf")).any())
    assert act.equal(torch.where(plain > 0, plain, torch.zeros_like(plain)))
    B.abft_plan_destroy(plan)
