"""Eight wavefronts sharing a 32 x 32 tile along k (few tiles, long k loops): whole and short last k tiles, k loops
that leave some wavefronts a tile less, ragged outputs, convolutions, every scheme, a fault in each share."""
import numpy as np
import pytest

import oracle
from gpu_util import DT, DeviceConv, c_close, run_gemm
from paper_2104_09455_amd import binding as B
from paper_2104_09455_amd import workloads as wl

pytestmark = pytest.mark.gpu

# K in bytes of fp16 / int8: whole k tiles (32 of them, the fewest; 33), a short last tile of one and of seven chunks
SHAPES = [(49, 512, 32), (33, 40, 33), (1, 100, 32.125), (96, 257, 40.875)]


@pytest.mark.parametrize("dtype", ["f16", "bf16", "i8"])
@pytest.mark.parametrize("shape", SHAPES)
def test_eight_shares_of_a_long_k_loop(shape, dtype):
    M, N, tiles = shape
    K = int(tiles * 128) // (1 if dtype == "i8" else 2)
    dt = DT[dtype]
    A, Bm = wl.gemm_operands(M, N, K, dtype, seed=M + N, dist_a="uniform_01", dist_b="weights")
    C_ref = oracle.gemm(A, Bm, dtype)
    modes = [B.NONE, B.GLOBAL, B.THREAD, B.REPLICA, B.THREAD_HALF, B.TWOSIDED] + ([B.GLOBAL_WEIGHTED] if dtype != "bf16" else [])
    for mode in modes:
        print("case", shape, dtype, mode, flush=True)
        r = run_gemm(A, Bm, dtype, mode, use_beta=mode in (B.GLOBAL, B.GLOBAL_WEIGHTED))
        assert c_close(r.C, C_ref, dtype) and r.flag == 0, mode
        if mode == B.NONE:
            continue
        assert r.report.worst_ratio < 0.5 and r.report.tiles == -(-M // 32) * -(-N // 32)
        parts = B.abft_k_parts(M, N, K, dt, mode)
        assert len(parts) == 8 and sorted(k for p in parts for k in p) == list(range(K))
        ks = B.abft_tile_shape(M, N, K, dt)[2]
        # the finished value, the last share's finished partial sum, and every share's running one
        for t, k_after in enumerate([-2, -1] + [ks * (w + 1) for w in range(8)]):
            i, j = (13 * t + 3) % M, (29 * t + 7) % N
            bad = run_gemm(A, Bm, dtype, mode, inject=B.Fault(i, j, 30, k_after), want_report=False)
            assert bad.flag == 1, (mode, k_after)
            if dtype == "i8":
                kw = {} if k_after == -2 else dict(k_after=k_after, k_set=parts[oracle.part_of(parts, (K if k_after < 0 else k_after) - 1)])
                want = oracle.inject(A, Bm, C_ref, dtype, i, j, 30, **kw)
                assert np.array_equal(bad.C, ((want + 2 ** 31) % 2 ** 32) - 2 ** 31), (mode, k_after)


@pytest.mark.parametrize("dtype", ["f16", "bf16", "i8"])
@pytest.mark.parametrize("conv", [wl.Conv(1, 7, 7, 512, 96, 3, 3, 1, 1), wl.Conv(2, 9, 8, 464, 40, 3, 3, 2, 1)], ids=str)
def test_convolutions_with_long_k_loops(conv, dtype):
    d = DeviceConv(conv, dtype, seed=9)
    A = oracle.im2col(d.x, dtype, conv.KH, conv.KW, conv.stride, conv.pad)
    C_ref = oracle.gemm(A, d.Wm, dtype)
    assert B.abft_k_ways(d.M, d.N, d.K, d.dt, B.THREAD)[0] == 8
    for mode in (B.NONE, B.GLOBAL, B.THREAD):
        print("case", conv, dtype, mode, flush=True)
        flag, rep = d.run(mode)
        assert c_close(d.C(), C_ref, dtype) and flag == 0, mode
        assert mode == B.NONE or rep.worst_ratio < 0.5
