"""Products of at most sixteen rows, whose 16-column workgroups share the k loop over eight wavefronts: edges of rows,
columns, k tiles and chunks, rows at any alignment, every wavefront-level scheme, with a report and without."""
import math

import numpy as np
import pytest

import oracle
from gpu_util import DT, c_close, run_gemm
from paper_2104_09455_amd import binding as B
from paper_2104_09455_amd import workloads as wl

pytestmark = pytest.mark.gpu

# (M, N, K in 16-byte chunks, elements more): one chunk, a part of a k tile, one, one per wavefront and one more, two (the most
# that is in flight at once) and a part of a third, the k loops in which one, seven and all wavefronts take the loop without
# conditions (their fifth own tile: 33, 39, 40 k tiles, the last one whole or cut), longer ones, by an odd number of tiles too
SHAPES = [(1, 1, 1, 0), (16, 16, 8, 0), (3, 17, 3, 0), (16, 33, 9, 0), (8, 24, 8 * 8, 0), (8, 24, 8 * 9, 0), (5, 40, 8 * 16, 0), (16, 100, 8 * 17 + 3, 0),
          (16, 34, 8 * 32, 0), (16, 34, 8 * 33, 0), (5, 18, 8 * 32 + 1, 0), (11, 40, 8 * 39, 0), (16, 16, 8 * 39 + 7, 0), (2, 31, 8 * 64, 0),
          (16, 16, 8 * 129, 0), (7, 70, 8 * 300 + 5, 0),
          (1, 512, 1, 5), (16, 15, 8, 1), (4, 65, 15, 7), (16, 48, 8 * 16, 3), (16, 34, 8 * 32, 1), (3, 20, 8 * 33, 5), (16, 17, 8 * 39 + 7, 7),
          (9, 33, 8 * 129, 1), (16, 20, 8 * 160 + 7, 7)]


@pytest.mark.parametrize("dtype", ["f16", "bf16", "i8"])
@pytest.mark.parametrize("shape", SHAPES)
def test_every_scheme_at_the_edges(shape, dtype):
    M, N, chunks, more = shape
    K = chunks * (16 if dtype == "i8" else 8) + more
    A, Bm = wl.gemm_operands(M, N, K, dtype, seed=M + N, dist_a="uniform_01", dist_b="weights")
    C_ref = oracle.gemm(A, Bm, dtype)
    aligned = more == 0
    ways = {}
    for mode in (B.NONE, B.THREAD, B.REPLICA, B.THREAD_HALF, B.TWOSIDED):
        for kw in (dict(), dict(want_report=False), dict(want_report=False, lda_pad=8, ldb_pad=16, ldc_pad=3), dict(misalign=1)):
            print("case", shape, dtype, mode, kw, flush=True)
            r = run_gemm(A, Bm, dtype, mode, **kw)
            assert c_close(r.C, C_ref, dtype) and r.flag == 0
            if not kw.get("misalign"):
                ways.setdefault(mode, []).append(r.C)
            if mode != B.NONE and not kw:
                tm, tn, _ = B.abft_tile_shape(M, N, K, DT[dtype], aligned)
                assert r.report.tiles == math.ceil(M / tm) * math.ceil(N / tn) and r.report.worst_ratio == 0.0
    # one result, whatever the scheme and whether a report is asked for
    for got in ways.values():
        assert all(np.array_equal(np.asarray(g).view(np.uint8), np.asarray(ways[B.NONE][0]).view(np.uint8)) for g in got)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("K", [64, 1000, 1003])
def test_what_is_no_number_is_flagged_and_nothing_outside_c_is_touched(K, dtype):
    import torch
    t = {"f16": torch.float16, "bf16": torch.bfloat16}[dtype]
    gen = torch.Generator(device="cuda:0").manual_seed(K)
    M, N, ldc = 9, 41, 50
    A, W = (torch.randn(s, device="cuda:0", generator=gen).to(t) for s in ((M, K), (N, K)))
    flag = torch.zeros(1, dtype=torch.int32, device="cuda:0")
    for value, want in ((None, 0), (float("nan"), 1), (float("inf"), 1), (-3e38 if dtype == "bf16" else -float("inf"), 1)):
        A2 = A.clone()
        if value is not None:
            A2[8, K - 1] = value
        C = torch.full((M + 2, ldc), 77, dtype=t, device="cuda:0")
        flag.zero_()
        B.abft_gemm(M, N, K, A2, K, W, K, B.B_NK, C[1:], ldc, DT[dtype], B.THREAD, fault_flag=flag)
        torch.cuda.synchronize()
        assert int(flag.item()) == want, value
        assert bool((C[0] == 77).all()) and bool((C[M + 1] == 77).all()) and bool((C[:, N:] == 77).all())
        ref = A2[:8].float() @ W.float().t()
        assert torch.allclose(C[1:9, :N].float(), ref, rtol=1e-2, atol=1e-2 * float(ref.square().mean().sqrt()))


@pytest.mark.parametrize("dtype", ["f16", "i8"])
def test_layers_of_few_rows_share_a_launch_at_any_alignment(dtype):
    """Aligned rows, rows of thirteen values and a single column in one launch: bit by bit what they give alone."""
    import torch
    from test_gpu_shared_launch import Pass
    for mode in (B.NONE, B.THREAD):
        p = Pass(dtype, mode)
        # (rows of one k tile, 16 to 128 bytes, of many columns: by themselves on the 16 x 64 tile)
        for M, N, K in ((1, 512, 32), (16, 40, 29), (16, 1, 256), (7, 1024, 1040), (3, 96, 4096), (16, 33, 8400),
                        (16, 5000, 17), (2, 7001, 61), (11, 20, 128 if dtype == "i8" else 63)):
            p.add((M, N, K), p.rnd(M, K), p.out(M, N, pad=N % 3), relu=N == 40)
        p.both_ways(shared=1)
    assert torch.cuda.is_available()


# a tiling of four shares (32 x 32 streaming tiles, the four-group tile), of eight, of one (16 x 64): aligned rows, rows at multiples of
# four bytes, rows at any address
FAULTS = [(16, 100, 1920, "S32", 4), (3, 33, 1000, "S32", 4), (16, 40, 8192, "S32W", 8), (9, 64, 4096 + 16, "S32W", 8),
          (9, 70, 2050, "G64K", 4), (16, 33, 4099, "G64K", 4), (7, 40, 402, "G16", 1), (16, 70, 211, "G16", 1)]


@pytest.mark.parametrize("dtype", ["f16", "bf16", "i8"])
@pytest.mark.parametrize("shape", FAULTS, ids=str)
def test_a_planted_fault_changes_its_element_and_no_other_and_is_seen(shape, dtype):
    """Faults of every kind run on the kernel of the call without one: every other element is that call's bit by bit, int8
    carries exactly the flip of the sum that the tiling's shares make of it, and the flag is raised with a report and without."""
    M, N, K, name, ways = shape
    K = 2 * K + K % 2 if dtype == "i8" else K
    A, Bm = wl.gemm_operands(M, N, K, dtype, seed=M + N + K, dist_a="normal", dist_b="normal")
    C_ref = oracle.gemm(A, Bm, dtype)
    aligned = name[0] == "S"
    ks = B.abft_tile_shape(M, N, K, DT[dtype], aligned)[2]
    last = (K - 1) // ks * ks
    rng = np.random.default_rng(K)
    for mode in (B.NONE, B.THREAD, B.REPLICA, B.THREAD_HALF, B.TWOSIDED):
        assert B.abft_kernel_name(M, N, K, DT[dtype], mode, aligned) == name
        parts = B.abft_k_parts(M, N, K, DT[dtype], mode, aligned)
        assert len(parts) == ways
        for report in (False, True) if mode != B.NONE else (False,):
            kw = dict(want_report=report, misalign=K % 2 if dtype == "i8" else 0)
            clean = run_gemm(A, Bm, dtype, mode, **kw)
            assert c_close(clean.C, C_ref, dtype) and clean.flag == 0
            for k_after in (-1, -2, ks, 6 * ks if 6 * ks < K else ks, last):
                i, j = int(rng.integers(M)), int(rng.integers(N))
                print("case", shape, dtype, mode, report, k_after, i, j, flush=True)
                bad = run_gemm(A, Bm, dtype, mode, inject=B.Fault(i, j, 30, k_after), **kw)
                same = bad.C == clean.C
                assert not same[i, j]
                same[i, j] = True
                assert same.all() and bad.flag == (mode != B.NONE), (mode, report, k_after)
                if dtype == "i8":
                    part = {} if k_after == -2 else dict(k_after=k_after, k_set=parts[oracle.part_of(parts, (K if k_after < 0 else k_after) - 1)])
                    want = oracle.inject(A, Bm, C_ref, dtype, i, j, 30, **part)
                    assert np.array_equal(bad.C, ((want + 2 ** 31) % 2 ** 32) - 2 ** 31), (mode, report, k_after)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("K,misalign", [(256, 0), (4096, 0), (2050, 0), (4099, 1)])
def test_the_verdict_does_not_depend_on_a_report(K, misalign, dtype):
    """Sixteen columns of small sums beside sixteen of large ones: a fault among the small ones that is beyond the tolerance of
    its own columns and within that of all 32 raises the flag with a report (whose ratio says so) and without."""
    M, N = 11, 64
    assert B.abft_tile_shape(M, N, K, DT[dtype], K % 8 == 0)[1] == 32
    A, Bm = wl.gemm_operands(M, N, K, dtype, seed=K, dist_a="uniform_01", dist_b="uniform_01")
    large = np.ones(N, dtype=bool)
    large[32:48] = False
    # (times 32: exact in both types, whose values here are all normal numbers or zero)
    Bm[:, large] = Bm[:, large] * np.float16(32) if dtype == "f16" else np.where(Bm[:, large] != 0, Bm[:, large] + (5 << 7), 0)
    C_ref = oracle.gemm(A, Bm, dtype)
    i, j = M - 2, 37
    seen = set()
    for bit in range(2, 23):
        C_bad = oracle.inject(A, Bm, C_ref, dtype, i, j, bit)
        own, both = (oracle.tile_check(A, Bm, C_bad, dtype, 0, M, c0, c1) for c0, c1 in ((32, 48), (32, 64)))
        beyond = abs(own.residual) >= 2 * own.tau
        within = abs(own.residual) <= own.tau / 2
        if not (beyond or within) or (beyond and abs(both.residual) > both.tau / 2):
            continue
        print("case", K, misalign, dtype, bit, own.residual, own.tau, both.tau, flush=True)
        seen.add(beyond)
        for report in (False, True):
            r = run_gemm(A, Bm, dtype, B.THREAD, misalign=misalign, want_report=report, inject=B.Fault(i, j, bit, -2))
            assert r.flag == beyond, (bit, report)
            if report:
                assert (r.report.worst_ratio > 1) == beyond
    assert True in seen
