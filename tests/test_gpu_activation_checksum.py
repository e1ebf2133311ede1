"""The pass over A of the global scheme (activation checksum and its dot products with the weight checksums) where its edges
lie: rows shorter than a 16-byte chunk, of exactly one, cut inside one, up to and past the k range of a workgroup; row blocks
that end inside and at the end of the rows that are on their way together; more column blocks than lanes."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import DEV, DT, run_gemm, to_dev
from paper_2104_09455_amd import binding as B
from paper_2104_09455_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f16", "bf16", "i8"])
def test_column_sums(dtype):
    """Sums of the columns of A, exactly: int8 in int64; fp16 / bf16 values between 2^-24 and 8 add up in fp64 without rounding."""
    chunk = 16 if dtype == "i8" else 8
    wide = torch.int64 if dtype == "i8" else torch.float64
    for K in (1, 3, chunk - 1, chunk, chunk + 1, 2 * chunk - 1, 3 * chunk, 32 * chunk - 1, 32 * chunk, 32 * chunk + 1, 70 * chunk + 5):
        for M in (1, 7, 31, 32, 33, 64, 65, 97, 700):
            for pad, shift in ((0, 0), (3, 1)):
                print("case", dtype, M, K, pad, shift, flush=True)
                A = wl.random_matrix((M, K), dtype, "int8" if dtype == "i8" else "normal", M + K)
                buf = np.zeros(M * (K + pad) + shift, dtype=A.dtype)
                buf[shift:].reshape(M, K + pad)[:, :K] = A
                d = to_dev(buf, dtype)
                alpha = torch.full((K + 1,), 77, dtype=wide, device=DEV)
                B.abft_activation_checksum(M, K, d.data_ptr() + shift * A.itemsize, K + pad, DT[dtype], alpha)
                torch.cuda.synchronize()
                want = oracle.widen(A, dtype).sum(axis=0)
                got = alpha.cpu().numpy()
                assert np.array_equal(got[:K], want) and got[K] == 77


@pytest.mark.parametrize("dtype", ["f16", "i8"])
@pytest.mark.parametrize("shape", [(5, 70, 15), (3, 40, 1), (1, 33, 16), (16, 300, 255), (33, 2150, 17), (97, 130, 513), (65, 66, 511),
                                   (129, 100, 1025), (64, 2200, 512), (2000, 1700, 77), (1900, 1601, 300)], ids=str)
def test_dot_products_with_the_weight_checksums(shape, dtype):
    """A clean product passes (int8: every tile's two sides are equal), a planted fault does not."""
    M, N, K = shape
    A, Bm = wl.gemm_operands(M, N, K, dtype, seed=M + N + K, dist_a="normal", dist_b="normal")
    for layout in (B.B_NK, B.B_KN):
        for use_beta in (False, True):
            print("case", shape, dtype, layout, use_beta, flush=True)
            r = run_gemm(A, Bm, dtype, B.GLOBAL, layout=layout, misalign=1, use_beta=use_beta)
            assert r.flag == 0 and (r.report.worst_ratio == 0 if dtype == "i8" else r.report.worst_ratio < 0.5)
            r = run_gemm(A, Bm, dtype, B.GLOBAL, layout=layout, misalign=1, use_beta=use_beta, inject=B.Fault(M - 1, N - 1, 30, -1))
            assert r.flag == 1
