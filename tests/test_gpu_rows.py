"""The row-streaming kernel (very many rows, weights resident in LDS; unprotected and wavefront-level schemes) at
the edges of its range: one and several k tiles, fewer k tiles than are loaded ahead and more, one and several column
blocks, rows and columns that fill no tile, leading dimensions that rule out wide stores, convolutions whose rows
wrap over several images."""
import numpy as np
import pytest

import oracle
from gpu_util import DT, DeviceConv, DeviceGemm, c_close, edge_rows, run_gemm, sample_rows
from paper_2104_09455_amd import binding as B
from paper_2104_09455_amd import workloads as wl

pytestmark = pytest.mark.gpu

WAVE = [B.NONE, B.THREAD, B.REPLICA, B.THREAD_HALF, B.TWOSIDED]
# (M, N, K): a single k tile with 1, 4 and 20 (all of LDS) column blocks; 2, 3, 4 (as many as are loaded ahead), 5, 9
# and 20 k tiles; ragged rows and columns
SHAPES = [(131072, 64, 64), (131105, 256, 64), (131104, 1280, 64), (131536, 64, 128), (131072, 40, 192),
          (131081, 64, 256), (131072, 64, 320), (131072, 64, 576), (131103, 33, 1280)]
# those of them that run on it unprotected too
UNPROTECTED = [(131105, 256, 64), (131104, 1280, 64), (131536, 64, 128), (131072, 40, 192), (131081, 64, 256)]


def _huge_flip(A, Bm, dtype, i, j, k_after):
    """The exponent bit whose flip makes the accumulator of (i, j) astronomically large."""
    real = wl.bf16_bits_to_f32 if dtype == "bf16" else (lambda x: x.astype(np.float64))
    k = A.shape[1] if k_after < 0 else k_after
    return 30 if abs(float(real(A[i, :k]) @ real(Bm[:k, j]))) < 2 else 29


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("shape", SHAPES)
def test_products_of_very_many_rows(shape, dtype):
    M, N, K = shape
    d = DeviceGemm(M, N, K, dtype, seed=M + N + K)
    assert (d.tm, d.tn, d.k_step) == (32, 64, 64)
    rows = sample_rows(M, 3000)
    C_ref = oracle.gemm(d.A[rows], d.Bm, dtype)
    rng = np.random.default_rng(K)
    for mode in WAVE:
        print("case", shape, dtype, mode, flush=True)
        d.dC.fill_(7.0)
        flag, rep = d.run(mode)
        assert c_close(d.C(rows), C_ref, dtype) and flag == 0, mode
        kernel = B.abft_kernel_name(M, N, K, d.dt, mode)
        if mode == B.NONE:
            assert (kernel == "R64") == (shape in UNPROTECTED)
            continue
        assert kernel == "R64"
        if mode == B.THREAD:
            whole = d.dC.clone()
        assert d.dC.equal(whole)     # (every wavefront-level scheme stores the same product)
        assert rep.worst_ratio < 0.5 and rep.tiles == -(-M // 32) * -(-N // 64)
        # a fault anywhere in a finished or running accumulator is seen: first and last tile, a tile in between
        for i, j, k_after in [(0, 0, -1), (M - 1, N - 1, -1), (int(rng.integers(M)), int(rng.integers(N)), -2),
                              (int(rng.integers(M)), int(rng.integers(N)), (K - 1) // 64 * 64 or -1)]:
            bit = _huge_flip(d.A, d.Bm, dtype, i, j, k_after)
            flag, _ = d.run(mode, inject=B.Fault(i, j, bit, k_after), want_report=False)
            assert flag == 1, (mode, i, j, bit, k_after)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_leading_dimensions_without_wide_stores(dtype):
    A, Bm = wl.gemm_operands(131084, 64, 128, dtype, seed=5, dist_a="normal", dist_b="normal")
    C_ref = oracle.gemm(A, Bm, dtype)
    for mode in (B.NONE, B.THREAD):
        r = run_gemm(A, Bm, dtype, mode, lda_pad=8, ldb_pad=16, ldc_pad=1)
        assert c_close(r.C, C_ref, dtype) and r.flag == 0


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("conv", [
    wl.Conv(12, 106, 105, 64, 64, 3, 3, 1, 1),     # nine k tiles, padding taps, rows that end inside a tile
    wl.Conv(2700, 7, 7, 64, 64, 3, 3, 1, 1),       # a step of rows spans several images
    wl.Conv(36, 123, 121, 32, 64, 2, 2, 2, 0),     # two taps per k tile, stride 2
    wl.Conv(12, 215, 214, 3, 64, 7, 7, 2, 3),      # three channels: lowered to row segments, three k tiles
], ids=str)
def test_convolutions_of_very_many_rows(conv, dtype):
    d = DeviceConv(conv, dtype, seed=31)
    A = oracle.im2col(d.x, dtype, conv.KH, conv.KW, conv.stride, conv.pad)
    assert d.M >= 131072
    K = d.K if conv.Cin % 8 == 0 else 192     # (lowered: seven segments of 24, filled up to whole k tiles)
    rows = sample_rows(d.M, 3000)
    C_ref = oracle.gemm(A[rows], d.Wm, dtype)
    for mode in (B.NONE, B.THREAD, B.TWOSIDED):
        assert B.abft_kernel_name(d.M, d.N, K, d.dt, mode, conv=True) == "R64"
        print("case", conv, dtype, mode, flush=True)
        flag, rep = d.run(mode)
        assert c_close(d.C(rows), C_ref, dtype) and flag == 0, mode
        if mode == B.THREAD:
            whole = d.dC.clone()
        if mode != B.NONE:
            assert d.dC.equal(whole) and rep.worst_ratio < 0.5
            bit = _huge_flip(A, d.Wm, dtype, d.M - 3, 5, -1)
            flag, _ = d.run(mode, inject=B.Fault(d.M - 3, 5, bit, -1), want_report=False)
            assert flag == 1


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("conv", [
    wl.Conv(45, 54, 55, 64, 64, 3, 3, 1, 1),       # a pixel is a k tile: strips that meet two images, last tile short
    wl.Conv(45, 109, 56, 64, 40, 2, 2, 1, 0),      # no border, fewer columns than the tile
    wl.Conv(20, 211, 70, 64, 64, 1, 3, 1, 1),      # a filter of one row, a border above it
    wl.Conv(14, 225, 161, 3, 64, 7, 7, 2, 3),      # rows of an odd number of elements, both ends cut chunks; 21 chunks of k
    wl.Conv(24, 107, 105, 4, 64, 3, 3, 1, 0),      # no border: rows start whole, end cut; an even number of chunks
    wl.Conv(40, 118, 121, 1, 33, 5, 5, 2, 2),      # one channel, one k tile; columns that rule out wide stores
    wl.Conv(9, 242, 246, 3, 64, 3, 3, 2, 1),       # short windows
    # strides that leave rows at an image's foot unread, as many as the next image's first windows reach, and (odd height) none
    wl.Conv(15, 200, 200, 4, 64, 1, 1, 2, 0), wl.Conv(15, 201, 200, 4, 64, 1, 1, 2, 0), wl.Conv(16, 227, 227, 2, 64, 3, 3, 5, 0),
    wl.Conv(15, 190, 204, 4, 64, 1, 3, 2, 0), wl.Conv(10, 202, 150, 4, 48, 2, 3, 6, 1),
], ids=str)
def test_convolutions_whose_input_rows_stay_in_lds(conv, dtype):
    """The strip kernel: every tap read from input rows that were copied into LDS once, with their border."""
    if conv.batch * conv.OH * conv.OW < 131072:
        conv = wl.Conv(-(-131072 // (conv.OH * conv.OW)), *[getattr(conv, f) for f in
                       ("H", "W", "Cin", "Cout", "KH", "KW", "stride", "pad")])
    d = DeviceConv(conv, dtype, seed=37)
    A = oracle.im2col(d.x, dtype, conv.KH, conv.KW, conv.stride, conv.pad)
    rows = np.unique(np.concatenate([sample_rows(d.M, 3000), edge_rows(conv)]))
    C_ref = oracle.gemm(A[rows], d.Wm, dtype)
    for mode in WAVE:
        print("case", conv, dtype, mode, flush=True)
        d.dC.fill_(7.0)
        flag, rep = d.run(mode)
        assert c_close(d.C(rows), C_ref, dtype) and flag == 0, mode
        if mode == B.NONE:
            continue
        if mode == B.THREAD:
            whole = d.dC.clone()
        assert d.dC.equal(whole) and rep.worst_ratio < 0.5 and rep.tiles == -(-d.M // 32)
        for i, j in [(0, 0), (d.M - 1, d.N - 1), (d.M // 2, 7)]:
            flag, _ = d.run(mode, inject=B.Fault(i, j, _huge_flip(A, d.Wm, dtype, i, j, -1), -1), want_report=False)
            assert flag == 1, (mode, i, j)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("conv", [
    wl.Conv(37, 64, 64, 3, 64, 1, 1, 2, 0), wl.Conv(40, 120, 120, 3, 64, 1, 1, 2, 0), wl.Conv(16, 227, 227, 2, 64, 3, 3, 5, 0),
    wl.Conv(64, 65, 70, 3, 40, 3, 3, 2, 1),
], ids=str)
def test_lowered_convolutions_of_fewer_rows_on_strips(conv, dtype):
    """All of C, where a strip's rows of C come from two images and its stride leaves input rows unread."""
    d = DeviceConv(conv, dtype, seed=47)
    A = oracle.im2col(d.x, dtype, conv.KH, conv.KW, conv.stride, conv.pad)
    C_ref = oracle.gemm(A, d.Wm, dtype)
    for mode in (B.NONE, B.THREAD, B.REPLICA):
        print("case", conv, dtype, mode, flush=True)
        d.dC.fill_(7.0)
        flag, rep = d.run(mode)
        assert c_close(d.C(), C_ref, dtype) and flag == 0, mode
        assert mode == B.NONE or (rep.worst_ratio < 0.5 and rep.tiles == -(-d.M // 32))


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("conv", [
    wl.Conv(328, 20, 20, 20, 64, 3, 3, 1, 1),      # runs of 60 elements
    wl.Conv(330, 22, 19, 12, 33, 5, 5, 1, 2),
    wl.Conv(35, 63, 63, 30, 64, 2, 2, 1, 0),       # two filter rows
], ids=str)
def test_padded_copies_whose_runs_are_a_whole_k_tile(conv, dtype):
    """Lowered convolutions whose strips do not fit LDS: their product reads the padded copy, whose rows and pixels have
    pitches of their own, although a run is as long as the pixels that the strip kernel takes."""
    d = DeviceConv(conv, dtype, seed=43)
    assert d.M >= 131072 and B.abft_kernel_name(d.M, d.N, 64 * conv.KH, d.dt, B.THREAD, conv=True) == "R64"
    A = oracle.im2col(d.x, dtype, conv.KH, conv.KW, conv.stride, conv.pad)
    rows = np.union1d(sample_rows(d.M, 3000), edge_rows(conv))
    C_ref = oracle.gemm(A[rows], d.Wm, dtype)
    for mode in WAVE:
        print("case", conv, dtype, mode, flush=True)
        d.dC.fill_(7.0)
        flag, rep = d.run(mode)
        assert c_close(d.C(rows), C_ref, dtype) and flag == 0, mode
        if mode == B.NONE:
            continue
        if mode == B.THREAD:
            whole = d.dC.clone()
        assert d.dC.equal(whole) and rep.worst_ratio < 0.5 and rep.tiles == -(-d.M // 32)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_activation_and_sums_left_for_the_next_layer(dtype):
    """A thread-level layer on this kernel applies ReLU, and leaves the column sums of what it stores to a layer under
    the global scheme, whose comparison they enter."""
    import torch
    from gpu_util import DEV, c_to_host, to_dev
    M, dt = 131072 + 32, DT[dtype]
    widths = [64, 128, 128]
    x = wl.random_matrix((M, widths[0]), dtype, "uniform_01", 3)
    ws = [wl.random_matrix((widths[i], widths[i + 1]), dtype, "weights", 10 + i) for i in range(2)]
    dws = [to_dev(np.ascontiguousarray(w.T), dtype) for w in ws]
    layers = [B.Layer(M, widths[i + 1], widths[i], dt, B.B_NK, 0, B.Conv(), dws[i].data_ptr(), widths[i]) for i in range(2)]
    plan = B.abft_plan_create(layers)
    B.abft_plan_set_mode(plan, 0, B.THREAD)
    B.abft_plan_set_mode(plan, 1, B.GLOBAL)
    B.abft_plan_set_activation(plan, 0, B.ACT_RELU)
    t = {"f16": torch.float16, "bf16": torch.bfloat16}[dtype]
    dx = to_dev(x, dtype)
    outs = [torch.zeros((M, w), dtype=t, device=DEV) for w in widths[1:]]
    flag = torch.zeros(1, dtype=torch.int32, device=DEV)
    before = B.abft_handover_launches()
    B.abft_plan_run_chain(plan, 0, 2, dx, widths[0], outs, widths[1:], flag)
    torch.cuda.synchronize()
    assert B.abft_handover_launches() == before + 1
    assert int(flag.item()) == 0
    ref = np.maximum(oracle.gemm(x, ws[0], dtype), 0)
    assert c_close(c_to_host(outs[0], dtype), ref, dtype)
    stored = outs[0].double().cpu().numpy()
    w1 = dws[1].double().cpu().numpy().T
    assert c_close(c_to_host(outs[1], dtype), stored @ w1, dtype)
    B.abft_plan_set_diagnostics(plan, 1, None, B.Fault(M - 5, 77, 30, -1))
    B.abft_plan_run_chain(plan, 0, 2, dx, widths[0], outs, widths[1:], flag)
    torch.cuda.synchronize()
    assert int(flag.item()) == 1
    B.abft_plan_destroy(plan)


def test_rows_up_to_the_largest_count():
    """2^31 - 128 rows (a 1 x 8 filter over 128 images of one very long line): the loads that run ahead of the last
    tiles count rows past 2^31, and must neither read there nor take those rows for rows of C."""
    import torch
    from gpu_util import DEV
    batch, ow, cin, kw = 128, 2 ** 24 - 1, 8, 8
    W, M, K = ow + kw - 1, batch * ow, kw * cin
    assert M == 2 ** 31 - 128 and B.abft_tile_shape(M, 1, K, B.F16)[:2] == (32, 64)
    x = torch.empty(batch * W * cin, dtype=torch.float16, device=DEV)
    n = 1 << 22
    x[:n].normal_(generator=torch.Generator(device=DEV).manual_seed(1))
    while n < x.numel():
        m = min(n, x.numel() - n)
        x[n:n + m] = x[:m]
        n += m
    w = torch.randn(K, device=DEV, generator=torch.Generator(device=DEV).manual_seed(2)).half()
    C = torch.full((M,), 7.0, dtype=torch.float16, device=DEV)
    flag = torch.zeros(1, dtype=torch.int32, device=DEV)
    conv = B.Conv(batch, 1, W, cin, 1, kw, 1, 0)
    print("case", M, 1, K, flush=True)
    B.abft_conv(conv, 1, x, w, K, B.B_NK, C, 1, B.F16, B.THREAD, fault_flag=flag)
    torch.cuda.synchronize()
    assert int(flag.item()) == 0
    rows = torch.cat([torch.arange(0, 4096), torch.arange(M // 2, M // 2 + 4096), torch.arange(M - 16384, M)]).to(DEV)
    at = (rows // ow) * (W * cin) + (rows % ow) * cin
    ref = torch.empty(rows.numel(), dtype=torch.float64, device=DEV)
    for i in range(0, rows.numel(), 4096):
        ref[i:i + 4096] = (x[at[i:i + 4096, None] + torch.arange(K, device=DEV)].double() * w.double()).sum(1)
    assert c_close(C[rows].double().cpu().numpy(), ref.cpu().numpy(), "f16")
    del x, C
    torch.cuda.empty_cache()


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("conv", [
    wl.Conv(44, 111, 109, 9, 64, 7, 7, 2, 3),      # lowered to segments of a whole k tile that start at multiples of four bytes
    wl.Conv(44, 112, 110, 64, 256, 1, 1, 2, 0),    # one tap, stride 2, four column blocks
    wl.Conv(44, 55, 56, 64, 33, 3, 3, 1, 1),       # one tap per k tile, nine of them
    wl.Conv(44, 55, 56, 32, 64, 3, 3, 1, 1),       # two taps per k tile and half a tile left: not on this kernel
], ids=str)
def test_convolutions_with_one_tap_per_k_tile(conv, dtype):
    d = DeviceConv(conv, dtype, seed=41)
    A = oracle.im2col(d.x, dtype, conv.KH, conv.KW, conv.stride, conv.pad)
    assert d.M >= 131072
    rows = sample_rows(d.M, 3000)
    C_ref = oracle.gemm(A[rows], d.Wm, dtype)
    for mode in (B.NONE, B.THREAD, B.THREAD_HALF):
        print("case", conv, dtype, mode, flush=True)
        d.dC.fill_(7.0)
        flag, rep = d.run(mode)
        assert c_close(d.C(rows), C_ref, dtype) and flag == 0, mode
        if mode != B.THREAD:
            continue
        # finished and running accumulators, first and last rows and columns
        for i, j, k_after in [(0, conv.Cout - 1, -1), (d.M - 1, 0, -1), (d.M // 3, 5, 64), (d.M - 2, 32, (d.K - 1) // 64 * 64)]:
            if not 0 < k_after < d.K:
                k_after = -1
            bit = _huge_flip(A, d.Wm, dtype, i, j, k_after)
            flag, _ = d.run(mode, inject=B.Fault(i, j, bit, k_after), want_report=False)
            assert flag == 1, (i, j, bit, k_after)
