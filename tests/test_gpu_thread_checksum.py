"""Clean comparisons of the thread-level scheme (fp16, bf16) on every kernel whose wavefront tiles hold several B
fragments, with operands under which every element of a tile rounds alike (constant ones, constant rows) and with
long k loops of one sign: a checksum side that does not go through the product's own roundings drifts away from it
there, by several tolerances."""
import ctypes

import pytest
import torch

from gpu_util import DEV, DT, read_report
from paper_2104_09455_amd import binding as B

pytestmark = pytest.mark.gpu
TORCH = {"f16": torch.float16, "bf16": torch.bfloat16}

# (M, N, K) -> wavefront tile: streaming 32 x 64 and 64 x 64 (partial sums of four wavefronts are added), direct-to-LDS
# with two and with four B fragments, the generic kernel, the row-streaming kernel with several and with one k tile
STREAMING = {(512, 1024, 1024): (32, 64), (1024, 1024, 1024): (64, 64), (1024, 1024, 65536): (64, 64)}
ALONE = {(2048, 2048, 1024): (64, 64), (2048, 2048, 65536): (64, 64), (4096, 4096, 4096): (32, 128), (1024, 1000, 192): (32, 128),
         (2048, 2048, 1001): (64, 64), (131072, 64, 576): (32, 64), (131104, 256, 64): (32, 64)}


def _operand(kind, rows, K, dtype, gen):
    if kind == "constant":
        return torch.full((rows, K), 0.1, device=DEV).to(TORCH[dtype])
    x = torch.rand((rows, 1 if kind == "rows" else K), device=DEV, generator=gen)
    return x.expand(rows, K).to(TORCH[dtype]).contiguous()


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("shape", [*STREAMING, *ALONE], ids=str)
def test_clean_products_whose_elements_round_alike(shape, dtype):
    M, N, K = shape
    dt = DT[dtype]
    tile = STREAMING.get(shape) or ALONE[shape]
    assert B.abft_tile_shape(M, N, K, dt, K % 8 == 0)[:2] == tile
    for kind in ("constant", "rows", "uniform"):
        if kind == "rows" and shape in STREAMING and K > 4096:
            continue    # (the final addition's own roundings, alike in a row, reach the tolerance: not the checksum's)
        gen = torch.Generator(device=DEV).manual_seed(M + K)
        A, W = _operand(kind, M, K, dtype, gen), _operand(kind, N, K, dtype, gen)
        C = torch.empty((M, N), dtype=TORCH[dtype], device=DEV)
        flag = torch.zeros(1, dtype=torch.int32, device=DEV)
        rep = torch.zeros(ctypes.sizeof(B.Report), dtype=torch.uint8, device=DEV)
        print("case", shape, dtype, kind, flush=True)
        B.abft_gemm(M, N, K, A, K, W, K, B.B_NK, C, N, dt, B.THREAD, fault_flag=flag, report=rep)
        torch.cuda.synchronize()
        r = read_report(rep)
        assert int(flag.item()) == 0, (kind, r.worst_ratio)
        # one wavefront (or groups added element by element) forms both sides alike: equal up to fp64 sums
        assert r.worst_ratio < (0.5 if shape in STREAMING else 1e-6), (kind, r.worst_ratio)
