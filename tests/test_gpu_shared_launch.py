"""A pass over a plan's layers (abft_plan_run_all) in which layers share kernel launches gives, bit by bit, what
the layers give one by one, whatever depends on whatever."""
import pytest

from paper_2104_09455_amd import binding as B

pytestmark = pytest.mark.gpu

DT = {"f16": B.F16, "bf16": B.BF16, "i8": B.I8}
GUARD = 77


def _tensors(dtype, seed):
    import torch
    gen = torch.Generator(device="cuda:0").manual_seed(seed)
    t = {"f16": torch.float16, "bf16": torch.bfloat16, "i8": torch.int8}[dtype]

    def rnd(*shape):
        if dtype == "i8":
            return torch.randint(-128, 128, shape, dtype=t, device="cuda:0", generator=gen)
        return torch.randn(shape, device="cuda:0", generator=gen).to(t)
    return rnd, (torch.int32 if dtype == "i8" else t)


class Pass:
    """Layers of one plan: (M, N, K) or a convolution, on buffers that the caller names."""

    def __init__(self, dtype, mode, seed=1):
        self.dt, self.mode = DT[dtype], mode
        self.rnd, self.ct = _tensors(dtype, seed)
        self.descs, self.io, self.keep = [], [], []

    def add(self, shape, A, C, relu=False):
        import torch
        if isinstance(shape, B.Conv):
            c = shape
            oh, ow = (c.H + 2 * c.pad - c.KH) // c.stride + 1, (c.W + 2 * c.pad - c.KW) // c.stride + 1
            M, N, K = c.batch * oh * ow, C.shape[1], c.KH * c.KW * c.Cin
        else:
            (M, N, K), c = shape, None
        W = self.rnd(N, K)
        if W.dtype != torch.int8:
            W = W * 0.05
        self.keep.append(W)
        self.descs.append(B.Layer(M, N, K, self.dt, B.B_NK, 0 if c is None else 1, c or B.Conv(), W.data_ptr(), K))
        self.io.append((A, K, C, C.stride(0), relu))

    def out(self, M, N, pad=0):
        import torch
        return torch.full((M, N + pad), GUARD, dtype=self.ct, device="cuda:0")

    def run(self, together):
        import torch
        plan = B.abft_plan_create(self.descs)
        flag = torch.zeros(1, dtype=torch.int32, device="cuda:0")
        for i, x in enumerate(self.io):
            B.abft_plan_set_mode(plan, i, self.mode)
            if x[4]:
                B.abft_plan_set_activation(plan, i, B.ACT_RELU)
        before = B.abft_shared_launches()
        try:
            if together:
                B.abft_plan_run_all(plan, B.PlanIO([x[0] for x in self.io], [x[1] for x in self.io],
                                                   [x[2] for x in self.io], [x[3] for x in self.io]), flag)
            else:
                for i, (A, lda, C, ldc, _) in enumerate(self.io):
                    B.abft_plan_run(plan, i, A, lda, C, ldc, flag)
            torch.cuda.synchronize()
        finally:
            B.abft_plan_destroy(plan)
        return int(flag.item()), B.abft_shared_launches() - before

    def both_ways(self, shared=None, flag=0):
        """Run one by one, then together from the same start; every output buffer has to agree."""
        import torch
        bufs = list({id(x[2]): x[2] for x in self.io}.values()) + list({id(x[0]): x[0] for x in self.io}.values())
        start = [b.clone() for b in bufs]
        f1, n1 = self.run(False)
        want = [b.clone() for b in bufs]
        for b, s in zip(bufs, start):
            b.copy_(s)
        f2, n2 = self.run(True)
        assert n1 == 0 and (shared is None or n2 == shared), n2
        assert f1 == f2 == flag
        for b, w in zip(bufs, want):
            assert torch.equal(b.view(torch.uint8), w.view(torch.uint8))


# a layer of each streaming tiling (abft_kernel_name), by the product's size and by a convolution's
KINDS = {"S32": (196, 256, 1024), "S32W": (49, 512, 2048), "S64": (784, 512, 128), "S128": (784, 1024, 512)}
CONVS = {"S32": (1, 28, 128, 128, 3, 1, 1), "S32W": (1, 7, 512, 512, 3, 1, 1), "S64": (1, 56, 256, 512, 1, 2, 0),
         "S128": (4, 56, 64, 64, 3, 1, 1)}


@pytest.mark.parametrize("dtype", ["f16", "bf16", "i8"])
@pytest.mark.parametrize("mode", [B.NONE, B.GLOBAL, B.THREAD])
def test_layers_of_every_streaming_tiling(mode, dtype):
    p = Pass(dtype, mode)
    for kind, (M, N, K) in KINDS.items():
        K = K * 2 if dtype == "i8" else K
        for rep in range(3 if kind == "S32" else 2):
            p.add((M - rep, N, K), p.rnd(M - rep, K), p.out(M - rep, N)[:, :N], relu=rep == 1)
        b, H, Cin, Cout, k, st, pad = CONVS[kind]
        Cin = Cin * 2 if dtype == "i8" else Cin
        oh = (H + 2 * pad - k) // st + 1
        p.add(B.Conv(b, H, H, Cin, k, k, st, pad), p.rnd(b, H, H, Cin), p.out(b * oh * oh, Cout))
    names = {B.abft_kernel_name(d.M, d.N, d.K, d.dtype, mode, conv=bool(d.has_conv)) for d in p.descs}
    assert {"S32", "S64", "S128"} <= names
    # (what runs on another tiling under some scheme runs by itself)
    p.both_ways(shared=len([n for n in names if n.startswith("S")]))


def test_one_round_two_and_more_and_more_layers_than_a_launch_takes():
    # (a launch takes 16 layers, and a 17th by itself is no shared launch; 70 layers: a window of 64 and one of 6)
    for layers, shared in ((2, 1), (5, 1), (17, 1), (40, 3), (70, 5)):
        p = Pass("f16", B.THREAD, seed=layers)
        for i in range(layers):
            M = 32 * (1 + i % 4) - i % 3
            p.add((M, 96 + i % 2, 256), p.rnd(M, 256), p.out(M, 96 + i % 2, pad=i % 5), relu=i % 2 == 0)
        p.both_ways(shared=shared)
    for M in (1024, 2048, 4096):        # 4 x 64 .. 256 workgroups: one round, two, four
        p = Pass("bf16", B.GLOBAL, seed=M)
        for i in range(4):
            p.add((M, 64, 128), p.rnd(M, 128), p.out(M, 64))
        p.both_ways(shared=1)


def test_dependences():
    import torch
    # two chains side by side, of unequal length, one of them through a layer of another kind
    p = Pass("f16", B.THREAD)
    x, y = p.rnd(64, 256), p.rnd(64, 256)
    for i in range(3):
        c = p.out(64, 256)
        p.add((64, 256, 256), x, c, relu=True)
        x = c
    for i in range(5):
        c = p.out(64, 256)
        p.add((64, 256, 256), y, c)
        y = c
    p.both_ways(shared=3)
    # a layer writes what an earlier one reads; two write the same matrix (the later one stays); parts of one buffer
    p = Pass("f16", B.NONE)
    buf, c1 = p.rnd(192, 256), p.out(64, 256)
    p.add((64, 256, 256), buf[:64], c1)                # reads rows 0 .. 63
    p.add((64, 256, 256), p.rnd(64, 256), buf[32:96])   # overwrites half of them
    p.add((64, 256, 256), p.rnd(64, 256), buf[96:160])  # beside them
    p.add((64, 256, 256), buf[128:192], c1)             # reads some of that; the same output again
    p.add((64, 256, 256), c1, buf[0:64])
    p.both_ways(shared=2)                               # layers 0 and 2, then 1 and 3
    # columns of one matrix: ranges that interleave are taken for ranges that meet
    p = Pass("f16", B.THREAD)
    wide = p.out(64, 512)
    for j in range(4):
        p.add((64, 128, 256), p.rnd(64, 256), wide[:, 128 * j:128 * (j + 1)])
    p.both_ways(shared=0)
    # weights that an earlier layer of the pass writes
    p = Pass("f16", B.NONE)
    w = p.out(128, 256)
    p.add((128, 256, 256), p.rnd(128, 256), w)
    p.add((64, 128, 256), p.rnd(64, 256), p.out(64, 128))
    p.descs[1].B = w.data_ptr()
    p.both_ways(shared=0)
    assert torch.isfinite(w).all()


def test_a_fault_in_a_shared_launch_raises_the_flag_and_diagnostics_keep_their_place():
    import torch
    for bad in range(3):
        p = Pass("f16", B.THREAD)
        for i in range(3):
            A = p.rnd(64, 256)
            if i == bad:
                A[5, 7] = float("nan")
            p.add((64, 128, 256), A, p.out(64, 128))
        p.both_ways(shared=1, flag=1)
    # a layer with a planted fault runs by itself, between the others
    p = Pass("f16", B.THREAD)
    for i in range(5):
        p.add((64, 128, 256), p.rnd(64, 256), p.out(64, 128))
    plan = B.abft_plan_create(p.descs)
    flag = torch.zeros(1, dtype=torch.int32, device="cuda:0")
    B.abft_plan_set_diagnostics(plan, 2, None, B.Fault(3, 4, 30, -1))
    before = B.abft_shared_launches()
    B.abft_plan_run_all(plan, B.PlanIO(*[[x[q] for x in p.io] for q in range(4)]), flag)
    assert int(flag.item()) == 1 and B.abft_shared_launches() - before == 2
    B.abft_plan_destroy(plan)


def test_a_refused_layer_leaves_the_ones_before_it_done():
    import torch
    p = Pass("f16", B.THREAD)
    for i in range(4):
        p.add((64, 128, 256), p.rnd(64, 256), p.out(64, 128))
    plan = B.abft_plan_create(p.descs)
    flag = torch.zeros(1, dtype=torch.int32, device="cuda:0")
    io = B.PlanIO([x[0] for x in p.io], [256] * 4, [x[2] for x in p.io], [128, 128, 100, 128])
    with pytest.raises(B.AbftError) as e:
        B.abft_plan_run_all(plan, io, flag)
    torch.cuda.synchronize()
    assert e.value.code == -3
    done = [not bool((x[2] == GUARD).all()) for x in p.io]
    assert done == [True, True, False, False]
    B.abft_plan_destroy(plan)


def test_captured_into_a_graph():
    import torch
    p = Pass("f16", B.THREAD)
    x = p.rnd(64, 256)
    for i in range(6):
        c = p.out(64, 256)
        p.add((64, 256, 256), x if i % 2 else p.rnd(64, 256), c)
        x = c
    plan = B.abft_plan_create(p.descs)
    flag = torch.zeros(1, dtype=torch.int32, device="cuda:0")
    io = B.PlanIO(*[[x[q] for x in p.io] for q in range(4)])
    B.abft_plan_run_all(plan, io, flag)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        B.abft_plan_run_all(plan, io, flag)
    for rep in range(3):
        for q in range(0, 6, 2):
            p.io[q][0].copy_(p.rnd(64, 256))
        B.abft_plan_run_all(plan, io, flag)
        torch.cuda.synchronize()
        want = [x[2].clone() for x in p.io]
        for x in p.io:
            x[2].fill_(GUARD)
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(x[2], w) for x, w in zip(p.io, want)) and int(flag.item()) == 0
    B.abft_plan_destroy(plan)


@pytest.mark.parametrize("dtype", ["f16", "bf16", "i8"])
@pytest.mark.parametrize("mode", [B.NONE, B.THREAD])
def test_products_of_one_k_tile_at_any_address_beside_streaming_ones(mode, dtype):
    """k of 16 to 128 bytes: whole and cut chunks and k steps, tiles that C cuts, with and without a launch that takes them."""
    elements = (9, 13, 15, 17, 33, 47, 63) if dtype != "i8" else (17, 19, 33, 65, 97, 113, 127)
    for i, K in enumerate(elements):
        for h, host in enumerate((None, KINDS["S32"], KINDS["S64"], KINDS["S128"])):
            M, N = (17, 64, 65, 250)[(i + h) % 4], (1, 31, 64, 100, 130)[(i + 2 * h) % 5]
            assert B.abft_kernel_name(M, N, K, DT[dtype], mode, False) == "G64"
            p = Pass(dtype, mode, seed=K)
            p.add((M, N, K), p.rnd(M, K), p.out(M, N, pad=i % 3), relu=i % 2 == 0)
            if host:
                m, n, k = host[0], host[1], host[2] * (2 if dtype == "i8" else 1)
                p.add((m, n, k), p.rnd(m, k), p.out(m, n))
            p.both_ways(shared=1 if host else 0)
    # one that waits for the only launch of its depth's kind, and one whose output that launch reads
    K = elements[2]
    p = Pass(dtype, mode)
    k = 512 if dtype == "i8" else 256
    x = p.out(64, k)
    p.add((64, k, K), p.rnd(64, K), x)
    p.add((64, 96, k), x, p.out(64, 96))
    p.both_ways(shared=0)
    p.add((33, 50, K), p.rnd(33, K), p.out(33, 50))
    p.both_ways(shared=0)   # (two of them at one depth, none with a launch to join)


@pytest.mark.parametrize("dtype,shape,name", [("f16", (3136, 256, 64), "F64T"), ("bf16", (3101, 250, 64), "F64T"), ("i8", (3136, 256, 128), "F64T"),
                                              ("f16", (12544, 256, 64), "F128T"), ("bf16", (6272, 256, 128), "F64T")])
@pytest.mark.parametrize("mode", [B.NONE, B.GLOBAL, B.THREAD])
def test_direct_to_lds_tiles_share_a_launch(mode, dtype, shape, name):
    """Two at once; one that waits for a later one of its kind; one that cannot, since a layer in between reads what it leaves."""
    M, N, K = shape
    if mode == B.THREAD:
        assert B.abft_kernel_name(M, N, K, DT[dtype], mode) == name
    takes = mode != B.GLOBAL and B.abft_kernel_name(M, N, K, DT[dtype], mode) == name
    p = Pass(dtype, mode)
    for rep in range(2):
        p.add(shape, p.rnd(M, K), p.out(M, N, pad=2 * rep), relu=rep == 1)
    p.both_ways(shared=1 if takes else 0)

    def later(reads):
        p = Pass(dtype, mode)
        first, x, y = p.out(M, N), p.out(M, K), p.out(M, 40)
        p.add(shape, p.rnd(M, K), first)
        p.add((M, K, K), p.rnd(M, K), x)
        if reads:
            p.add((M, 40, N), first, y)
            p.add((M, K, 40), y, x)
        p.add(shape, x, p.out(M, N))
        return p
    if dtype != "i8":
        later(False).both_ways(shared=1 if takes else None)
        later(True).both_ways()


# layers that share a launch of the skinny kernel (rows at any alignment), of the direct-to-LDS kernel's two tiles, of a streaming
# tiling with a product of less than one k tile
FLAGGED = {"skinny": [(16, 96, 4096), (3, 33, 37), (9, 40, 1030)], "F64T": [(3136, 256, 64), (3101, 250, 64)],
           "F128T": [(12544, 256, 64), (12500, 256, 64)], "shallow": [KINDS["S32"], (70, 100, 13), (64, 64, 64)],
           "shallow beside S64": [KINDS["S64"], (70, 100, 33)], "shallow beside S128": [KINDS["S128"], (33, 50, 15)]}


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("kind", FLAGGED)
def test_what_is_no_number_in_any_member_of_a_shared_launch_raises_the_flag(kind, dtype):
    """In the last row and the last k of one layer's input: the launch's workgroups all know the flag, and compare."""
    for bad in range(len(FLAGGED[kind])):
        p = Pass(dtype, B.THREAD, seed=bad)
        for i, (M, N, K) in enumerate(FLAGGED[kind]):
            if kind in ("F64T", "F128T"):
                assert B.abft_kernel_name(M, N, K, DT[dtype], B.THREAD) == kind
            A = p.rnd(M, K)
            if i == bad:
                A[M - 1, K - 1] = float("nan")
            p.add((M, N, K), A, p.out(M, N))
        p.both_ways(shared=1, flag=1)
