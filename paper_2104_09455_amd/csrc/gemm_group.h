// Several independent products in ONE launch of the streaming kernel for gfx950 (MI355X): the layers
// of a network that do not wait for one another (the two MLPs of a recommendation model, the
// downsampling and the first convolution of a block, blocks whose inputs are all at hand).
//
// A latency-bound layer occupies the chip for the 3 to 10 us of one workgroup's k loop, whatever its
// number of workgroups, so layers launched one behind the other leave most of the compute units
// idle most of the time.  Here every workgroup looks up which product it belongs to and runs the
// streaming kernel's own tile routine on it: results, checks and flag are those of the layer's own launch.
// Where all workgroups fit the chip in one round they get the stages of a launch of their own; else
// fewer, so that two to four workgroups share a compute unit and one's copies run under another's
// products and epilogue.
#pragma once
#include "gemm_configs.h"
#include "gemm_fast.h"
#include "gemm_skinny.h"
#include "gemm_stream.h"

namespace abft {

constexpr int GROUP_MAX = 16;   // products per launch: 2.8 KB of kernel arguments

// what the tile routine needs of GemmArgs
struct GroupItem {
    const char* A;
    const char* B;
    char* C;
    const char* beta_k;
    const char* beta_p;
    long long lda, ldb, ldc, imgpitch, rowpitch;
    double tol_coeff, tol_l1;
    int M, N, K, tiles_m, tiles_n, act;
    int conv, H, W, Cin, KH, KW, stride, pad, OH, OW, pix;
    int bytes;   // skinny kernel: rows at addresses that are no multiples of four
    int shallow; // streaming kernel's launches: a product for shallow_tile
};

struct GroupArgs {
    int first[GROUP_MAX];   // first workgroup of each product; unused entries: INT_MAX
    unsigned* flag;
    GroupItem item[GROUP_MAX];
};
static_assert(sizeof(GroupArgs) <= 4096, "kernel arguments");

// The product that workgroup bid works on; bid becomes its index among that product's workgroups.
__device__ __forceinline__ GemmArgs group_product(const GroupArgs& a, int& bid, bool* shallow = nullptr) {
    int i = 0;
#pragma unroll
    for (int q = 1; q < GROUP_MAX; ++q) i += bid >= a.first[q] ? 1 : 0;
    const GroupItem& L = a.item[i];
    bid -= a.first[i];

    GemmArgs g;
    g.A = L.A; g.B = L.B; g.C = L.C;
    g.M = L.M; g.N = L.N; g.K = L.K;
    g.lda = L.lda; g.ldb = L.ldb; g.ldc = L.ldc;
    g.b_sn = L.ldb; g.b_sk = 1;
    g.a_vec = g.b_vec = 1;
    g.conv = L.conv;
    g.H = L.H; g.W = L.W; g.Cin = L.Cin; g.KH = L.KH; g.KW = L.KW;
    g.stride = L.stride; g.pad = L.pad; g.OH = L.OH; g.OW = L.OW;
    g.imgpitch = L.imgpitch; g.rowpitch = L.rowpitch; g.pix = L.pix;
    g.beta_k = L.beta_k; g.beta_p = L.beta_p; g.beta_r = nullptr;
    g.partial_dots = nullptr; g.n_parts = 0;
    g.tol_l1 = L.tol_l1; g.tol_coeff = L.tol_coeff;
    g.flag = a.flag; g.report = nullptr;
    g.f_row = g.f_col = -1; g.f_bit = 0; g.f_kt = -1;
    g.tiles_m = L.tiles_m; g.tiles_n = L.tiles_n;
    g.act = L.act;
    g.alpha_out = nullptr; g.ld_alpha_out = 0; g.alpha_in = nullptr;
    if (shallow) *shallow = L.shallow != 0;
    return g;
}

// A 64 x 64 tile of a product whose k ends within one k tile (16 to 128 bytes of k, rows at any address): the generic kernel's
// tile for such products, every wavefront with its 32 x 32 MFMA block straight from memory, in registers, since no wavefront
// reads a row of A or B more than one other does.  Bound: the latency of one load.  DLRM's first layer (K = 13) so goes out
// with the first of the other MLP, which takes 32 workgroups beside 256: batch 256 27.0 -> 23.6 us a pass (five launches instead of six).
// BYTES (a product by itself): rows off multiples of four bytes, in whole dwords shifted down (gemm_skinny.h says why, and why that leaves
// no row's dwords).
template <int DT, int MODE, bool BYTES>
__device__ __forceinline__ void shallow_tile(const GemmArgs& p, int tile_m, int tile_n, char* smem) {
    typedef typename CfgOf<DT, CFG_G64>::type CFG;
    typedef Mma<DT, 32> MMA;
    static_assert(CFG::TM == 1 && CFG::TN == 1 && CFG::MI == 32 && !CFG::INTERLEAVED, "one MFMA block per wavefront");
    static_assert(MODE == MODE_NONE || MODE == MODE_THREAD, "nothing is compared across wavefronts");
    constexpr int ES = CFG::ESIZE;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m = tile_m * CFG::BM + wave / CFG::WAVES_N * 32 + (lane & 31);
    const int n = tile_n * CFG::BN + wave % CFG::WAVES_N * 32 + (lane & 31);
    const int kb = p.K * ES;
    // (rows outside A and B: another row's address, and zeros in its place)
    const char* const a = p.A + (long long)min(m, p.M - 1) * p.lda * ES;
    const char* const b = p.B + (long long)min(n, p.N - 1) * p.ldb * ES;
    const i32x4 zero = {0, 0, 0, 0};
    // the chunk at byte c of a row: one that K cuts short is the row's last 16 bytes shifted down, one beyond K zeros
    i32x4 va[4], vb[4];
    int more_a[4], more_b[4];
    auto fetch = [](const char* from, i32x4& v, int& more) {
        if constexpr (BYTES) {
            const int off = (int)(reinterpret_cast<uintptr_t>(from) & 3u);
            v = ld16u(from - off);
            more = ld4u(from - off + (off ? 16 : 12));
        } else {
            v = ld16u(from);
        }
    };
    auto whole = [](const char* from, const i32x4& v, int more) {
        if constexpr (!BYTES) return v;
        const unsigned off = (unsigned)(reinterpret_cast<uintptr_t>(from) & 3u);
        i32x4 x;
#pragma unroll
        for (int d = 0; d < 4; ++d) x[d] = (int)__builtin_amdgcn_alignbyte((unsigned)(d < 3 ? v[d + 1] : more), (unsigned)v[d], off);
        return x;
    };
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        const int off = min(32 * kk + 16 * (lane >> 5), kb - 16);
        va[kk] = vb[kk] = zero;
        more_a[kk] = more_b[kk] = 0;
        if (32 * kk < kb) {
            fetch(a + off, va[kk], more_a[kk]);
            fetch(b + off, vb[kk], more_b[kk]);
        }
    }
    typename MMA::Acc acc[1][1], chk[CheckRegs<CFG, MODE>::N];
#pragma unroll
    for (int r = 0; r < MMA::NACC; ++r) acc[0][0][r] = 0;
    clear_check<CFG, MODE, true>(chk);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        if (32 * kk >= kb) break;
        const int c = 32 * kk + 16 * (lane >> 5), off = min(c, kb - 16), early = c - off;
        i32x4 fa[1] = {whole(a + off, va[kk], more_a[kk])}, fb[1] = {whole(b + off, vb[kk], more_b[kk])};
        if (32 * kk + 32 > kb) {
            fa[0] = early < 16 ? shift_down(fa[0], early & 15) : zero;
            fb[0] = early < 16 ? shift_down(fb[0], early & 15) : zero;
        }
        fa[0] = m < p.M ? fa[0] : zero;
        fb[0] = n < p.N ? fb[0] : zero;
        acc[0][0] = MMA::run(fa[0], fb[0], acc[0][0]);
        if constexpr (MODE == MODE_THREAD) check_step<CFG, MODE>(fa, fb, chk);
    }
    epilogue<CFG, MODE>(acc, chk, p, tile_m, tile_n, smem);
}

// One such product by itself, its tiles in the generic kernel's order.
template <int DT, int MODE, bool BYTES>
__global__ __launch_bounds__((CfgOf<DT, CFG_G64>::type::THREADS)) void gemm_shallow_kernel(const GemmArgs p) {
    int tile_m, tile_n;
    generic_tile_of_block((int)blockIdx.x, p.tiles_m, p.tiles_n, tile_m, tile_n);
    shallow_tile<DT, MODE, BYTES>(p, tile_m, tile_n, nullptr);
}

template <int DT, int ID, int NST, int MODE>
__global__ __launch_bounds__((64 * CfgOf<DT, ID>::KWAYS)) void gemm_group_kernel(const GroupArgs a) {
    typedef typename CfgOf<DT, ID>::type CFG;
    constexpr int KWAYS = CfgOf<DT, ID>::KWAYS;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    int bid = (int)blockIdx.x;
    bool shallow;
    const GemmArgs g = group_product(a, bid, &shallow);
    int tile_m, tile_n;
    tile_of_block(bid, g.tiles_m, g.tiles_n, tile_m, tile_n);
    if constexpr (KWAYS == 4 && MODE != MODE_GLOBAL) {
        if (shallow) {
            // (off dwords too without whole dwords: a second body's 6 KB of code cost launches that hold no such product, too: ResNet-50 at
            // batch 1 89.5 -> 91.2 us, DLRM at 256 23.55 -> 23.8)
            shallow_tile<DT, MODE, false>(g, tile_m, tile_n, smem);
            return;
        }
    }
    if (g.conv) stream_tile<CFG, NST, KWAYS, MODE, false, true, false, false>(g, tile_m, tile_n, smem);
    else stream_tile<CFG, NST, KWAYS, MODE, false, false, false, false>(g, tile_m, tile_n, smem);
}

// The direct-to-LDS kernel's tiles: matrices (1 x 1 convolutions among them) with few tiles and short k loops, of which several fit a
// compute unit at once and one launch of its own fills hardly half of the chip.  Bound: the latency of load, product, store.
// ResNet-50 at batch 1, the four layers 3136 x 256 x 64 (98 tiles each): two launches instead of four, 101.0 -> 90.0 us a pass.
template <int DT, int ID, int MODE>
__global__ __launch_bounds__((CfgOf<DT, ID>::type::THREADS)) __attribute__((amdgpu_waves_per_eu(min_waves_per_simd<typename CfgOf<DT, ID>::type, MODE>())))
void gemm_fast_group_kernel(const GroupArgs a) {
    int bid = (int)blockIdx.x;
    const GemmArgs g = group_product(a, bid);
    fast_tile<typename CfgOf<DT, ID>::type, CfgOf<DT, ID>::NSTAGE, MODE, false, false>(g, bid);
}

// Products of at most sixteen rows: the skinny kernel's tile routine, with the loads that each product's rows allow.
template <int DT, int MODE>
__global__ __launch_bounds__(64 * SKINNY_WAVES) void gemm_skinny_group_kernel(const GroupArgs a) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int bid = (int)blockIdx.x;
    int i = 0;
#pragma unroll
    for (int q = 1; q < GROUP_MAX; ++q) i += bid >= a.first[q] ? 1 : 0;
    const GroupItem& L = a.item[i];
    GemmArgs g;
    g.A = L.A; g.B = L.B; g.C = L.C;
    g.M = L.M; g.N = L.N; g.K = L.K;
    g.lda = L.lda; g.ldb = L.ldb; g.ldc = L.ldc;
    g.tol_coeff = L.tol_coeff;
    g.flag = a.flag; g.report = nullptr;
    g.act = L.act;
    int tile_m, tile_n;
    tile_of_block(bid - a.first[i], 1, L.tiles_n, tile_m, tile_n);
    if (L.bytes) skinny_tile<DT, 1, MODE, true, false>(g, tile_n, smem);
    else skinny_tile<DT, 1, MODE, false, false>(g, tile_n, smem);
}

// blocks: workgroups of all products together; mode: MODE_NONE, MODE_GLOBAL or MODE_THREAD (direct-to-LDS kernel: not MODE_GLOBAL)
hipError_t launch_group_f16(int cfg, int mode, int blocks, const GroupArgs& args, hipStream_t stream);
hipError_t launch_group_bf16(int cfg, int mode, int blocks, const GroupArgs& args, hipStream_t stream);
hipError_t launch_group_i8(int cfg, int mode, int blocks, const GroupArgs& args, hipStream_t stream);
// one product for shallow_tile (mode: MODE_NONE or MODE_THREAD; bytes: rows at addresses that are no multiples of four)
hipError_t launch_shallow_f16(int mode, bool bytes, const GemmArgs& args, hipStream_t stream);
hipError_t launch_shallow_bf16(int mode, bool bytes, const GemmArgs& args, hipStream_t stream);
hipError_t launch_shallow_i8(int mode, bool bytes, const GemmArgs& args, hipStream_t stream);
// the skinny kernel: one product (mode: MODE_NONE or wavefront-level; args.f_row >= 0: with a planted fault; bytes: rows at addresses that are no multiples of four; columns: of the
// comparisons that a report counts, 16 or 32), several
hipError_t launch_skinny_f16(int mode, bool bytes, int columns, const GemmArgs& args, hipStream_t stream);
hipError_t launch_skinny_bf16(int mode, bool bytes, int columns, const GemmArgs& args, hipStream_t stream);
hipError_t launch_skinny_i8(int mode, bool bytes, int columns, const GemmArgs& args, hipStream_t stream);
hipError_t launch_skinny_group_f16(int mode, int blocks, const GroupArgs& args, hipStream_t stream);
hipError_t launch_skinny_group_bf16(int mode, int blocks, const GroupArgs& args, hipStream_t stream);
hipError_t launch_skinny_group_i8(int mode, int blocks, const GroupArgs& args, hipStream_t stream);

}  // namespace abft
