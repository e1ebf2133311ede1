// Row-streaming ABFT-protected MFMA kernel for gfx950 (MI355X): products of very many rows whose
// whole weight matrix fits in LDS (a CNN's first stage: 64 input or output channels), unprotected
// or under a wavefront-level scheme.
//
// One workgroup per compute unit copies the weights into LDS once and stays.  After that no
// wavefront waits for another: each walks its own 32-row tiles of C (32 x 64 at a
// time) and loads the k tiles (128 bytes of k) of its rows of A straight into MFMA fragments, two to
// four k tiles ahead and across tile boundaries, so that the next rows are on their way while this tile
// is checked and stored.  (A wavefront tile of 32 rows meets no other reader of its rows of A in
// the workgroup; rings of two LDS stages beside 72 KB of weights took 50 us where this form takes 41.)
// Matrices: twelve wavefronts, three per SIMD, with two k tiles ahead, so that checks and stores run under
// the others' loads: thread-level fp16 200704 x 256 x 64 33 -> 31 us, 131104 x 1280 x 64 87 -> 83 (eight with four
// ahead before; sixteen: registers spill, 38 and 92); unprotected level (27 and 74).  Bound: HBM (the rows in, C
// out; 200704 x 64 x 256 thread-level 31 us, 4.1 TB/s) and, for convolutions whose input rows do not fit LDS (else:
// the strip kernel), the rate at which the vector memory path serves fragments of 32 rows at a time.
#pragma once
#include "gemm_fast.h"

namespace abft {

template <class CFG>
struct RowsLayout {
    static constexpr int B_TILE = CFG::BN * 128;              // one k tile of 64 columns
    static constexpr int LDS_MAX = 160 * 1024;
    static constexpr int MAX_B_TILES = LDS_MAX / B_TILE;
    static_assert(CFG::MI == 32 && CFG::TM == 1 && CFG::TN == 2 && CFG::WAVES_M == 1 && CFG::WAVES_N == 1 && CFG::BKB == 128,
                  "a 32 x 64 register tile per wavefront");
};

// K is whole k tiles; one column block of 64 (p.tiles_n == 1), or several with a single k tile.
// Grid: any number of workgroups.  FORM: how a row of A is read.
enum { ROWS_MATRIX = 0, ROWS_CONV = 1, ROWS_CONV_ONE_TAP = 2 };  // (one tap: Cin a multiple of the k tile)
constexpr int rows_waves(int form) { return form == ROWS_MATRIX ? 12 : 8; }
template <class CFG, int MODE, bool INJ, int FORM>
__global__ __launch_bounds__((64 * rows_waves(FORM))) void gemm_rows_kernel(const GemmArgs p) {
    typedef RowsLayout<CFG> LAY;
    constexpr int DT = CFG::DT;
    typedef Mma<DT, 32> MMA;
    typedef typename MMA::Acc Acc;
    constexpr int TN = CFG::TN, BM = CFG::BM, BN = CFG::BN, BK = CFG::BK, ESIZE = CFG::ESIZE, EPC = CFG::EPC;
    constexpr int ROWB = 128, WAVES = rows_waves(FORM), AHEAD = FORM == ROWS_MATRIX ? 2 : 4;
    constexpr bool CONV = FORM != ROWS_MATRIX, ONE_TAP = FORM == ROWS_CONV_ONE_TAP;
    static_assert(MODE == MODE_NONE || mode_is_wave_level(MODE), "no scheme that compares across wavefronts");
    static_assert(CFG::CSIZE == 2, "16-bit outputs");

    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int M = p.M, N = p.N;
    const int nkt = p.K / BK, ncb = p.tiles_n, b_tiles = nkt * ncb;

    // contiguous runs of tiles per workgroup, consecutive runs on one die (its L2 holds the input
    // rows that neighbouring tiles of a convolution share)
    const int G = (int)gridDim.x;
    int run = (int)blockIdx.x;
    if ((G & 7) == 0) run = (run & 7) * (G >> 3) + (run >> 3);
    const int t_lo = (int)((long long)run * p.tiles_m / G), t_hi = (int)((long long)(run + 1) * p.tiles_m / G);

    // ---- the weights, once: tile (column block c, k tile t) at (c * nkt + t) * B_TILE; lane fills slot
    // `lane` of a 1 KB block (8 rows x 8 chunks): row lane/8, position lane%8, which holds chunk
    // (lane%8) ^ key(row), key(row) = (row >> 1) & 7; block q starts at row 8q
    for (int i = wave; i < b_tiles * (BN / 8); i += WAVES) {
        const int tile = i / (BN / 8), q = i - tile * (BN / 8);
        const int c = tile / nkt, t = tile - c * nkt;
        const int n = c * BN + CFG::b_row_of(q * 8 + (lane >> 3)), ck = (lane & 7) ^ ((lane >> 4) + 4 * (q & 1));
        const char* src = n < N ? p.B + ((long long)n * p.ldb + (long long)t * BK) * ESIZE + ck * 16 : g_zero_chunk + ck * 16;
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                         (__attribute__((address_space(3))) void*)(smem + i * 1024), 16, 0, 0);
    }

    // ---- this wavefront's sequence of k tiles: tiles t_lo + wave, + WAVES, ... of C, nkt each
    const int n_own = t_lo + wave < t_hi ? (t_hi - t_lo - wave + WAVES - 1) / WAVES : 0;
    const int total = n_own * nkt;

    // Fragments of a k tile: lane l holds row l%32, chunks 4 (l/32) .. + 3, one per k step (the same
    // choice for B: within a k tile the order of k is free): 64 contiguous bytes of a row per lane.
    const int frow = lane & 31, fgrp = lane >> 5, fx = (lane >> 1) & 7;
    int pos[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) pos[kk] = frow * ROWB + ((4 * fgrp + kk) ^ fx) * 16;

    // this lane's row of the tile whose loads go out next (they run AHEAD k tiles before the product;
    // unsigned: up to AHEAD steps of rows past M, which may be close to 2^31)
    unsigned m_next = (unsigned)(t_lo + wave) * BM + frow;
    const unsigned m_end = (unsigned)t_hi * BM < (unsigned)M ? (unsigned)t_hi * BM : (unsigned)M;
    const char* aptr = p.A;            // its first chunk; convolutions: its top-left input pixel, possibly outside
    int a_ih0 = 0, a_iw0 = 0;
    // filter taps: one wavefront-uniform tap where all chunks of a k tile lie in it, else one per chunk
    constexpr int NT = FORM == ROWS_CONV ? 4 : 1;
    int tap_c[NT], tap_kh[NT], tap_kw[NT];
    long long tap_off[NT];
    int u_c = 0, u_kh = 0, u_kw = 0;
    long long u_off = 0;
    auto first_taps = [&]() {
        if constexpr (ONE_TAP) {
            u_c = u_kh = u_kw = 0;
            u_off = 0;
        } else {
#pragma unroll
            for (int h = 0; h < NT; ++h) {
                const int k = (4 * fgrp + h) * EPC;
                const int tap = k / p.Cin;
                tap_c[h] = k - tap * p.Cin;
                tap_kh[h] = tap / p.KW;
                tap_kw[h] = tap - tap_kh[h] * p.KW;
                tap_off[h] = (tap_kh[h] * p.rowpitch + (long long)tap_kw[h] * p.pix + tap_c[h]) * ESIZE;
            }
        }
    };
    // rows WAVES tiles further on: so many input rows and columns, so many bytes; past the end of an
    // output row / of an image: the way to the start of the next
    int d_ih = 0, d_iw = 0, end_iw = 0, end_ih = 0;
    long long d_ptr = 0, d_row = 0, d_img = 0;
    if constexpr (CONV) {
        first_taps();
        const int d_oh = WAVES * BM / p.OW, d_ow = WAVES * BM - d_oh * p.OW;
        d_ih = d_oh * p.stride;
        d_iw = d_ow * p.stride;
        end_iw = p.OW * p.stride - p.pad;
        end_ih = p.OH * p.stride - p.pad;
        d_ptr = (d_ih * p.rowpitch + (long long)d_iw * p.pix) * ESIZE;
        d_row = (p.stride * p.rowpitch - (long long)p.OW * p.stride * p.pix) * ESIZE;
        d_img = (p.imgpitch - (long long)p.OH * p.stride * p.rowpitch) * ESIZE;
        const int m = m_next < (unsigned)M ? (int)m_next : 0;
        const int img = m / (p.OH * p.OW);
        const int rem = m - img * (p.OH * p.OW);
        const int oh = rem / p.OW, ow = rem - oh * p.OW;
        a_ih0 = oh * p.stride - p.pad;
        a_iw0 = ow * p.stride - p.pad;
        aptr += ((long long)img * p.imgpitch + a_ih0 * p.rowpitch + (long long)a_iw0 * p.pix) * ESIZE;
    } else {
        d_ptr = (long long)(WAVES * BM) * p.lda * ESIZE;
        aptr += (long long)m_next * p.lda * ESIZE + fgrp * 64;   // (not read where the row is beyond m_end)
    }
    int i_kt = 0;                      // k tile of the next loads
    auto load = [&](i32x4 (&f)[4]) {
        if constexpr (CONV) {
            if constexpr (ONE_TAP) {
                const bool ok = m_next < m_end && (unsigned)(a_ih0 + u_kh) < (unsigned)p.H && (unsigned)(a_iw0 + u_kw) < (unsigned)p.W;
                const char* src = ok ? aptr + u_off + fgrp * 64 : g_zero_chunk;
                // (a lowered row's segment can be a whole k tile; it starts at a multiple of four bytes)
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) f[kk] = ld16u(src + kk * 16);
            } else {
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) {
                    // a chunk never straddles a filter tap (Cin is a multiple of the chunk length); rows
                    // lowered to segments start at multiples of four bytes
                    const bool ok = m_next < m_end && (unsigned)(a_ih0 + tap_kh[kk]) < (unsigned)p.H &&
                                    (unsigned)(a_iw0 + tap_kw[kk]) < (unsigned)p.W;
                    f[kk] = ld16u(ok ? aptr + tap_off[kk] : g_zero_chunk);
                }
            }
        } else {
            const char* src = m_next < m_end ? aptr + i_kt * 128 : g_zero_chunk;
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) f[kk] = ld16g(src + kk * 16);
        }
        if (++i_kt < nkt) {
            if constexpr (CONV) {
                if constexpr (ONE_TAP) {
                    u_c += BK;
                    u_off += 128;
                    if (u_c == p.Cin) {
                        u_c = 0;
                        u_off += (p.pix - p.Cin) * ESIZE;
                        if (++u_kw == p.KW) {
                            u_kw = 0;
                            ++u_kh;
                            u_off += (p.rowpitch - (long long)p.KW * p.pix) * ESIZE;
                        }
                    }
                } else {
#pragma unroll
                    for (int h = 0; h < NT; ++h) {
                        tap_c[h] += BK;
                        tap_off[h] += 128;
                        while (tap_c[h] >= p.Cin) {
                            tap_c[h] -= p.Cin;
                            tap_off[h] += (p.pix - p.Cin) * ESIZE;
                            if (++tap_kw[h] == p.KW) {
                                tap_kw[h] = 0;
                                ++tap_kh[h];
                                tap_off[h] += (p.rowpitch - (long long)p.KW * p.pix) * ESIZE;
                            }
                        }
                    }
                }
            }
            return;
        }
        // on to this wavefront's next rows
        i_kt = 0;
        m_next += WAVES * BM;
        aptr += d_ptr;
        if constexpr (CONV) {
            first_taps();
            a_ih0 += d_ih;
            a_iw0 += d_iw;
            if (a_iw0 >= end_iw) {
                a_iw0 -= p.OW * p.stride;
                a_ih0 += p.stride;
                aptr += d_row;
            }
            while (a_ih0 >= end_ih) {
                a_ih0 -= p.OH * p.stride;
                aptr += d_img;
            }
        }
    };

    i32x4 fa[AHEAD][4];
    // (always all of them, and one tile's loads for every tile multiplied, so that the number of loads
    // behind the one that is waited for is known when the kernel is compiled: loads past this
    // workgroup's last tile read the zeros)
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) load(fa[u]);
    // the weights have landed for everyone; from here on no wavefront waits for another
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    __syncthreads();

    Acc acc[1][TN];
    constexpr int NCHK = CheckRegs<CFG, MODE>::N;
    Acc chk[NCHK];
    auto clear = [&]() {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[0][j][r] = 0;
        clear_check<CFG, MODE, true>(chk);
    };
    clear();
    int kt = 0, tile_m = t_lo + wave;
    auto multiply = [&](const i32x4 (&f)[4], const char* bt) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            const i32x4 a[1] = {f[kk]};
            i32x4 b[TN];
#pragma unroll
            for (int c = 0; c < TN; ++c) b[c] = *reinterpret_cast<const i32x4*>(bt + c * 32 * ROWB + pos[kk]);
#pragma unroll
            for (int c = 0; c < TN; ++c) acc[0][c] = MMA::run(a[0], b[c], acc[0][c]);
            if constexpr (mode_is_wave_level(MODE)) check_step<CFG, MODE>(a, b, chk);
        }
    };
    auto finish = [&](int cb) {
        if constexpr (INJ) {
            if (p.f_kt < 0) inject_fault<CFG>(acc, p, TileCoords<CFG>(tile_m, cb, 0));
        }
        epilogue<CFG, MODE>(acc, chk, p, tile_m, cb, nullptr, true, 0);
        clear();
    };
    for (int j = 0; j < total; j += AHEAD) {
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            bool last = false;
            if (j + u < total) {
                multiply(fa[u], smem + kt * LAY::B_TILE);
                if constexpr (INJ) {
                    if (kt == p.f_kt) inject_fault<CFG>(acc, p, TileCoords<CFG>(tile_m, 0, 0));
                }
                last = ++kt == nkt;
            }
            if (last) {
                kt = 0;
                // (several column blocks: a single k tile)
                for (int cb = 0; cb + 1 < ncb; ++cb) {
                    finish(cb);
                    multiply(fa[u], smem + (cb + 1) * LAY::B_TILE);
                }
            }
            // (whatever path was taken: the count of loads stays the same; before the last of the tile's
            // checks and stores, which take as long as the loads: behind them the stem took 100 us, so 86)
            load(fa[u]);
            if (last) {
                finish(ncb - 1);
                tile_m += WAVES;
            }
        }
    }
}

}  // namespace abft
