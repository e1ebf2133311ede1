// Strip ABFT-protected MFMA kernel for gfx950 (MI355X): convolutions of very many rows with few
// channels (a CNN's stem and first stage), unprotected or under a wavefront-level scheme.
//
// An input pixel of such a convolution is read by KH KW / stride^2 output pixels.  Fetched from memory for
// every one of them, 16 bytes of 32 rows at a time, the reads are bound by the vector memory path (row-streaming
// kernel: 49 taps of three channels, 86 us where the bytes take 20; nine of 64 channels, 46 where they take 8).  Here a
// workgroup takes consecutive 32-row tiles of C (one per wavefront, the row-streaming kernel's tiles), copies the
// input rows under them into LDS once, in whole cache lines and with their zero border, and takes every tap from
// there; the weights are resident beside them.  The next tiles' input is on its way into registers while
// these are multiplied, checked and stored.
//   STRIP_RUNS: twelve wavefronts, three per SIMD, so that one's epilogue and fragment reads run under the others'
//     MFMAs (eight: 64 us, twelve 57), and two strips in LDS, one barrier per strip.  The padded copy that the
//     row-streaming kernel needs, 14 us, is gone.
//   STRIP_TAPS: nine k tiles of weights leave LDS for one strip; eight wavefronts, four steps' fragments read ahead.
// Thread-level fp16: stem of 64 images (802816 x 64, 7 x 7 x 3) 88 -> 47-50 us, its padded copy among them; 3 x 3 convolution
// 64 -> 64 on 200704 rows 46 -> 38.  Bound: vector work (500 instructions a 32 x 64 stem tile, the epilogue's half of them),
// then the store of C.
#pragma once
#include "gemm_configs.h"

namespace abft {

// STRIP_RUNS: few channels, p.B in the order (filter row, run of p.strip_seg elements: its KW Cin taps and
//   zeros up to whole chunks), p.K the whole k tiles of that order.
// STRIP_TAPS: a pixel's channels are one k tile (128 bytes).
template <int FORM>
struct StripLayout {
    static constexpr int WAVES = strip_waves(FORM), THREADS = 64 * WAVES;
    static constexpr int STRIP_MAX = strip_max_bytes(FORM);
    static constexpr int AHEAD = STRIP_MAX / (THREADS * 16);   // chunks of the next strip per thread
};

// Input rows in LDS are "virtual" rows: v = img Hv + (row of the padded image), Hv the padded rows that one image's
// windows reach.  The pitch covers a whole padded row.  One column block (N <= 64), at most Hv rows in a strip, OW > 1.
template <class CFG, int MODE, bool INJ, int FORM>
__global__ __launch_bounds__(StripLayout<FORM>::THREADS, StripLayout<FORM>::WAVES / 4) void gemm_strip_kernel(const GemmArgs p) {
    typedef RowsLayout<CFG> LAY;
    constexpr int DT = CFG::DT;
    typedef Mma<DT, 32> MMA;
    typedef typename MMA::Acc Acc;
    constexpr int TN = CFG::TN, BM = CFG::BM, BN = CFG::BN, BK = CFG::BK, ESIZE = CFG::ESIZE;
    constexpr int ROWB = 128, WAVES = StripLayout<FORM>::WAVES, THREADS = 64 * WAVES, AHEAD = StripLayout<FORM>::AHEAD;
    static_assert(MODE == MODE_NONE || mode_is_wave_level(MODE), "no scheme that compares across wavefronts");

    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int M = p.M, N = p.N, nkt = p.K / BK, pitch = p.strip_pitch;
    char* const strip = smem + nkt * LAY::B_TILE;
    const int strip_bytes = p.strip_rows * pitch;
    int* const table = reinterpret_cast<int*>(strip + strip_buffers(FORM) * strip_bytes);   // STRIP_RUNS: where each chunk of k starts

    // contiguous runs of tiles per workgroup, consecutive runs on one die
    const int G = (int)gridDim.x;
    int run = (int)blockIdx.x;
    if ((G & 7) == 0) run = (run & 7) * (G >> 3) + (run >> 3);
    const int t_lo = (int)((long long)run * p.tiles_m / G), t_hi = (int)((long long)(run + 1) * p.tiles_m / G);

    // ---- the weights, once (the row-streaming kernel's layout)
    for (int i = wave; i < nkt * (BN / 8); i += WAVES) {
        const int t = i / (BN / 8), q = i - t * (BN / 8);
        const int n = CFG::b_row_of(q * 8 + (lane >> 3)), ck = (lane & 7) ^ ((lane >> 4) + 4 * (q & 1));
        const char* src = n < N ? p.B + ((long long)n * p.ldb + (long long)t * BK) * ESIZE + ck * 16 : g_zero_chunk + ck * 16;
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                         (__attribute__((address_space(3))) void*)(smem + i * 1024), 16, 0, 0);
    }
    int steps = nkt * 4;
    if constexpr (FORM == STRIP_RUNS) {
        // chunk q of k: filter row q / cpr, chunk q % cpr of its run; past the last one (the zero weights that
        // fill up a k step) the last one again
        const int cpr = p.strip_seg * ESIZE / 16, chunks = p.KH * cpr;
        steps = (chunks + 1) >> 1;
        for (int q = tid; q < 8 * nkt; q += THREADS) {
            const int c = q < chunks ? q : chunks - 1;
            const int kh = c / cpr;
            table[((q & 1) * nkt + (q >> 3)) * 4 + ((q >> 1) & 3)] = kh * pitch + (c - kh * cpr) * 16;
        }
    }

    // ---- the strip's copy: chunk i = tid + THREADS u of its rows, LDS row i / (chunks of a row).  `from`: its source's
    // distance from the strip's first input row, -1: border only.  The two chunks of a row that the input row's ends
    // cut (STRIP_RUNS: a border of channels fills no chunk) are left to one lane each, which reads them from within
    // the row and shifts them: four wavefronts' work on one chunk instead of everyone's on all
    const int pixB = p.Cin * ESIZE, WB = p.W * pixB, padB = p.pad * pixB;
    const int Hv = (p.OH - 1) * p.stride + p.KH;
    const int row_chunks = pitch >> 4, all_chunks = p.strip_rows * row_chunks;
    const int left = padB >> 4, right = (padB + WB) >> 4;   // chunks of a row that the input row's ends cut, if they do
    const bool cut_left = (padB & 15) != 0, cut_right = ((padB + WB) & 15) != 0;
    constexpr int NEVER = 0x7fffffff;
    int slot[AHEAD], from[AHEAD], to[AHEAD];
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) {
        const int i = tid + THREADS * u;
        slot[u] = i / row_chunks;
        const int j = i - slot[u] * row_chunks, e0 = j * 16 - padB;
        from[u] = e0 >= 0 && e0 + 16 <= WB ? slot[u] * WB + e0 : -1;
        if constexpr (FORM == STRIP_RUNS) to[u] = i * 16;
        else to[u] = slot[u] * pitch + (j >> 3) * 128 + ((j & 7) ^ ((j >> 4) & 7)) * 16;   // (pixel j / 8)
        if (i >= all_chunks || (FORM == STRIP_RUNS && ((cut_left && j == left) || (cut_right && j == right)))) slot[u] = NEVER;
    }
    const bool ends = FORM == STRIP_RUNS && wave < STRIP_ROWS_MAX / 32;   // lanes 2 r, 2 r + 1: the ends of row r
    int e_slot = NEVER, e_from = -1, e_to = 0, e_bits = 0;   // bits > 0: towards higher addresses
    if (ends) {
        const int r = tid >> 1;
        if (r < p.strip_rows && (tid & 1 ? cut_right : cut_left)) {
            e_slot = r;
            e_from = r * WB + (tid & 1 ? WB - 16 : 0);
            e_bits = 8 * (tid & 1 ? (WB - 16) - (right * 16 - padB) : padB - left * 16);
            e_to = r * pitch + (tid & 1 ? right : left) * 16;
        }
    }
    i32x4 pre[AHEAD], pre_end = {0, 0, 0, 0};
    // the strip whose input is in `pre`: input rows, virtual row of the first; output column and row of its first row of C
    int n_rows = 0, v_pre = 0, c_img = 0, c_oh, c_ow;
    {
        const int m0 = t_lo * BM, r0 = m0 / p.OW;
        c_img = r0 / p.OH;
        c_oh = r0 - c_img * p.OH;
        c_ow = m0 - r0 * p.OW;
    }
    const unsigned by_ow = 0xffffffffu / (unsigned)p.OW + 1u;   // x / OW = x by_ow >> 32 (x below 2^16, OW from 2 on)
    const int d_oh = WAVES * BM / p.OW, d_ow = WAVES * BM - d_oh * p.OW;
    auto fetch = [&](int t) {
        const int tiles = t + WAVES < t_hi ? WAVES : t_hi - t;
        const int last = tiles * BM < M - t * BM ? tiles * BM - 1 : M - t * BM - 1;
        const int down = (int)__umulhi((unsigned)(c_ow + last), by_ow);
        // (the strip's rows meet at most two images)
        n_rows = down * p.stride + p.KH + (c_oh + down >= p.OH ? p.KH - p.stride : 0);
        const int ihp0 = c_oh * p.stride;
        v_pre = c_img * Hv + ihp0;
        const char* const base = p.A + ((long long)c_img * p.H + ihp0 - p.pad) * WB;
        if (c_oh + down < p.OH && ihp0 >= p.pad && ihp0 - p.pad + n_rows <= p.H) {
            // all of it inside one image (most strips): rows and their chunks lie in order.  (The rows alone do not tell:
            // at an image's foot there can be as many that no window reaches as the next image's first windows need)
            const unsigned end = (unsigned)(n_rows * WB);
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) pre[u] = ld16u((unsigned)from[u] < end ? base + from[u] : g_zero_chunk);
            if (ends) pre_end = ld16u((unsigned)e_from < end ? base + e_from : g_zero_chunk);
        } else {
        const int over = Hv - ihp0, skip = (Hv - p.H) * WB;   // first row of the next image
        auto source = [&](int sl, int fr) {
            const bool next = sl >= over;
            const int ih = sl - (next ? over : -ihp0) - p.pad;
            const bool ok = sl < n_rows && fr >= 0 && (unsigned)ih < (unsigned)p.H;
            return ok ? base + (fr - (next ? skip : 0)) : g_zero_chunk;
        };
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) pre[u] = ld16u(source(slot[u], from[u]));
        if (ends) pre_end = ld16u(source(e_slot, e_from));
        }
        // on to the next strip's first row of C
        c_ow += d_ow;
        c_oh += d_oh;
        if (c_ow >= p.OW) {
            c_ow -= p.OW;
            ++c_oh;
        }
        while (c_oh >= p.OH) {
            c_oh -= p.OH;
            ++c_img;
        }
    };
    auto place = [&](char* buf) {
#pragma unroll
        for (int u = 0; u < AHEAD; ++u)
            if (slot[u] < n_rows) *reinterpret_cast<i32x4*>(buf + to[u]) = pre[u];
        if (ends && e_slot < n_rows) {
            typedef unsigned long long u64x2 __attribute__((ext_vector_type(2)));
            u64x2 w = bitcast<u64x2>(pre_end);
            const int b = e_bits < 0 ? -e_bits : e_bits, c = b & 63;
            if (e_bits > 0) {
                if (b >= 64) w = u64x2{0ull, w[0]};
                if (c) w = u64x2{w[0] << c, (w[1] << c) | (w[0] >> (64 - c))};
            } else {
                if (b >= 64) w = u64x2{w[1], 0ull};
                if (c) w = u64x2{(w[0] >> c) | (w[1] << (64 - c)), w[1] >> c};
            }
            *reinterpret_cast<i32x4*>(buf + e_to) = bitcast<i32x4>(w);
        }
    };

    // ---- this lane's row of the wavefront's tile: output column, output row of its image, virtual row
    // of its window's top; WAVES tiles further on with every strip
    const int frow = lane & 31, fgrp = lane >> 5, fx = (lane >> 1) & 7;
    int pos[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) pos[kk] = frow * ROWB + ((2 * kk + fgrp) ^ fx) * 16;
    int ow, oh, v;
    {
        const long long m = (long long)(t_lo + wave) * BM + frow;
        const int mm = m < M ? (int)m : 0;
        const int r = mm / p.OW, img = r / p.OH;
        ow = mm - r * p.OW;
        oh = r - img * p.OH;
        v = img * Hv + oh * p.stride;
    }
    auto next_rows = [&]() {
        ow += d_ow;
        int down = d_oh;
        if (ow >= p.OW) {
            ow -= p.OW;
            ++down;
        }
        oh += down;
        v += down * p.stride;
        while (oh >= p.OH) {
            oh -= p.OH;
            v += Hv - p.OH * p.stride;
        }
    };

    Acc acc[1][TN];
    constexpr int NCHK = CheckRegs<CFG, MODE>::N;
    Acc chk[NCHK];
    // fragments of DIST steps (a k tile has four); those of the step DIST further on are read as each step's are multiplied
    constexpr int DIST = FORM == STRIP_RUNS ? 2 : 4;
    i32x4 fa[DIST], fb[DIST][TN];
    const char* top = strip;   // this lane's window in the strip
    int x0 = 0;
    int kh = 0, kw = 0;
    auto read_tap = [&](int kt, i32x4& off) -> const char* {
        if constexpr (FORM == STRIP_RUNS) {
            off = *reinterpret_cast<const i32x4*>(table + (fgrp * nkt + kt) * 4);
            return top;
        } else {
            const int x = x0 + kw, key = (x >> 1) & 7;
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) off[kk] = ((2 * kk + fgrp) ^ key) * 16;
            const char* const px = top + kh * pitch + x * 128;
            if (++kw == p.KW) {
                kw = 0;
                ++kh;
            }
            return px;
        }
    };
    auto read_step = [&](const char* px, const i32x4& off, const char* bt, int kk) {
        struct __attribute__((packed, aligned(4))) Any { i32x4 v; };   // (runs start at multiples of four bytes)
        if constexpr (FORM == STRIP_RUNS) fa[kk % DIST] = reinterpret_cast<const Any*>(px + off[kk])->v;
        else fa[kk % DIST] = *reinterpret_cast<const i32x4*>(px + off[kk]);
#pragma unroll
        for (int c = 0; c < TN; ++c) fb[kk % DIST][c] = *reinterpret_cast<const i32x4*>(bt + c * 32 * ROWB + pos[kk]);
    };
    auto multiply = [&](int kk) {
        const i32x4 a[1] = {fa[kk % DIST]};
#pragma unroll
        for (int c = 0; c < TN; ++c) acc[0][c] = MMA::run(a[0], fb[kk % DIST][c], acc[0][c]);
        if constexpr (mode_is_wave_level(MODE)) check_step<CFG, MODE>(a, fb[kk % DIST], chk);
    };

    if (t_lo < t_hi) fetch(t_lo);
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));   // (the weights as well)
    char* buf = strip;
    for (int t = t_lo; t < t_hi; t += WAVES) {
        place(buf);
        const int v0 = v_pre;
        __syncthreads();
        if (t + WAVES < t_hi) fetch(t + WAVES);
        const int tile_m = t + wave;
        if (tile_m < t_hi) {
            // (rows past M read the strip's first row)
            const bool inside = frow < M - tile_m * BM;
            top = buf + (inside ? (v - v0) * pitch : 0);
            x0 = inside ? ow * p.stride : 0;
            if constexpr (FORM == STRIP_RUNS) top += x0 * pixB;
            kh = kw = 0;
            i32x4 off;
            const char* px = read_tap(0, off);
#pragma unroll
            for (int kk = 0; kk < DIST; ++kk) read_step(px, off, smem, kk);
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[0][j][r] = 0;
            clear_check<CFG, MODE, true>(chk);
            const char* bt = smem;
            for (int kt = 0; kt + 1 < nkt; ++kt) {
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) {
                    multiply(kk);
                    if (kk + DIST == 4) {
                        px = read_tap(kt + 1, off);
                        bt += LAY::B_TILE;
                    }
                    read_step(px, off, bt, (kk + DIST) & 3);
                }
                if constexpr (INJ) {
                    if (kt == p.f_kt) inject_fault<CFG>(acc, p, TileCoords<CFG>(tile_m, 0, 0));
                }
            }
            // (the last k tile: no more steps than there are chunks)
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                if (kk == 0 || FORM == STRIP_TAPS || 4 * (nkt - 1) + kk < steps) multiply(kk);
                if (kk + DIST < 4) read_step(px, off, bt, kk + DIST);
            }
            if (M - tile_m * BM < BM) {
                // rows past M count as zeros
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const bool past = 8 * (r >> 2) + 4 * fgrp + (r & 3) >= M - tile_m * BM;
#pragma unroll
                    for (int c = 0; c < TN; ++c) acc[0][c][r] = past ? 0.f : acc[0][c][r];
                    if constexpr (mode_is_wave_level(MODE)) {
#pragma unroll
                        for (int c = 0; c < NCHK; ++c) chk[c][r] = past ? 0.f : chk[c][r];
                    }
                }
            }
            if constexpr (INJ) {
                if (p.f_kt < 0) inject_fault<CFG>(acc, p, TileCoords<CFG>(tile_m, 0, 0));
            }
            epilogue<CFG, MODE>(acc, chk, p, tile_m, 0, nullptr, true, 0);
            next_rows();
        }
        // with two buffers, whoever writes the next strip has met everyone behind their use of the one before this
        if constexpr (strip_buffers(FORM) == 2) buf = buf == strip ? strip + strip_bytes : strip;
        else __syncthreads();   // everyone is done with the strip
    }
}

}  // namespace abft
