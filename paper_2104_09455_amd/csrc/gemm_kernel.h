// Generic ABFT-protected MFMA GEMM kernel for gfx950 (MI355X): any shape, alignment,
// weight layout, and convolutions read as an implicit im2col matrix.
//
// Data flow per workgroup: global loads -> registers -> LDS (double buffered, padded rows) ->
// ds_read_b128 MFMA fragments -> accumulators -> checksum epilogue -> C.  Rows that are contiguous
// along k are read 16 bytes at a time whatever their alignment (the last chunk of a row from the
// last 16 bytes of the row, shifted down); weights stored K x N are read four bytes of a row at a
// time, eight rows of k per thread, and turned in registers on the way to LDS.  Only convolutions
// whose channels fill no chunk, and rows of less than 16 bytes, are gathered by the element.
// Bound: LDS traffic and the latency of a k tile's loads (one tile in registers on its way, one in LDS, per
// group of wavefronts), so where the chip has room KG groups of wavefronts share a tile along k.  Loaders chosen
// at run time with a condition per lane / at compile time without one, unprotected: 511 x 1000 x 2047
// fp16, weights K x N, 19.3 / 16.4 us (thread-level 21.4 / 18.3), N x K 19.1 / 16.2; 2048 x 2048 x 2047 65 / 38;
// 2048 x 4096 x 4096, weights K x N, 117 / 107, int8 77 / 69 (thread-level 175 / 131); 1 x 512 x 13 3.1 / 2.5.
#pragma once
#include "gemm_common.h"

namespace abft {

// ---------------------------------------------------------------------------
// The kernel.  KG groups of CFG::THREADS threads each own the whole workgroup tile and take the k
// tiles t with t % KG == group, each with LDS buffers of its own; at the end the groups' partial
// tiles (and redundant accumulators) are added in group order and group 0 checks and stores.
// LD: how the operands are read.  VEC: both in aligned 16-byte chunks (a_vec and b_vec); an instance of its own,
// since the other loaders' registers and branches cost such products a fifth (4000 x 4000 x 1000 fp16
// unprotected 74 us, so 59; int8 thread-level, K = 4016, 283 / 199; 5 x 5 convolution 40 -> 120 on 100352 rows 76 / 53).
// ROWS: both contiguous along k, at any alignment; TURN: A so, weights K x N.  These know their loaders at compile
// time; a load is a base that the wavefront shares and 32 bits per lane, without a condition (what lies outside reads
// something that is inside and becomes zeros on the way to LDS, in the tiles that have such).  64-bit products per
// load, a condition each, and the loads behind the products / so, thread-level fp16, weights K x N, us: 2048 x 4096 x 4096
// 113 / 97, 1900 x 4000 x 4000 121 / 115, 16 x 4096 x 4096 25.6 / 21.5, 1 x 1024 x 1024 8.5 / 7.2; 2000 x 600 x 4090 60 / 58.  (Two or three k
// tiles on their way in registers: 511 x 1000 x 2047 15.4 -> 16.5, 17.5: the tiles read past the end cost more.)
// TURN_RUNS: weights K x N of 2 GiB and more, whose offsets start again with every run of k.  ANY / 64-bit products / so, us:
// 64 x 65536 x 20000 fp16 thread-level 774 / 740 / 648, unprotected 652 / 579 / 508, 8 x 152064 x 8192 bf16 495 / 456 / 456.  (For all weights:
// the four-group tile 128 x 2048 x 4096 18.1 -> 19.3, 16 x 4096 x 4096 19.8 -> 20.6.)
// ---------------------------------------------------------------------------
enum { LD_ANY = 0, LD_VEC = 1, LD_ROWS = 2, LD_TURN = 3, LD_TURN_RUNS = 4 };
template <class CFG, int MODE, bool INJ, bool CONV, int KG, int LD>
__global__ __launch_bounds__(CFG::THREADS * KG) __attribute__((amdgpu_waves_per_eu(INJ || KG > 1 ? 1 : min_waves_per_simd<CFG, MODE>())))
void gemm_kernel(const GemmArgs p) {
    typedef Mma<CFG::DT, CFG::MI> MMA;
    typedef typename MMA::Acc Acc;
    typedef typename MMA::AccT AccT;
    constexpr int MI = CFG::MI, TM = CFG::TM, TN = CFG::TN;
    constexpr int ESIZE = CFG::ESIZE, EPC = CFG::EPC;
    constexpr int BM = CFG::BM, BN = CFG::BN, BK = CFG::BK, BKB = CFG::BKB;
    constexpr int STRIDE = CFG::LDS_STRIDE, CPR = CFG::CPR, RPP = CFG::ROWS_PER_PASS;
    constexpr int NA = CFG::NA, NB = CFG::NB;
    constexpr int KSTEPS = BKB / MMA::KBYTES;
    constexpr int NGRP = 64 / MI;  // k-groups per fragment (2 or 4)
    constexpr bool IS_INT = CFG::DT == DT_I8;

    extern __shared__ __attribute__((aligned(16))) char smem_all[];

    const int grp = KG > 1 ? __builtin_amdgcn_readfirstlane((int)threadIdx.x / CFG::THREADS) : 0;
    const int tid = KG > 1 ? (int)threadIdx.x - grp * CFG::THREADS : (int)threadIdx.x;
    char* const smem = smem_all + grp * CFG::LDS_BYTES;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wave_m = wave / CFG::WAVES_N, wave_n = wave % CFG::WAVES_N;
    const int lrow = lane % MI, lgrp = lane / MI;

    int tile_m, tile_n;
    generic_tile_of_block((int)blockIdx.x, p.tiles_m, p.tiles_n, tile_m, tile_n);
    const int bm0 = tile_m * BM, bn0 = tile_n * BN;

    const int M = p.M, N = p.N, K = p.K;
    const int nkt = (K + BK - 1) / BK;

    // this thread's chunk column (same for all its chunks) and first row
    const int kc = tid % CPR;
    const int r0 = tid / CPR;

    // ---- implicit-GEMM row state: image offset and top-left input pixel per chunk row
    constexpr int NCONV = CONV ? NA : 1;
    long long a_row_off[NCONV];
    int a_ih0[NCONV], a_iw0[NCONV];
    int tap_c = 0, tap_kh = 0, tap_kw = 0;  // decomposition of this thread's k for the current tile
    if constexpr (CONV) {
#pragma unroll
        for (int t = 0; t < NA; ++t) {
            int m = bm0 + r0 + t * RPP;
            int mm = m < M ? m : 0;
            int img = mm / (p.OH * p.OW);
            int rem = mm - img * (p.OH * p.OW);
            int oh = rem / p.OW, ow = rem - oh * p.OW;
            a_row_off[t] = (long long)img * p.imgpitch;
            a_ih0[t] = oh * p.stride - p.pad;
            a_iw0[t] = ow * p.stride - p.pad;
        }
        int k = grp * BK + kc * EPC;
        int tap = k / p.Cin;
        tap_c = k - tap * p.Cin;
        tap_kh = tap / p.KW;
        tap_kw = tap - tap_kh * p.KW;
    } else {
        a_row_off[0] = 0;
        a_ih0[0] = 0;
        a_iw0[0] = 0;
    }

    // rows read 16 bytes at a time at any alignment: a chunk that K cuts short is read as the last 16
    // bytes of its row and shifted down when it goes to LDS
    constexpr bool VEC = LD == LD_VEC, STREAM = LD >= LD_ROWS;
    constexpr bool ROWS = LD == LD_ROWS;
    static_assert(!STREAM || !CONV, "matrices only");
    const bool a_vec = VEC || (!STREAM && p.a_vec), b_vec = VEC || (!STREAM && p.b_vec);
    const bool a_row = !STREAM && (!CONV && !a_vec && K >= EPC);
    const bool b_row = !STREAM && !b_vec && p.b_sk == 1 && K >= EPC;
    // weights stored K x N: units of eight k times four bytes of n (four bytes of a row end inside it)
    constexpr int NPD = 4 / ESIZE;                     // columns per four bytes
    constexpr int NGN = BN / NPD;                      // such groups per row of the tile
    constexpr int UNITS = NB / 2;                      // units per thread
    static_assert(NB % 2 == 0 && CFG::THREADS * UNITS == NGN * (BK / 8), "units of the transposing loader");
    const bool b_turn = !STREAM && !b_vec && !b_row && p.b_sn == 1 && N >= NPD;
    auto load_a = [&](int kt, i32x4(&regs)[NA]) {
        const int k0 = kt * BK + kc * EPC;  // first k of this thread's chunk
        if constexpr (!CONV) {
            if (a_row) {
                const int ks = k0 + EPC <= K ? k0 : K - EPC;
#pragma unroll
                for (int t = 0; t < NA; ++t) {
                    const int m = bm0 + r0 + t * RPP;
                    i32x4 v = {0, 0, 0, 0};
                    if (m < M && k0 < K) v = ld16u(p.A + ((long long)m * p.lda + ks) * ESIZE);
                    regs[t] = v;
                }
            } else if (a_vec) {
#pragma unroll
                for (int t = 0; t < NA; ++t) {
                    int m = bm0 + r0 + t * RPP;
                    i32x4 v = {0, 0, 0, 0};
                    if (m < M && k0 < K) v = ld16(p.A + ((long long)m * p.lda + k0) * ESIZE);
                    regs[t] = v;
                }
            } else {
#pragma unroll
                for (int t = 0; t < NA; ++t) {
                    int m = bm0 + r0 + t * RPP;
                    int nv = (m < M) ? (K - k0) : 0;
                    regs[t] = gather16<ESIZE>(p.A + ((long long)(m < M ? m : 0) * p.lda + k0) * ESIZE, ESIZE, nv);
                }
            }
        } else {
        if (a_vec) {
            // a chunk never straddles a filter tap (Cin is a multiple of the chunk length)
#pragma unroll
            for (int t = 0; t < NA; ++t) {
                int m = bm0 + r0 + t * RPP;
                int ih = a_ih0[t] + tap_kh, iw = a_iw0[t] + tap_kw;
                i32x4 v = {0, 0, 0, 0};
                if (m < M && k0 < K && ih >= 0 && ih < p.H && iw >= 0 && iw < p.W)
                    v = ld16(p.A + (a_row_off[t] + (long long)ih * p.rowpitch + (long long)iw * p.pix + tap_c) * ESIZE);
                regs[t] = v;
            }
        } else {
            // element gather (channel counts that are no multiple of the chunk): the filter taps of
            // this thread's EPC values of k are the same for all its rows, so they are taken apart once
            int e_kh[EPC], e_kw[EPC];
            long long e_off[EPC];
            {
                int c = tap_c, kh = tap_kh, kw = tap_kw;
#pragma unroll
                for (int e = 0; e < EPC; ++e) {
                    e_kh[e] = k0 + e < K ? kh : (1 << 28);  // beyond K: never in range
                    e_kw[e] = kw;
                    e_off[e] = kh * p.rowpitch + (long long)kw * p.pix + c;
                    if (++c == p.Cin) {
                        c = 0;
                        if (++kw == p.KW) {
                            kw = 0;
                            ++kh;
                        }
                    }
                }
            }
#pragma unroll
            for (int t = 0; t < NA; ++t) {
                const int m = bm0 + r0 + t * RPP;
                i32x4 v = {0, 0, 0, 0};
                if (m < M) {
                    const char* base = p.A + (a_row_off[t] + a_ih0[t] * p.rowpitch + (long long)a_iw0[t] * p.pix) * ESIZE;
#pragma unroll
                    for (int e = 0; e < EPC; ++e) {
                        const unsigned ih = (unsigned)(a_ih0[t] + e_kh[e]), iw = (unsigned)(a_iw0[t] + e_kw[e]);
                        unsigned x = 0;
                        if (ih < (unsigned)p.H && iw < (unsigned)p.W) {
                            const char* src = base + e_off[e] * ESIZE;
                            x = ESIZE == 2 ? (unsigned)*reinterpret_cast<const unsigned short*>(src)
                                           : (unsigned)*reinterpret_cast<const unsigned char*>(src);
                        }
                        if constexpr (ESIZE == 2) v[e >> 1] |= (int)(x << (16 * (e & 1)));
                        else v[e >> 2] |= (int)(x << (8 * (e & 3)));
                    }
                }
                regs[t] = v;
            }
        }
        }
    };
    // advance this thread's filter-tap decomposition to its group's next k-tile
    auto advance_taps = [&]() {
        if constexpr (CONV) {
            tap_c += KG * BK;
            while (tap_c >= p.Cin) {
                tap_c -= p.Cin;
                if (++tap_kw == p.KW) {
                    tap_kw = 0;
                    ++tap_kh;
                }
            }
        }
    };
    auto load_b = [&](int kt, i32x4(&regs)[NB]) {
        const int k0 = kt * BK + kc * EPC;
        if (b_row) {
            const int ks = k0 + EPC <= K ? k0 : K - EPC;
#pragma unroll
            for (int t = 0; t < NB; ++t) {
                const int n = bn0 + r0 + t * RPP;
                i32x4 v = {0, 0, 0, 0};
                if (n < N && k0 < K) v = ld16u(p.B + ((long long)n * p.ldb + ks) * ESIZE);
                regs[t] = v;
            }
        } else if (b_turn) {
            // (rows past K and columns past N read valid elements, dropped on the way to LDS)
#pragma unroll
            for (int t = 0; t < UNITS; ++t) {
                const int u = tid + t * CFG::THREADS, n = bn0 + (u % NGN) * NPD;
                const char* src = p.B + (long long)(n + NPD <= N ? n : N - NPD) * ESIZE;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int k = kt * BK + (u / NGN) * 8 + e;
                    regs[2 * t + (e >> 2)][e & 3] = ld4u(src + (long long)(k < K ? k : K - 1) * p.ldb * ESIZE);
                }
            }
        } else if (b_vec) {
#pragma unroll
            for (int t = 0; t < NB; ++t) {
                int n = bn0 + r0 + t * RPP;
                i32x4 v = {0, 0, 0, 0};
                if (n < N && k0 < K) v = ld16(p.B + ((long long)n * p.ldb + k0) * ESIZE);
                regs[t] = v;
            }
        } else {
#pragma unroll
            for (int t = 0; t < NB; ++t) {
                int n = bn0 + r0 + t * RPP;
                int nv = (n < N) ? (K - k0) : 0;
                regs[t] = gather16<ESIZE>(p.B + ((long long)(n < N ? n : 0) * p.b_sn + (long long)k0 * p.b_sk) * ESIZE,
                                          p.b_sk * ESIZE, nv);
            }
        }
    };
    // units of the transposing loader, turned on the way to LDS
    auto store_turned = [&](char* bs, int kt, const i32x4(&rb)[NB]) {
        const bool cut = (kt + 1) * BK > K;
        const bool edge = cut || bn0 + BN > N;
#pragma unroll
        for (int t = 0; t < UNITS; ++t) {
            const int u = tid + t * CFG::THREADS, nl = (u % NGN) * NPD, kl = (u / NGN) * 8;
            unsigned d[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) d[e] = (unsigned)rb[2 * t + (e >> 2)][e & 3];
            if (edge) {
                const int over = bn0 + nl + NPD - N;   // columns of the group beyond N (read early by as many)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    if (over > 0) d[e] = over >= NPD ? 0u : d[e] >> (8 * ESIZE * over);
                    if (kt * BK + kl + e >= K) d[e] = 0u;
                }
            }
            if constexpr (ESIZE == 2) {
                i32x4 c0, c1;   // eight k of column nl, of column nl + 1
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    c0[q] = (int)__builtin_amdgcn_perm(d[2 * q + 1], d[2 * q], 0x05040100u);
                    c1[q] = (int)__builtin_amdgcn_perm(d[2 * q + 1], d[2 * q], 0x07060302u);
                }
                *reinterpret_cast<i32x4*>(bs + nl * STRIDE + kl * 2) = c0;
                *reinterpret_cast<i32x4*>(bs + (nl + 1) * STRIDE + kl * 2) = c1;
            } else {
                i32x2 c[4];     // eight k of each of four columns
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const unsigned x01 = __builtin_amdgcn_perm(d[4 * h + 1], d[4 * h], 0x05010400u);
                    const unsigned x23 = __builtin_amdgcn_perm(d[4 * h + 3], d[4 * h + 2], 0x05010400u);
                    const unsigned y01 = __builtin_amdgcn_perm(d[4 * h + 1], d[4 * h], 0x07030602u);
                    const unsigned y23 = __builtin_amdgcn_perm(d[4 * h + 3], d[4 * h + 2], 0x07030602u);
                    c[0][h] = (int)__builtin_amdgcn_perm(x23, x01, 0x05040100u);
                    c[1][h] = (int)__builtin_amdgcn_perm(x23, x01, 0x07060302u);
                    c[2][h] = (int)__builtin_amdgcn_perm(y23, y01, 0x05040100u);
                    c[3][h] = (int)__builtin_amdgcn_perm(y23, y01, 0x07060302u);
                }
#pragma unroll
                for (int n = 0; n < 4; ++n) *reinterpret_cast<i32x2*>(bs + (nl + n) * STRIDE + kl) = c[n];
            }
        }
    };
    auto store_tiles = [&](int buf, int kt, const i32x4(&ra)[NA], const i32x4(&rb)[NB]) {
        char* as = smem + buf * CFG::STAGE_BYTES;
        char* bs = as + BM * STRIDE;
        // (bytes by which a chunk that K cuts short was read early; a whole chunk: 0)
        const int k0 = kt * BK + kc * EPC;
        const int early = k0 < K && k0 + EPC > K ? (k0 + EPC - K) * ESIZE : 0;
        const bool cut = (kt + 1) * BK > K;
        if (a_row && cut) {
#pragma unroll
            for (int t = 0; t < NA; ++t)
                *reinterpret_cast<i32x4*>(as + (r0 + t * RPP) * STRIDE + kc * 16) = shift_down(ra[t], early);
        } else {
#pragma unroll
            for (int t = 0; t < NA; ++t)
                *reinterpret_cast<i32x4*>(as + (r0 + t * RPP) * STRIDE + kc * 16) = ra[t];
        }
        if (b_turn) {
            store_turned(bs, kt, rb);
        } else if (b_row && cut) {
#pragma unroll
            for (int t = 0; t < NB; ++t)
                *reinterpret_cast<i32x4*>(bs + (r0 + t * RPP) * STRIDE + kc * 16) = shift_down(rb[t], early);
        } else {
#pragma unroll
            for (int t = 0; t < NB; ++t)
                *reinterpret_cast<i32x4*>(bs + (r0 + t * RPP) * STRIDE + kc * 16) = rb[t];
        }
    };

    // ---- ROWS and TURN: bases that the workgroup shares, this thread's rows as offsets from them
    const unsigned kb = (unsigned)K * ESIZE, lda_b = (unsigned)(p.lda * ESIZE), ldb_b = (unsigned)(p.ldb * ESIZE);
    const char* const a_base = p.A + (long long)bm0 * p.lda * ESIZE;
    const char* const b_base = ROWS ? p.B + (long long)bn0 * p.ldb * ESIZE : p.B;
    unsigned a_off[NA], b_off[ROWS ? NB : UNITS], b_col[ROWS ? 1 : UNITS], a_out = 0, b_out = 0;
    if constexpr (STREAM) {
        // (rows outside read chunks of 16 aligned bytes near the first row's, the same ones for all: off the dword, a row each costs
        // the vector memory path four times as much; up to 15 bytes behind the first row's, so only where there is a second)
        auto outside = [](const char* base, int rows) { return rows > 1 ? (unsigned)(-reinterpret_cast<uintptr_t>(base) & 15u) : 0u; };
        a_out = outside(a_base, M - bm0);
#pragma unroll
        for (int t = 0; t < NA; ++t) a_off[t] = r0 + t * RPP < M - bm0 ? (unsigned)(r0 + t * RPP) * lda_b : a_out;
        if constexpr (ROWS) {
            b_out = outside(b_base, N - bn0);
#pragma unroll
            for (int t = 0; t < NB; ++t) b_off[t] = r0 + t * RPP < N - bn0 ? (unsigned)(r0 + t * RPP) * ldb_b : b_out;
        } else {
#pragma unroll
            for (int t = 0; t < UNITS; ++t) {
                const int u = tid + t * CFG::THREADS;
                b_col[t] = (unsigned)(min(bn0 + (u % NGN) * NPD, N - NPD) * ESIZE);
                b_off[t] = (unsigned)((u / NGN) * 8) * ldb_b + b_col[t];
            }
        }
    }
    // rows of weights K x N whose offsets stay in 31 bits: a power of two, whole k tiles
    const int b_run = LD == LD_TURN_RUNS ? 1 << (31 - __builtin_clz(0x7fffffffu / ldb_b)) : 0;
    auto chunk_from = [&](int kt) { return min((unsigned)kt * BKB + (unsigned)kc * 16, kb - 16); };   // the byte of its row
    // first: chunks beyond K as rows outside (where there is one k tile, most of its chunks may be such).  (Zeros by address there, and no
    // selects behind them: products of one k tile gain 0.05 us, 511 x 1000 x 2047 K x N loses 0.3.)
    auto stream_load = [&](int kt, i32x4(&ra)[NA], i32x4(&rb)[NB], auto first) {
        const unsigned from = chunk_from(kt);
        const bool beyond = decltype(first)::value && (unsigned)kt * BKB + (unsigned)kc * 16 >= kb;
#pragma unroll
        for (int t = 0; t < NA; ++t) ra[t] = ld16u(a_base + (beyond ? a_out : a_off[t] + from));
        if constexpr (ROWS) {
#pragma unroll
            for (int t = 0; t < NB; ++t) rb[t] = ld16u(b_base + (beyond ? b_out : b_off[t] + from));
        } else {
            // (rows past K read the last one, dropped on the way to LDS)
            const int k0 = min(kt, nkt - 1) * BK;
            const int from_k = LD == LD_TURN_RUNS ? k0 & -b_run : 0, rows = LD == LD_TURN_RUNS ? min(K - from_k, b_run) : K;
            const char* const run = b_base + (long long)from_k * p.ldb * ESIZE;
#pragma unroll
            for (int t = 0; t < UNITS; ++t) {
                const unsigned row0 = (unsigned)(k0 - from_k) * ldb_b + b_off[t];
                const unsigned last = (unsigned)(rows - 1) * ldb_b + b_col[t];
#pragma unroll
                for (int e = 0; e < 8; ++e) rb[2 * t + (e >> 2)][e & 3] = ld4u(run + min(row0 + e * ldb_b, last));
            }
        }
    };
    auto stream_store = [&](int buf, int kt, i32x4(&ra)[NA], i32x4(&rb)[NB]) {
        char* as = smem + buf * CFG::STAGE_BYTES;
        char* bs = as + BM * STRIDE;
        const unsigned from = chunk_from(kt);
        const i32x4 zero = {0, 0, 0, 0};
        if ((kt + 1) * BK > K) {
            // (a chunk that K cuts was read early by so many bytes; one beyond K counts as zeros)
            const int early = (int)((unsigned)kt * BKB + (unsigned)kc * 16 - from);
#pragma unroll
            for (int t = 0; t < NA; ++t) ra[t] = early < 16 ? shift_down(ra[t], early) : zero;
            if constexpr (ROWS) {
#pragma unroll
                for (int t = 0; t < NB; ++t) rb[t] = early < 16 ? shift_down(rb[t], early) : zero;
            }
        }
        if (bm0 + BM > M) {
#pragma unroll
            for (int t = 0; t < NA; ++t) ra[t] = bm0 + r0 + t * RPP < M ? ra[t] : zero;
        }
#pragma unroll
        for (int t = 0; t < NA; ++t) *reinterpret_cast<i32x4*>(as + (r0 + t * RPP) * STRIDE + kc * 16) = ra[t];
        if constexpr (ROWS) {
            if (bn0 + BN > N) {
#pragma unroll
                for (int t = 0; t < NB; ++t) rb[t] = bn0 + r0 + t * RPP < N ? rb[t] : zero;
            }
#pragma unroll
            for (int t = 0; t < NB; ++t) *reinterpret_cast<i32x4*>(bs + (r0 + t * RPP) * STRIDE + kc * 16) = rb[t];
        } else {
            store_turned(bs, kt, rb);
        }
    };

    Acc acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < MMA::NACC; ++r) acc[i][j][r] = 0;
    constexpr int NCHK = CheckRegs<CFG, MODE>::N;
    Acc chk[NCHK];
    clear_check<CFG, MODE>(chk);

    // the products of one k tile, from LDS buffer `cur`
    auto multiply = [&](int cur) {
        const char* as = smem + cur * CFG::STAGE_BYTES + (wave_m * CFG::WM + lrow) * STRIDE + lgrp * 16;
        const char* bs = smem + cur * CFG::STAGE_BYTES + BM * STRIDE + (wave_n * CFG::WN + lrow) * STRIDE + lgrp * 16;
#pragma unroll
        for (int kk = 0; kk < KSTEPS; ++kk) {
            i32x4 a[TM], b[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i)
                a[i] = *reinterpret_cast<const i32x4*>(as + i * MI * STRIDE + kk * MMA::KBYTES);
#pragma unroll
            for (int j = 0; j < TN; ++j)
                b[j] = *reinterpret_cast<const i32x4*>(bs + j * MI * STRIDE + kk * MMA::KBYTES);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[i][j] = MMA::run(a[i], b[j], acc[i][j]);
            if constexpr (mode_is_wave_level(MODE)) check_step<CFG, MODE>(a, b, chk);
        }
    };
    // (every group goes through the same number of steps: they share the workgroup's barrier)
    const int nsteps = (nkt + KG - 1) / KG;
    i32x4 ra[NA], rb[NB];
    if constexpr (STREAM) {
        static_assert(!INJ, "injected faults go through the other loaders");
        // step s: tile s + 1 of the group moves from registers to LDS, the loads of tile s + 2 go out, the products of tile s
        // (LDS buffer s % 2) run while they are on their way
        stream_load(grp, ra, rb, std::true_type{});
        if (grp < nkt) stream_store(0, grp, ra, rb);
        if (grp + KG < nkt) stream_load(grp + KG, ra, rb, std::false_type{});
        __syncthreads();
        for (int s = 0; s < nsteps; ++s) {
            const int kt = s * KG + grp;
            if (kt + KG < nkt) stream_store((s & 1) ^ 1, kt + KG, ra, rb);
            if (kt + 2 * KG < nkt) stream_load(kt + 2 * KG, ra, rb, std::false_type{});
            if (KG == 1 || kt < nkt) multiply(s & 1);
            __syncthreads();
        }
    } else {
        if (grp < nkt) {
            load_a(grp, ra);
            load_b(grp, rb);
            store_tiles(0, grp, ra, rb);
        }
        __syncthreads();

        for (int s = 0; s < nsteps; ++s) {
            const int kt = s * KG + grp;   // this group's k tile of the step (none: >= nkt)
            const int cur = s & 1;
            const bool more = kt + KG < nkt;
            if (more) {
                advance_taps();
                load_a(kt + KG, ra);
                load_b(kt + KG, rb);
            }
            if (KG == 1 || kt < nkt) multiply(cur);
            if (more) store_tiles(cur ^ 1, kt + KG, ra, rb);
            __syncthreads();
            if constexpr (INJ) {
                if (kt == p.f_kt) inject_fault<CFG>(acc, p, TileCoords<CFG>(tile_m, tile_n, wave));
            }
        }
    }
    if constexpr (INJ) {
        // a fault in a finished accumulator: that of the group holding the last k tile
        if (p.f_kt == -1 && (KG == 1 || grp == (nkt - 1) % KG)) inject_fault<CFG>(acc, p, TileCoords<CFG>(tile_m, tile_n, wave));
    }
    if constexpr (KG > 1) {
        // the other groups leave their accumulators in LDS (every buffer is free: the loop ended with a
        // barrier), group 0 adds them in group order; the checks see the added-up tile and the
        // added-up redundant accumulators (checksum products of partial products add up to the
        // checksum product of the whole, Sec. 5.2.2)
        constexpr int NCHK_OUT = mode_is_wave_level(MODE) ? NCHK : 0;
        constexpr int NV = (TM * TN + NCHK_OUT) * MMA::NACC;     // values per lane
        static_assert((KG - 1) * NV * CFG::THREADS * 4 <= KG * CFG::LDS_BYTES, "LDS for the final sum");
        AccT* red = reinterpret_cast<AccT*>(smem_all);
        if (grp > 0) {
            AccT* out = red + ((long long)(grp - 1) * NV) * CFG::THREADS + tid;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int r = 0; r < MMA::NACC; ++r) out[((i * TN + j) * MMA::NACC + r) * CFG::THREADS] = acc[i][j][r];
#pragma unroll
            for (int i = 0; i < NCHK_OUT; ++i)
#pragma unroll
                for (int r = 0; r < MMA::NACC; ++r) out[((TM * TN + i) * MMA::NACC + r) * CFG::THREADS] = chk[i][r];
        }
        __syncthreads();
        if (grp > 0) return;
#pragma unroll
        for (int g = 1; g < KG; ++g) {
            const AccT* in = red + ((long long)(g - 1) * NV) * CFG::THREADS + tid;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int r = 0; r < MMA::NACC; ++r) acc[i][j][r] += in[((i * TN + j) * MMA::NACC + r) * CFG::THREADS];
#pragma unroll
            for (int i = 0; i < NCHK_OUT; ++i)
#pragma unroll
                for (int r = 0; r < MMA::NACC; ++r) chk[i][r] += in[((TM * TN + i) * MMA::NACC + r) * CFG::THREADS];
        }
        if constexpr (INJ) {
            if (p.f_kt == -2) inject_fault<CFG>(acc, p, TileCoords<CFG>(tile_m, tile_n, wave));
        }
    }
    (void)NGRP;

    epilogue<CFG, MODE>(acc, chk, p, tile_m, tile_n, smem, true, wave);
}

}  // namespace abft
