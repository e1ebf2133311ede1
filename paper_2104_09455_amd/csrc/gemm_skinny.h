// Skinny ABFT-protected MFMA kernel for gfx950 (MI355X): products of at most sixteen rows (decoding, recommendation
// models at small batches), unprotected or under a wavefront-level scheme; rows of A and B contiguous along k, at any
// alignment.
//
// The weights' bytes are all there is to do, so the columns are spread over the chip as thinly as an MFMA allows: a
// workgroup takes 16 columns (a 16 x 16 MFMA shape: no rows of zeros beside them), eight wavefronts share its k tiles (128
// bytes; wavefront w those with t % 8 == w).  A wavefront's rows travel through registers, two k tiles ahead, and through
// its own 4 KB of LDS into fragments; no barrier before the sums.  (Sixteen wavefronts, or three tiles ahead: DLRM at
// batch 1 19.6 and 18.5 us, so 18.2, in one run on one card; 16 x 4096 x 4096 bf16 8.6 and 8.4, so 8.1.  Against the 32 x 32 tiles'
// kernel, in turn, several cards: DLRM at batch 1 25.7-26.0 -> 22.3-22.6, 16 x 4096 x 4096 bf16 8.31 -> 8.02.)
// The partial tiles meet in LDS; one wavefront per 16 x 16 block adds them in wavefront order, its checksum blocks
// likewise, compares and stores.  On a clean tile both are the same bit for bit, which is all that is looked at without a
// report: sums over the lanes are formed only where they differ.
// Rows that start off a multiple of four bytes are read in whole dwords and shifted: the vector memory path serves 16 bytes
// a lane at such addresses at a quarter of its rate (1 KB in 64 clocks, else 17).  The dwords that a row's ends share with
// what lies before and behind it are read whole, which never leaves a dword that holds some of the row.
// Bound: the latency of one round trip to the weights, then the weights' bytes and A's (as many again, from L2: 16 x
// 4096 x 4096 takes 8.0 without them).
#pragma once
#include "gemm_common.h"

namespace abft {

constexpr int SKINNY_ROWS = 16, SKINNY_WAVES = 8, SKINNY_AHEAD = 2;
// columns of a workgroup: 16; with a report 32, the columns of the comparisons that it counts on 32 x 32 tiles
constexpr int skinny_lds_bytes(int tn) { return SKINNY_WAVES * (1 + tn) * 2048; }

// Rows of at least 16 bytes.  BYTES: rows at any address; else at multiples of four bytes.  INJ: with a planted fault (test
// hook): in the sum of those of the eight shares that the tiling whose place this kernel takes has in one (p.n_parts shares, k tile t in
// share t % p.n_parts), as it stands once that share has taken all its k tiles up to p.f_kt (-1: up to the last), or in the finished sum (-2).
// The loop and the comparison are those of a call without one, and so is every other element.
template <int DT, int TN, int MODE, bool BYTES, bool INJ>
__device__ __forceinline__ void skinny_tile(const GemmArgs& p, int tile_n, char* smem) {
    typedef Mma<DT, 16> MMA;
    typedef typename MMA::Acc Acc;
    typedef typename MMA::AccT AccT;
    constexpr int ES = DT == DT_I8 ? 1 : 2, EPC = 16 / ES, KW = SKINNY_WAVES, U = SKINNY_AHEAD;
    constexpr bool IS_INT = DT == DT_I8, CHECKED = MODE != MODE_NONE;
    typedef typename std::conditional<IS_INT, long long, double>::type Wide;
    static_assert(MODE == MODE_NONE || MODE == MODE_THREAD, "one block per fragment pair: the wavefront-level schemes are the same here");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lrow = lane & 15, lgrp = lane >> 4;
    const int M = p.M, N = p.N, K = p.K, n0 = tile_n * 16 * TN;
    const int kb = K * ES, nkt = (kb + 127) >> 7;
    const int n_own = nkt > wave ? (nkt - wave + KW - 1) / KW : 0;

    // Copies: lane l takes chunk l % 8 of rows l / 8 and 8 + l / 8 of a k tile (whole lines; with a lane per row, as the
    // fragments want them, an instruction of 1 KB takes the vector memory path 64 clocks, so 17), writes them to its
    // wavefront's own 128-byte rows in LDS (position chunk ^ ((row >> 1) & 7)), and reads fragments from there: LDS
    // operations of a wavefront execute in order, so nothing has to be waited for.
    constexpr int ROWS = 1 + TN, NQ = 2 * ROWS;   // blocks of 16 rows, of 8
    char* const own = smem + wave * (ROWS * 2048);
    const int crow = lane >> 3, chunk = (lane & 7) * 16;
    const char* row[NQ];
    bool in[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int r = (q & 1) * 8 + crow, n = n0 + (q >> 1) * 16 - 16 + r;
        in[q] = q < 2 ? r < M : n < N;   // (rows outside read zeros and stay there)
        row[q] = !in[q] ? g_zero_chunk : q < 2 ? p.A + (long long)r * p.lda * ES : p.B + (long long)n * p.ldb * ES;
    }
    i32x4 v_[U][NQ];
    int more[U][BYTES ? NQ : 1], sh[U][BYTES ? NQ : 1];
    auto fetch = [&](int u, int q, const char* from) {
        if constexpr (BYTES) {
            // (addresses off the dword cost four times the path's time: whole dwords, shifted down in registers)
            const int off = (int)(reinterpret_cast<uintptr_t>(from) & 3u);
            sh[u][q] = off;
            v_[u][q] = ld16u(from - off);
            more[u][q] = ld4u(from - off + (off ? 16 : 12));
        } else {
            v_[u][q] = ld16u(from);
        }
    };
    // own tile i (k tile wave + KW i) into slot u: a whole one, and one that K may cut (a chunk beyond K: zeros; one that
    // K cuts: the last 16 bytes of the row, shifted down before they are multiplied)
    auto load_whole = [&](int u, int i) {
        const int off = (wave + KW * i) * 128 + chunk;
#pragma unroll
        for (int q = 0; q < NQ; ++q) fetch(u, q, row[q] + (in[q] ? off : 0));
    };
    auto load = [&](int u, int i) {
        const int t = wave + KW * i;
        if ((t + 1) * 128 <= kb) {
            load_whole(u, i);
        } else {
            const int off = t * 128 + chunk, from = off + 16 > kb ? kb - 16 : off;
#pragma unroll
            for (int q = 0; q < NQ; ++q) fetch(u, q, in[q] && off < kb ? row[q] + from : g_zero_chunk);
        }
    };
    const int kx = (crow >> 1) * 16;   // (rows 8 further on: the key's top bit)
    int to[2], at[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) to[h] = (h * 8 + crow) * 128 + (chunk ^ (kx + 64 * h));
#pragma unroll
    for (int s = 0; s < 2; ++s) at[s] = lrow * 128 + ((4 * s + lgrp) ^ (lrow >> 1)) * 16;
    Acc acc[TN], chk[TN];
    AccT zero = 0;
    if constexpr (CHECKED) asm("" : "+v"(zero));   // (blocks that take the same products stay apart)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            acc[j][r] = 0;
            chk[j][r] = r == 0 ? zero : 0;
        }
    const int upto = INJ && p.f_kt >= 0 ? p.f_kt : nkt - 1;
    Acc then[INJ ? TN : 1];   // this wavefront's part of the share's sum up to there
    if constexpr (INJ) {
#pragma unroll
        for (int j = 0; j < TN; ++j) then[j] = acc[j];
    }
    auto multiply = [&](int u, int i, int cut) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            i32x4 x = v_[u][q];
            if constexpr (BYTES) {
#pragma unroll
                for (int d = 0; d < 4; ++d)
                    x[d] = (int)__builtin_amdgcn_alignbyte((unsigned)(d < 3 ? x[d + 1] : more[u][q]), (unsigned)x[d], (unsigned)sh[u][q]);
            }
            if (cut) x = shift_down(x, chunk < cut && chunk + 16 > cut ? chunk + 16 - cut : 0);
            *reinterpret_cast<i32x4*>(own + (q >> 1) * 2048 + to[q & 1]) = x;
        }
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const i32x4 a = *reinterpret_cast<const i32x4*>(own + at[s]);
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const i32x4 b = *reinterpret_cast<const i32x4*>(own + (1 + j) * 2048 + at[s]);
                acc[j] = MMA::run(a, b, acc[j]);
                if constexpr (CHECKED) chk[j] = MMA::run(a, b, chk[j]);
            }
        }
        if constexpr (INJ) {
            if (wave + KW * i <= upto) {
#pragma unroll
                for (int j = 0; j < TN; ++j) then[j] = acc[j];
            }
        }
    };
    int i = 0;
    if (n_own > 2 * U) {
        // (no condition between the loads, so that the number behind the one that is waited for is known)
#pragma unroll
        for (int u = 0; u < U; ++u) load_whole(u, u);
#pragma nounroll
        for (; i + 2 * U < n_own; i += U)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                multiply(u, i + u, 0);
                load_whole(u, i + U + u);
            }
    } else {
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (u < n_own) load(u, u);
    }
#pragma nounroll
    for (; i < n_own; i += U)
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i + u < n_own) {
                const int left = kb - (wave + KW * (i + u)) * 128;
                multiply(u, i + u, left < 128 && (left & 15) ? left : 0);   // (bytes of a tile whose last chunk K cuts)
                if (i + U + u < n_own) load(u, i + U + u);
            }

    // ---- the partial tiles meet; wavefront j adds block j, in wavefront order
    __syncthreads();   // (where the operands were)
    Acc* const red = reinterpret_cast<Acc*>(smem);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        red[(wave * TN + j) * 64 + lane] = acc[j];
        if constexpr (CHECKED) red[((KW + wave) * TN + j) * 64 + lane] = chk[j];
        if constexpr (INJ) red[((2 * KW + wave) * TN + j) * 64 + lane] = then[j];
    }
    __syncthreads();
    Acc v, w;
    if (wave < TN) {
        v = red[wave * 64 + lane];
        if constexpr (CHECKED) w = red[(KW * TN + wave) * 64 + lane];
#pragma unroll
        for (int q = 1; q < KW; ++q) {
            v += red[(q * TN + wave) * 64 + lane];
            if constexpr (CHECKED) w += red[((KW + q) * TN + wave) * 64 + lane];
        }
        const int col = n0 + 16 * wave + lrow;
        if constexpr (INJ) {
            Acc part = v;
            if (p.f_kt != -2) {
#pragma unroll
                for (int r = 0; r < 4; ++r) part[r] = 0;
#pragma unroll
                for (int q = 0; q < KW; ++q)
                    if (((q ^ upto) & (p.n_parts - 1)) == 0) part += red[((2 * KW + q) * TN + wave) * 64 + lane];
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const AccT flipped = bitcast<AccT>(bitcast<unsigned>(part[r]) ^ (1u << p.f_bit));
                if (col == p.f_col && p.f_row == 4 * lgrp + r) v[r] = p.f_kt == -2 ? flipped : v[r] - part[r] + flipped;
            }
        }
        if (col < N) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 4 * lgrp + r;
                const AccT o = p.act ? relu(v[r]) : v[r];
                if (row < M) {
                    char* const dst = p.C + ((long long)row * p.ldc + col) * (IS_INT ? 4 : 2);
                    if constexpr (DT == DT_F16) *reinterpret_cast<_Float16*>(dst) = (_Float16)o;
                    else if constexpr (DT == DT_BF16) *reinterpret_cast<__bf16*>(dst) = (__bf16)o;
                    else *reinterpret_cast<int*>(dst) = o;
                }
            }
        }
    }
    if constexpr (CHECKED) {
        // comparison (Sec. 5.2.2): the sum of a 16 x 16 block against that of its checksum block.  A report counts
        // comparisons of 32 columns where the tiling's tiles are that wide, and so gets the sums of two blocks, but the larger of their
        // ratios: what raises the flag is the same with a report and without.
        static_assert(TN <= 2, "the second block's sums go through LDS");
        Wide s = 0, c = 0;
        double F2 = 0.0, ratio = 0.0;
        if (wave < TN) {
            int differ = 0;
            float f2 = 0.f;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                differ |= bitcast<int>(v[r]) ^ bitcast<int>(w[r]);
                if constexpr (!IS_INT) f2 += v[r] * v[r];
            }
            // (64 sums of squares below 2^100 add up to a finite one; one that is none fails the comparison)
            if (TN == 1 && !p.report && !__any(differ != 0 || !(f2 < 1.2676506e30f))) return;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                s += (Wide)v[r];
                c += (Wide)w[r];
            }
            s = wave_sum(s);
            c = wave_sum(c);
            bool bad = s != c;
            ratio = bad ? __builtin_huge_val() : 0.0;
            if constexpr (!IS_INT) {
                F2 = (double)wave_sum(f2);
                const double tau = p.tol_coeff * __builtin_sqrt(F2), res = __builtin_fabs(s - c);
                // a sum of squares beyond the fp32 range cannot come from a fault-free tile
                const bool finite = __builtin_isfinite(s) && __builtin_isfinite(c) && __builtin_isfinite(F2);
                bad = !finite || !(res <= tau);
                ratio = !finite ? __builtin_huge_val() : (tau > 0.0 ? res / tau : (res > 0.0 ? __builtin_huge_val() : 0.0));
            }
            if (lane == 0 && bad) atomicOr(p.flag, 1u);
        }
        if constexpr (TN == 2) {
            __syncthreads();   // everyone has read the partial tiles
            Wide* const sums = reinterpret_cast<Wide*>(smem);
            double* const norms = reinterpret_cast<double*>(sums + 2);
            if (wave == 1 && lane == 0) {
                sums[0] = s;
                sums[1] = c;
                norms[0] = F2;
                norms[1] = ratio;
            }
            __syncthreads();
            s += sums[0];
            c += sums[1];
            F2 += norms[0];
            ratio = __builtin_fmax(ratio, norms[1]);
        }
        if (tid == 0 && p.report)
            report_update(p.report, ratio, (double)s, (double)c, IS_INT ? 0.0 : p.tol_coeff * __builtin_sqrt(F2), __builtin_sqrt(F2), 0.0, (unsigned)tile_n);
    }
}

template <int DT, int TN, int MODE, bool BYTES, bool INJ>
__global__ __launch_bounds__(64 * SKINNY_WAVES) void gemm_skinny_kernel(const GemmArgs p) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    int tile_m, tile_n;
    tile_of_block((int)blockIdx.x, 1, (int)gridDim.x, tile_m, tile_n);   // (a run of columns per die: whole lines of C and A once)
    skinny_tile<DT, TN, MODE, BYTES, INJ>(p, tile_n, smem);
}

}  // namespace abft
