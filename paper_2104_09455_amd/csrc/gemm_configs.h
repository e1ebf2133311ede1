// Tile configurations shared by the host-side dispatcher and the kernel instantiations.
#pragma once
#include "gemm_kernel.h"
#include "gemm_rows.h"

namespace abft {

// Index into the configuration table.
//  F* run the direct-to-LDS kernel (16-byte aligned operands and leading dimensions, K a multiple of 128 bytes):
//    F256W  256 x 256, wavefronts 2 x 4 of 128 x  64 (two per SIMD), 2 LDS stages   compute-bound products;
//                                                                    16x16x32 MFMA shapes (the others 32x32x16): no
//                                                                    wavefront-level scheme runs on it
//    F256N  256 x 128, wavefronts 4 x 2 of  64 x  64, 3 stages, 16x16x32 shapes       about one tile per compute unit,
//                                                                    unprotected / global
//    F256S  256 x  64, wavefronts 8 x 1 of  32 x  64, 3 stages, 16x16x32 shapes       outputs of at most 64 columns
//                                                                    (many rows), unprotected / global
//    F128   128 x 128, wavefronts 2 x 2 of  64 x  64, 2 stages       mid-size, unprotected / global
//    F128E  128 x 128, wavefronts 4 x 2 of  32 x  64 (two per SIMD), 3 stages, 16x16x32 shapes
//                                                                    at most one such tile per compute unit: the second
//                                                                    wavefront per SIMD and the third stage stand in for
//                                                                    the second workgroup that would hide the latencies;
//                                                                    unprotected / global
//    F128T  128 x 128, wavefronts 4 x 1 of  32 x 128, 2 stages       thread-level (wide tiles: two checksum
//                                                                    MFMAs per four), narrow outputs, K of one k tile
//    F64T    64 x 128, wavefronts 2 x 1 of  32 x 128, 3 stages       between the streaming tiles and F128
//  S* run the streaming kernel (same alignment, K any multiple of 16 bytes; four wavefronts split the k tiles of one
//  register tile between them, each with its own LDS stages, no barrier in the k loop):
//    S32     32 x  32, 4 stages per wavefront                         a few tiles only: latency-bound layers
//    S32W    32 x  32, eight wavefronts with 2 stages each             the same with long k loops
//    S64     32 x  64, 3 stages per wavefront
//    S128    64 x  64, 2 stages per wavefront                         up to about one tile per compute unit
//  R64 runs the row-streaming kernel (same alignment as F*; 16-bit types, unprotected or wavefront-level):
//    R64     32 x  64 per wavefront, weights resident in LDS         very many rows, 64 columns or a single k tile
//                                                                    (convolutions whose input rows fit beside them: the strip kernel)
//  G* run the generic kernel (any alignment, layout, K):
//    G128 128 x 128, G64 64 x 64 (32x32 MFMA shapes), G16 16 x 64 (16x16 shapes; M <= 16)
//    G64K 64 x 64 with four groups of four wavefronts sharing the k tiles: at most about one tile per compute unit
enum CfgId { CFG_F256W = 0, CFG_F128, CFG_F128T, CFG_F64T, CFG_S32, CFG_S64, CFG_S128, CFG_G128, CFG_G64, CFG_G16, CFG_F256N, CFG_F256S, CFG_F128E, CFG_G64K, CFG_R64, CFG_S32W, CFG_COUNT };

inline const char* cfg_name(int id) {
    static const char* const names[CFG_COUNT] = {"F256W", "F128", "F128T", "F64T", "S32", "S64", "S128", "G128", "G64", "G16",
                                                 "F256N", "F256S", "F128E", "G64K", "R64", "S32W"};
    return id >= 0 && id < CFG_COUNT ? names[id] : nullptr;
}

template <int DT, int ID>
struct CfgOf;
//                                             MI TM TN WM WN BKB
template <int DT> struct CfgOf<DT, CFG_F128>  { typedef Cfg<DT, 32, 2, 2, 2, 2, 128, true> type; static constexpr int NSTAGE = 2; static constexpr int KWAYS = 1; };
template <int DT> struct CfgOf<DT, CFG_F128T> { typedef Cfg<DT, 32, 1, 4, 4, 1, 128, true> type; static constexpr int NSTAGE = 2; static constexpr int KWAYS = 1; };
template <int DT> struct CfgOf<DT, CFG_F64T>  { typedef Cfg<DT, 32, 1, 4, 2, 1, 128, true> type; static constexpr int NSTAGE = 3; static constexpr int KWAYS = 1; };
template <int DT> struct CfgOf<DT, CFG_F256W> { typedef Cfg<DT, 16, 8, 4, 2, 4, 128, true> type; static constexpr int NSTAGE = 2; static constexpr int KWAYS = 1; };
template <int DT> struct CfgOf<DT, CFG_F256N> { typedef Cfg<DT, 16, 4, 4, 4, 2, 128, true> type; static constexpr int NSTAGE = 3; static constexpr int KWAYS = 1; };
template <int DT> struct CfgOf<DT, CFG_F256S> { typedef Cfg<DT, 16, 2, 4, 8, 1, 128, true> type; static constexpr int NSTAGE = 3; static constexpr int KWAYS = 1; };
template <int DT> struct CfgOf<DT, CFG_F128E> { typedef Cfg<DT, 16, 2, 4, 4, 2, 128, true> type; static constexpr int NSTAGE = 3; static constexpr int KWAYS = 1; };
template <int DT> struct CfgOf<DT, CFG_S32>   { typedef Cfg<DT, 32, 1, 1, 1, 1, 128> type; static constexpr int NSTAGE = 4; static constexpr int KWAYS = 4; };
template <int DT> struct CfgOf<DT, CFG_S32W>  { typedef Cfg<DT, 32, 1, 1, 1, 1, 128> type; static constexpr int NSTAGE = 2; static constexpr int KWAYS = 8; };
template <int DT> struct CfgOf<DT, CFG_S64>   { typedef Cfg<DT, 32, 1, 2, 1, 1, 128> type; static constexpr int NSTAGE = 3; static constexpr int KWAYS = 4; };
template <int DT> struct CfgOf<DT, CFG_S128>  { typedef Cfg<DT, 32, 2, 2, 1, 1, 128> type; static constexpr int NSTAGE = 2; static constexpr int KWAYS = 4; };
template <int DT> struct CfgOf<DT, CFG_R64>   { typedef Cfg<DT, 32, 1, 2, 1, 1, 128, true> type; static constexpr int NSTAGE = 2; static constexpr int KWAYS = 1; };
template <int DT> struct CfgOf<DT, CFG_G128>  { typedef Cfg<DT, 32, 2, 2, 2, 2, 128> type; static constexpr int NSTAGE = 0; static constexpr int KWAYS = 1; };
template <int DT> struct CfgOf<DT, CFG_G64>   { typedef Cfg<DT, 32, 1, 1, 2, 2, 128> type; static constexpr int NSTAGE = 0; static constexpr int KWAYS = 1; };
template <int DT> struct CfgOf<DT, CFG_G64K>  { typedef Cfg<DT, 32, 1, 1, 2, 2, 128> type; static constexpr int NSTAGE = 0; static constexpr int KWAYS = 4; };
template <int DT> struct CfgOf<DT, CFG_G16>   { typedef Cfg<DT, 16, 1, 1, 1, 4, 256> type; static constexpr int NSTAGE = 0; static constexpr int KWAYS = 1; };

constexpr bool cfg_is_rows(int id) { return id == CFG_R64; }
constexpr bool cfg_is_stream(int id) { return id == CFG_S32 || id == CFG_S32W || id == CFG_S64 || id == CFG_S128; }
constexpr bool cfg_is_generic(int id) { return id == CFG_G128 || id == CFG_G64 || id == CFG_G64K || id == CFG_G16; }

// threads: of one WAVES_M x WAVES_N grid of wavefronts (a launch has kways times as many);
// kway_bytes: bytes of k that one wavefront takes in turn when kways wavefronts share a tile
struct CfgInfo {
    int bm, bn, bk_bytes, wm, wn, threads, lds_bytes, fast, kways, kway_bytes, mi;
};

template <int ID>
constexpr CfgInfo cfg_info() {
    typedef typename CfgOf<DT_F16, ID>::type C;  // identical for every dtype (rows / columns / k bytes)
    constexpr int ns = CfgOf<DT_F16, ID>::NSTAGE;
    constexpr int kw = CfgOf<DT_F16, ID>::KWAYS;
    constexpr int lds = cfg_is_stream(ID) ? kw * ns * ((C::BM + C::BN) * 128 + 768)
                                          : (ns ? ns * ((C::BM + C::BN) * 128 + 1024) + 512 : kw * C::LDS_BYTES);
    return CfgInfo{C::BM, C::BN, C::BKB, C::WM, C::WN, C::THREADS, lds, ns ? 1 : 0, kw, kw > 1 ? C::BKB : 32, C::MI};
}

inline CfgInfo cfg_info_host(int id) {
    switch (id) {
        case CFG_F128: return cfg_info<CFG_F128>();
        case CFG_F128T: return cfg_info<CFG_F128T>();
        case CFG_F64T: return cfg_info<CFG_F64T>();
        case CFG_F256W: return cfg_info<CFG_F256W>();
        case CFG_F256N: return cfg_info<CFG_F256N>();
        case CFG_F256S: return cfg_info<CFG_F256S>();
        case CFG_F128E: return cfg_info<CFG_F128E>();
        case CFG_S32: return cfg_info<CFG_S32>();
        case CFG_S32W: return cfg_info<CFG_S32W>();
        case CFG_S64: return cfg_info<CFG_S64>();
        case CFG_S128: return cfg_info<CFG_S128>();
        case CFG_R64: return cfg_info<CFG_R64>();
        case CFG_G128: return cfg_info<CFG_G128>();
        case CFG_G64: return cfg_info<CFG_G64>();
        case CFG_G64K: return cfg_info<CFG_G64K>();
        default: return cfg_info<CFG_G16>();
    }
}

// the strip kernel (16-bit types; gemm_strip_<dtype>.hip)
hipError_t launch_strip_f16(int mode, bool inject, const GemmArgs& args, hipStream_t stream);
hipError_t launch_strip_bf16(int mode, bool inject, const GemmArgs& args, hipStream_t stream);
inline hipError_t launch_strip_i8(int, bool, const GemmArgs&, hipStream_t) { return hipErrorInvalidValue; }  // (never picked)
// Its two forms (see gemm_strip.h): wavefronts (three, resp. two, per SIMD), strips held at a time, and the bytes of one strip
// (3 resp. 10 chunks of the next one per thread)
enum { STRIP_RUNS = 0, STRIP_TAPS = 1 };
constexpr int strip_waves(int form) { return form == STRIP_RUNS ? 12 : 8; }
constexpr int strip_buffers(int form) { return form == STRIP_RUNS ? 2 : 1; }
constexpr int strip_max_bytes(int form) { return (form == STRIP_RUNS ? 3 : 10) * 64 * strip_waves(form) * 16; }
constexpr int STRIP_ROWS_MAX = 128;
// what it keeps in LDS: the weights, the strips, where each chunk of k starts
constexpr int strip_lds_bytes(int form, int nkt, int rows, int pitch) {
    return nkt * 64 * 128 + strip_buffers(form) * rows * pitch + nkt * 32;
}

// implemented once per dtype and family of configurations in gemm_<family>_<dtype>.hip
#define ABFT_DECLARE_LAUNCHES(dt)                                                                                  \
    hipError_t launch_fast_##dt(int cfg, int mode, bool inject, const GemmArgs& args, hipStream_t stream);    \
    hipError_t launch_stream_##dt(int cfg, int mode, bool inject, const GemmArgs& args, hipStream_t stream);  \
    hipError_t launch_generic_##dt(int cfg, int mode, bool inject, const GemmArgs& args, hipStream_t stream); \
    inline hipError_t launch_gemm_##dt(int cfg, int mode, bool inject, const GemmArgs& args, hipStream_t stream) { \
        if (args.strip_pitch) return launch_strip_##dt(mode, inject, args, stream);                           \
        if (cfg_is_stream(cfg)) return launch_stream_##dt(cfg, mode, inject, args, stream);                   \
        if (cfg_is_generic(cfg)) return launch_generic_##dt(cfg, mode, inject, args, stream);                 \
        return launch_fast_##dt(cfg, mode, inject, args, stream);                                             \
    }
ABFT_DECLARE_LAUNCHES(f16)
ABFT_DECLARE_LAUNCHES(bf16)
ABFT_DECLARE_LAUNCHES(i8)
#undef ABFT_DECLARE_LAUNCHES

}  // namespace abft
