// Dispatch of a mixed-launch tile to the template instantiation of its shape,
// per family; shared by the family kernels (mixed_fft.hip, mixed_scan.hip,
// mixed_tri.hip) and the class kernels (mixed_class.hip).
#pragma once

#include <type_traits>

#include "fft_device.h"
#include "mixed.h"
#include "scan_device.h"
#include "tridiag_wave_device.h"

namespace ppx {

// f(std::integral_constant<int, shape>{}) for a runtime shape in [LO, HI), by
// halving: a tile reaches its instantiation in log2(HI - LO) branches.  (A
// chain of one comparison per shape, each jumping over the body it guards,
// walks through up to 90 places of a kernel of several hundred KiB, most of
// them instruction-cache misses, before a tile's first load.)
template <int LO, int HI, typename F>
__device__ __forceinline__ void mix_dispatch(int shape, const F &f) {
    if constexpr (HI - LO == 1) {
        f(std::integral_constant<int, LO>{});
    } else {
        constexpr int MID = LO + (HI - LO) / 2;
        if (shape < MID) mix_dispatch<LO, MID>(shape, f);
        else mix_dispatch<MID, HI>(shape, f);
    }
}

// Whether shape (LOG2N, P, SPLIT) belongs to family FAM.
template <int FAM>
constexpr bool mix_fft_member(int log2n, int P, bool) {
    if (log2n < 4 || log2n > kFftLog2NMax || (1 << log2n) < P) return false;
    const int T = (1 << log2n) / P;
    if (FAM == kFamFft256) return T <= 256;
    return P == (FAM == kFamFft1024P8 ? 8 : 16) && T > 256 && T <= 1024;
}

template <int FAM>
__device__ __forceinline__ void mix_fft_dispatch(const MixJob &j, long long first, int count,
                                                 const float2 *__restrict__ tw, void *lds, int tx, int nt) {
    mix_dispatch<0, kMixFftShapes>(j.shape, [&](auto id) {
        constexpr int ID = decltype(id)::value;
        constexpr int LOG2N = ID / 6;
        constexpr int P = 4 << ((ID / 2) % 3);
        constexpr bool SPLIT = (ID & 1) != 0;
        if constexpr (mix_fft_member<FAM>(LOG2N, P, SPLIT)) {
            static_assert(mix_fft_shape(LOG2N, P, SPLIT) == ID, "shape code");
            fft_group_ct<P, P, SPLIT, LOG2N>(static_cast<const float2 *>(j.p[0]), static_cast<float2 *>(j.out), tw,
                                             first, count, (j.flags & 1) ? -1.0f : 1.0f, lds, tx, nt);
        }
    });
}

template <typename Wt>
__device__ __forceinline__ void mix_scan_dispatch(const MixJob &j, long long first, int count, Wt *wave_tot, int tx) {
    mix_dispatch<0, kMixScanShapes>(j.shape, [&](auto id) {
        constexpr int ID = decltype(id)::value;
        constexpr int DT = ID / 10;
        constexpr int LP = (ID / 2) % 5 + 1;
        constexpr int P = 1 << LP;
        constexpr int ALGO = (ID & 1) ? PPX_SCAN_LF : PPX_SCAN_KS;
        using T = typename std::conditional<DT == PPX_I32, int, typename std::conditional<DT == PPX_F32, float, double>::type>::type;
        if constexpr (DT != PPX_F64 || P <= kScanF64MaxElems) {
            static_assert(mix_scan_shape(DT, LP, ALGO == PPX_SCAN_LF) == ID, "shape code");
            const T *in = static_cast<const T *>(j.p[0]);
            T *out = static_cast<T *>(j.out);
            T *wt = reinterpret_cast<T *>(wave_tot);
            if (j.flags & 1) scan_block<T, P, ALGO, true>(in, out, j.log2n, first, count, wt, tx);
            else scan_block<T, P, ALGO, false>(in, out, j.log2n, first, count, wt, tx);
        }
    });
}

template <int FAM>
using TriwType = typename std::conditional<FAM == kFamTriW32 || FAM == kFamTriW32H, float, double>::type;
// Whether the family FAM holds the in-wave shape (ALGO, P).
template <int FAM>
constexpr bool triw_member(int algo, int P) {
    return mix_triw_family(FAM == kFamTriW64 || FAM == kFamTriW64H, algo, P) == FAM;
}

template <int FAM>
__device__ __forceinline__ void mix_triw_dispatch(const MixJob &j, long long first, int count, void *smem, int tx) {
    mix_dispatch<0, kMixTriwShapes>(j.shape, [&](auto id) {
        constexpr int ID = decltype(id)::value;
        using T = TriwType<FAM>;
        constexpr int ALGO = PPX_TRI_CR_PCR + ID / 4;
        constexpr int LP = ID % 4 + 1;
        constexpr int P = 1 << LP;
        if constexpr (triw_member<FAM>(ALGO, P)) {
            static_assert(mix_triw_shape(ALGO, LP) == ID, "shape code");
            tridiag_wave_block<T, ALGO, P>(static_cast<const T *>(j.p[0]), static_cast<const T *>(j.p[1]),
                                           static_cast<const T *>(j.p[2]), static_cast<const T *>(j.p[3]),
                                           static_cast<T *>(j.out), j.log2n, first, count, static_cast<T *>(smem), tx);
        }
    });
}

// The hybrid across waves: a tile is nt / (n / P) systems (nt the workgroup
// size), the lanes exchanging through LDS slots, which also stage the solution
// where a lane holds 64 bytes or more of it (tri_blk_lds_vals).
template <int FAM, int LP>
__device__ __forceinline__ void mix_trib_dispatch(const MixJob &j, long long first, int count, void *smem, int tx,
                                                  int nt) {
    if constexpr (LP <= 4) {
        using T = typename std::conditional<FAM == kFamTriBlk32 || FAM == kFamTriBlk32H, float, double>::type;
        constexpr int P = 1 << LP;
        if constexpr ((FAM == kFamTriBlk32H || FAM == kFamTriBlk64H) == (P == 16)) {
            if (j.shape == LP - 1) {
                tridiag_blk_block<T, P>(static_cast<const T *>(j.p[0]), static_cast<const T *>(j.p[1]),
                                        static_cast<const T *>(j.p[2]), static_cast<const T *>(j.p[3]),
                                        static_cast<T *>(j.out), j.log2n, first, count, static_cast<T *>(smem), tx,
                                        nt);
                return;
            }
        }
        mix_trib_dispatch<FAM, LP + 1>(j, first, count, smem, tx, nt);
    }
}

}  // namespace ppx
