// Tridiagonal families of the mixed launch: kernels whose tiles
// run the job's tuned solver.  Systems that fit a wave (n / P <= 64) run the
// in-wave variants (the CR -> PCR hybrid, CR, PCR with shuffles or with the
// LDS exchange, Wang & Mou, Ladner-Fischer) in 256-thread workgroups, one
// kernel per dtype and per
// register tier: a kernel's VGPR count is the maximum over its shapes, and
// the P = 16 solvers (and in float32 also the PCR ones, 94-100 VGPRs against
// 56-62 for CR, WM and LF) would otherwise halve the others' occupancy.
// Larger systems run the LDS CR or PCR in 1024-thread workgroups with
// 128 KiB of LDS.
#include "mixed_dispatch.h"
#include "tridiag_device.h"

namespace ppx {

// float64 with 16 equations per lane: at least three waves per SIMD, as for
// the single-call kernels of those shapes (tri_wave_min_waves); the other
// families with PCR shapes: four (left alone they take 129 and 132 VGPRs,
// just over what four waves have).
template <int FAM>
constexpr int triw_min_waves() { return FAM == kFamTriW64H ? 3 : FAM == kFamTriW32 ? 1 : 4; }

template <int FAM, bool ARGS>
__global__ __launch_bounds__(256, triw_min_waves<FAM>()) void k_mix_triw(MixArgs a, const float2 *) {
    extern __shared__ float4 smem[];  // PPX_TRI_PCR_REG exchange buffers, one per wave
    mix_tile_loop<FAM, ARGS>(a, [&](const MixJob &j, long long first, int count, int tx, int nt) {
        mix_triw_dispatch<FAM>(j, first, count, smem, tx);
    });
}

template <bool ARGS>
__global__ __launch_bounds__(1024) void k_mix_tril(MixArgs a, const float2 *) {
    extern __shared__ float4 smem[];
    mix_tile_loop<kFamTriLds, ARGS>(a, [&](const MixJob &j, long long first, int count, int tx, int nt) {
        switch (j.shape) {
            case mix_tril_shape(false, false):
                tridiag_block<float, PPX_TRI_CR>(static_cast<const float *>(j.p[0]), static_cast<const float *>(j.p[1]),
                                                 static_cast<const float *>(j.p[2]), static_cast<const float *>(j.p[3]),
                                                 static_cast<float *>(j.out), j.log2n, first, count,
                                                 reinterpret_cast<float *>(smem));
                break;
            case mix_tril_shape(false, true):
                tridiag_block<float, PPX_TRI_PCR>(static_cast<const float *>(j.p[0]), static_cast<const float *>(j.p[1]),
                                                  static_cast<const float *>(j.p[2]), static_cast<const float *>(j.p[3]),
                                                  static_cast<float *>(j.out), j.log2n, first, count,
                                                  reinterpret_cast<float *>(smem));
                break;
            case mix_tril_shape(true, false):
                tridiag_block<double, PPX_TRI_CR>(static_cast<const double *>(j.p[0]), static_cast<const double *>(j.p[1]),
                                                  static_cast<const double *>(j.p[2]), static_cast<const double *>(j.p[3]),
                                                  static_cast<double *>(j.out), j.log2n, first, count,
                                                  reinterpret_cast<double *>(smem));
                break;
            default:
                tridiag_block<double, PPX_TRI_PCR>(static_cast<const double *>(j.p[0]), static_cast<const double *>(j.p[1]),
                                                   static_cast<const double *>(j.p[2]), static_cast<const double *>(j.p[3]),
                                                   static_cast<double *>(j.out), j.log2n, first, count,
                                                   reinterpret_cast<double *>(smem));
                break;
        }
    });
}

template <int FAM, bool ARGS>
__global__ __launch_bounds__(mix_block(FAM)) void k_mix_trib(MixArgs a, const float2 *) {
    extern __shared__ float4 smem[];
    mix_tile_loop<FAM, ARGS>(a, [&](const MixJob &j, long long first, int count, int tx, int nt) {
        mix_trib_dispatch<FAM, 1>(j, first, count, smem, tx, nt);
    });
}

template <bool ARGS>
static const void *tri_kernel(int fam) {
    switch (fam) {
        case kFamTriW32: return reinterpret_cast<const void *>(&k_mix_triw<kFamTriW32, ARGS>);
        case kFamTriW32H: return reinterpret_cast<const void *>(&k_mix_triw<kFamTriW32H, ARGS>);
        case kFamTriW64: return reinterpret_cast<const void *>(&k_mix_triw<kFamTriW64, ARGS>);
        case kFamTriW64H: return reinterpret_cast<const void *>(&k_mix_triw<kFamTriW64H, ARGS>);
        case kFamTriLds: return reinterpret_cast<const void *>(&k_mix_tril<ARGS>);
        case kFamTriBlk32: return reinterpret_cast<const void *>(&k_mix_trib<kFamTriBlk32, ARGS>);
        case kFamTriBlk32H: return reinterpret_cast<const void *>(&k_mix_trib<kFamTriBlk32H, ARGS>);
        case kFamTriBlk64: return reinterpret_cast<const void *>(&k_mix_trib<kFamTriBlk64, ARGS>);
        case kFamTriBlk64H: return reinterpret_cast<const void *>(&k_mix_trib<kFamTriBlk64H, ARGS>);
        default: return nullptr;
    }
}

const void *mix_tri_kernel(int fam, bool args) { return args ? tri_kernel<true>(fam) : tri_kernel<false>(fam); }

}  // namespace ppx
