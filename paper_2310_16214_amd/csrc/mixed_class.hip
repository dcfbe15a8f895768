// Class kernels of the mixed launch: the tiles of several families in one
// kernel.  A launch of uneven jobs cut into one kernel per family runs them
// one after another, each with its own ramp and tail and many with fewer
// workgroups than CUs (64 FFTs of n = 16384 are 64 workgroups).  A class
// holds the float32 families of one workgroup size (or of both), so that
// their tiles fill the GPU together:
//   small: T <= 256 threads per problem -- FFT, scan and in-wave tridiagonal
//          tiles in workgroups of up to 256 threads;
//   large: T up to 1024 -- FFT (P = 8 and 16), scan and the hybrid across
//          waves in workgroups of up to 1024 threads.
//   all:   both, in workgroups of up to 1024 threads (a small family's tile
//          holds four times the problems) -- for launches small enough that a
//          second kernel costs more than the smaller workgroups save.
// A class kernel runs at its most demanding member's registers (94: five
// waves per SIMD) and at the LDS of the families present, which is why a
// family alone, or one whose tiles fill the GPU for long by themselves, keeps
// its own kernel (mix_class_families in fused.hip).  The tile body is inlined
// by attribute: the small class's is past the compiler's limit, and as a
// function it got the record through scratch memory (a launch of six small
// scans and one tridiagonal job 8.2 us instead of 4.8).  The float64 tridiagonal
// families and the LDS solvers need more registers or other LDS and stay
// apart.  The records come in the kernel arguments, tile b runs in workgroup
// b, by the same functions as in the family kernels.
#include "mixed_dispatch.h"

namespace ppx {

template <int CLS>
__global__ __launch_bounds__(mix_class_block(CLS), CLS == kClassLarge ? 4 : 5) void k_mix_class(MixClassArgs a) {
    extern __shared__ float4 lds[];
    __shared__ double wave_tot[mix_class_block(CLS) / kWave];
    typedef const __attribute__((address_space(4))) MixJob *job_ptr;
    const job_ptr recs = reinterpret_cast<job_ptr>(
        (const __attribute__((address_space(4))) char *)__builtin_amdgcn_kernarg_segment_ptr() +
        offsetof(MixClassArgs, jobs));
    const unsigned t = blockIdx.x;
    unsigned k = 0;
    while (k + 1 < a.njobs && recs[k + 1].first_tile <= t) ++k;
    const float2 *tw = a.tw;
    auto body = [&](const MixJob &j, long long first, int count, int tx, int nt) __attribute__((always_inline)) {
        constexpr bool small = CLS != kClassLarge, large = CLS != kClassSmall;
        if (large && j.family == kFamFft1024) mix_fft_dispatch<kFamFft1024>(j, first, count, tw, lds, tx, nt);
        else if (large && j.family == kFamFft1024P8) mix_fft_dispatch<kFamFft1024P8>(j, first, count, tw, lds, tx, nt);
        else if (large && j.family == kFamTriBlk32) mix_trib_dispatch<kFamTriBlk32, 1>(j, first, count, lds, tx, nt);
        else if (large && j.family == kFamTriBlk32H) mix_trib_dispatch<kFamTriBlk32H, 1>(j, first, count, lds, tx, nt);
        else if (small && j.family == kFamFft256) mix_fft_dispatch<kFamFft256>(j, first, count, tw, lds, tx, nt);
        else if (small && j.family == kFamTriW32) mix_triw_dispatch<kFamTriW32>(j, first, count, lds, tx);
        else if (small && j.family == kFamTriW32H) mix_triw_dispatch<kFamTriW32H>(j, first, count, lds, tx);
        else mix_scan_dispatch(j, first, count, wave_tot, tx);
    };
    mix_run_tile(mix_load_job(recs + k), t, (int)blockDim.x, body);
}

const void *mix_class_kernel(int cls) {
    return cls == kClassSmall   ? reinterpret_cast<const void *>(&k_mix_class<kClassSmall>)
           : cls == kClassLarge ? reinterpret_cast<const void *>(&k_mix_class<kClassLarge>)
                                : reinterpret_cast<const void *>(&k_mix_class<kClassAll>);
}

}  // namespace ppx
