// FFT families of the mixed launch: kernels whose tiles run the
// log2 n-specialised stage sequence of the job's tuned (radix = P) shape,
// with its exchange (complex values, or real and imaginary parts in turn).
// 256-thread workgroups take the shapes with at most 256 threads per problem
// (P in {4, 8, 16}); 1024-thread workgroups the larger ones (n >= 4096), one
// family for P = 8 and one for P = 16 (P = 8 needs half the LDS and fewer
// registers, so two of its workgroups fit a CU).  Each tile runs the same function as the single-call kernel
// of its shape (fft_group_ct), and the two give the same bits; the exchange
// is part of the shape because it changes how the compiler contracts the
// butterflies' products and sums into fused multiply-adds (a tile with the
// split exchange differs in the last bits from the single call with the
// complex one).
#include "mixed_dispatch.h"

namespace ppx {

template <int FAM, bool ARGS>
__global__ __launch_bounds__(mix_block(FAM)) void k_mix_fft(MixArgs a, const float2 *tw) {
    extern __shared__ float4 lds[];
    mix_tile_loop<FAM, ARGS>(a, [&](const MixJob &j, long long first, int count, int tx, int nt) {
        mix_fft_dispatch<FAM>(j, first, count, tw, lds, tx, nt);
    });
}

template <bool ARGS>
static const void *fft_kernel(int fam) {
    if (fam == kFamFft256) return reinterpret_cast<const void *>(&k_mix_fft<kFamFft256, ARGS>);
    if (fam == kFamFft1024) return reinterpret_cast<const void *>(&k_mix_fft<kFamFft1024, ARGS>);
    if (fam == kFamFft1024P8) return reinterpret_cast<const void *>(&k_mix_fft<kFamFft1024P8, ARGS>);
    return nullptr;
}

const void *mix_fft_kernel(int fam, bool args) {
    return args ? fft_kernel<true>(fam) : fft_kernel<false>(fam);
}

}  // namespace ppx
