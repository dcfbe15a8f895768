// Scan families of the mixed launch: kernels whose tiles run the
// job's tuned scan shape (values per thread, lane network, inclusive or
// exclusive) on whole problems of T = n/P threads: 256-thread workgroups for
// T <= 256, 1024-thread ones above.
#include "mixed_dispatch.h"

namespace ppx {

// Two workgroups of 1024 threads per CU, eight waves per SIMD: 64 registers.
// Left alone the compiler takes 70 for float64 with 16 values per thread and
// one workgroup fits (20 scans of 1024 and 2048 values, 61.0 us against 49.0);
// bounded, that shape alone keeps 13 registers in scratch memory.
template <int FAM, bool ARGS>
__global__ __launch_bounds__(mix_block(FAM), 8) void k_mix_scan(MixArgs a, const float2 *) {
    __shared__ double wave_tot[mix_block(FAM) / kWave];  // int and float totals use its start
    mix_tile_loop<FAM, ARGS>(a, [&](const MixJob &j, long long first, int count, int tx, int nt) {
        mix_scan_dispatch(j, first, count, wave_tot, tx);
    });
}

template <bool ARGS>
static const void *scan_kernel(int fam) {
    if (fam == kFamScan256) return reinterpret_cast<const void *>(&k_mix_scan<kFamScan256, ARGS>);
    if (fam == kFamScan1024) return reinterpret_cast<const void *>(&k_mix_scan<kFamScan1024, ARGS>);
    return nullptr;
}

const void *mix_scan_kernel(int fam, bool args) {
    return args ? scan_kernel<true>(fam) : scan_kernel<false>(fam);
}

}  // namespace ppx
