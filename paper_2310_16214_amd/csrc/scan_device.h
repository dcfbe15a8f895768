// Batched inclusive and exclusive sum scans (Sec. III "Scan Operator" of
// arXiv:2310.16214), int32 (modulo 2^32), float32 and float64, for gfx950.
//
// A workgroup of L threads (whole waves: launch_scan sees to it) scans G_b
// problems of size n, i.e. G_b*n contiguous elements, P per thread: each wave
// takes 64*P consecutive elements, as R =
// P / V rows of 64 vectors (V elements, 16 bytes; fewer where P is), and lane
// l holds vector l of each row.  So every load and store instruction moves
// 1 KiB of consecutive bytes.  (With a thread's P elements consecutive
// instead, a lane's 16-byte words lie P * sizeof(T) bytes apart and each
// store covers a quarter or less of every line it touches: 64 MiB of float32
// at n = 16384, P = 16, took 36.0 us that way and takes 27.6 in rows (P = 32,
// persistent: 25.4); 128 MiB of float64 at n = 8192, P = 8, took 60.4 us and
// takes 51.1.  A copy of these sizes takes 23.3 and 44.2 us: HBM bounds the
// scan.)  Steps:
//   1. thread-serial scan of each row's V values (registers);
//   2. per row, inclusive scan of the vectors' totals across the lanes of
//      each problem segment (min(n / V, 64) lanes) with a wave64 lane network:
//      Kogge-Stone (DPP row shifts + row broadcasts) or Ladner-Fischer
//      (swizzle broadcasts) -- the two prefix circuits the paper tunes; where
//      a problem spans several rows of a wave, the sum of its earlier rows'
//      totals (wave-uniform) is carried along;
//   3. when a problem spans several waves, each wave's total goes to one LDS
//      slot and every wave adds the totals of the earlier waves of its problem
//      (the paper's per-problem shared-memory slots, one per wave): the
//      lanes of a 16-lane row read one slot each and sum them by rotations,
//      four steps instead of up to 15 dependent reads.  (Vectors of 8 bytes
//      have them read in turn: with rotations their persistent kernels were up
//      to 23% slower, 2^24 float32 of n = 256 in 1024 threads 30.5 us against
//      24.9, and none of their shapes is the fastest of its size.)
//   4. add the exclusive prefix to the values and store; a vector's prefix is
//      the inclusive lane result of the lane before it plus the sums of
//      earlier rows and waves, so every term of an output is a sum of
//      elements at or before that output.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "device.h"
#include "ppx_internal.h"

namespace ppx {

// Elements of a lane's vector (16 bytes, or all P elements where they are
// fewer), rows per thread, and elements per row of a wave.
template <typename T, int P>
constexpr int scan_vec() { return P * (int)sizeof(T) < 16 ? P : 16 / (int)sizeof(T); }
template <typename T, int P>
constexpr int scan_rows() { return P / scan_vec<T, P>(); }
template <typename T, int P>
constexpr int scan_row_elems() { return kWave * scan_vec<T, P>(); }

// Index within the workgroup's elements of the thread's first vector (row 0);
// row j's lies j * scan_row_elems further.
template <typename T, int P>
__device__ __forceinline__ int scan_first(int tx) {
    return (tx & ~(kWave - 1)) * P + (tx & (kWave - 1)) * scan_vec<T, P>();
}

// Sum over the 16 lanes of a row, in every lane (DPP row rotations).
constexpr int kDppRowRor = 0x120;  // + rotation (1..15), within 16-lane rows
template <int D, typename T>
__device__ __forceinline__ T dpp_row_ror(T v) {
    return per_word(v, [](int x) { return __builtin_amdgcn_update_dpp(0, x, kDppRowRor + D, 0xf, 0xf, false); });
}
template <typename T>
__device__ __forceinline__ T row16_sum(T x) {
    x += dpp_row_ror<8>(x);
    x += dpp_row_ror<4>(x);
    x += dpp_row_ror<2>(x);
    x += dpp_row_ror<1>(x);
    return x;
}

// Steps 1-4 on the P values a thread holds (row j's vector in v[j V ...
// j V + V - 1]).  `wave_tot` holds one value per wave; with more
// than 64 P elements per problem there is one barrier, which every thread of
// the workgroup must reach.
// EXCL: the exclusive scan (each output the sum of the inputs before it):
// step 1 is then the thread-serial exclusive scan, the rest is unchanged.
// tx: the thread's index in the workgroup.
template <typename T, int P, int ALGO, bool EXCL = false, typename U>
__device__ __forceinline__ void scan_values(U (&v)[P], int log2n, T *wave_tot, int tx) {
    constexpr int V = scan_vec<T, P>(), R = scan_rows<T, P>();
    constexpr int LV = V == 2 ? 1 : 2, LR = R == 1 ? 0 : R == 2 ? 1 : R == 4 ? 2 : 3;
    static_assert((1 << LV) == V && (1 << LR) == R, "2 or 4 values per vector, 1 to 8 rows");
    const int lane = tx & (kWave - 1);
    const int seg = log2n >= LV + 6 ? kWave : (1 << (log2n - LV));  // lanes of a problem within a row
    // 1. serial scan within each vector
    U incl[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
        if constexpr (EXCL) {
            U run = U(0);
#pragma unroll
            for (int e = j * V; e < j * V + V; ++e) {
                const U x = v[e];
                v[e] = run;
                run = run + x;
            }
            incl[j] = run;
        } else {
#pragma unroll
            for (int e = j * V + 1; e < j * V + V; ++e) v[e] = v[e] + v[e - 1];
            incl[j] = v[j * V + V - 1];
        }
    }
    // 2. lane network over the vectors' totals, per row
    if constexpr (ALGO == PPX_SCAN_LF) lanes_scan_lf<U, R>(incl, seg, lane);
    else lanes_scan_ks<U, R>(incl, seg, lane);
    // Exclusive prefix of a vector within the segment: the previous lane's
    // inclusive value (0 at the segment's first lane), moved by a one-lane
    // shift.  Forming it as inclusive value minus own total instead would
    // cancel: every output would then carry rounding on the scale of the
    // vector and of the elements after it, not of the sum the output is
    // defined by.
    U prefix[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const U prev = dpp_wave_shr1(incl[j]);
        prefix[j] = (lane & (seg - 1)) == 0 ? U(0) : prev;
    }
    // earlier rows of the same problem (a problem of `rows` rows starts at a
    // multiple of that many)
    U carry = incl[0];  // R = 1: the wave's total, in its last lane
    if constexpr (R > 1) {
        if (log2n > LV + 6) {
            const int rows = log2n >= LV + 6 + LR ? R : 1 << (log2n - LV - 6);
#pragma unroll
            for (int j = 0; j < R; ++j) {
                if ((j & (rows - 1)) == 0) carry = U(0);
                prefix[j] = prefix[j] + carry;
                carry = carry + per_word(incl[j], [](int w) { return __builtin_amdgcn_readlane(w, kWave - 1); });
            }
        }
    }

    // 3. earlier waves of the same problem
    U before = U(0);
    constexpr int LW = LV + LR + 6;  // log2 of a wave's elements
    if (log2n > LW) {
        const int w = tx >> 6;
        if (lane == kWave - 1) wave_tot[w] = __builtin_bit_cast(T, carry);
        __syncthreads();
        const int w0 = w & ~((1 << (log2n - LW)) - 1);
        if constexpr (V * sizeof(T) == 8) {
            for (int u = w0; u < w; ++u) prefix[0] = prefix[0] + __builtin_bit_cast(U, wave_tot[u]);
        } else {
            const int u = lane & 15;  // at most 16 waves per workgroup
            const bool earlier = u >= w0 && u < w;
            const U slot = __builtin_bit_cast(U, wave_tot[earlier ? u : w]);
            before = row16_sum(earlier ? slot : U(0));
        }
    }

    // 4. add the prefix
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const U p = prefix[j] + before;
#pragma unroll
        for (int e = j * V; e < j * V + V; ++e) v[e] = v[e] + p;
    }
}

// Integer adds wrap modulo 2^32: they are done on unsigned values.
template <typename T>
using ScanArith = typename std::conditional<std::is_same<T, int>::value, unsigned, T>::type;

// Store policy: a wave's store of 16-byte vectors covers whole lines, and goes
// out non-temporal: with float32, 2^24 elements, n = 256 takes 24.2 us against
// 25.2, n = 8192 (P = 8) 25.7 against 26.8; 2^25 elements 46.8 against 49.4;
// float64, n = 512, 44.6 against 46.5 (interleaved runs on rotating buffers).
// Eight-byte vectors (P = 2, 4-byte types) keep the default policy.
__device__ __forceinline__ void scan_store_word(u32x4 *p, u32x4 w) { store_nt(p, w); }
__device__ __forceinline__ void scan_store_word(u32x2 *p, u32x2 w) { *p = w; }

// One workgroup's share: problems [p0, p0 + nprob) (lanes of problems beyond
// nprob compute on zeros and store nothing).  `wave_tot` holds
// one value per wave; tx is the thread's index in the workgroup.
// Used by k_scan and by the mixed launch's tiles.
template <typename T, int P, int ALGO, bool EXCL = false>
__device__ __forceinline__ void scan_block(const T *in, T *out, int log2n, long long p0, int nprob,
                                           T *wave_tot, int tx) {
    using U = ScanArith<T>;
    constexpr int V = scan_vec<T, P>(), R = scan_rows<T, P>();
    const int first = scan_first<T, P>(tx);
    const int total = nprob << log2n;
    const U *src = reinterpret_cast<const U *>(in) + (p0 << log2n) + first;
    U *dst = reinterpret_cast<U *>(out) + (p0 << log2n) + first;
    using W = typename std::conditional<V * sizeof(T) == 16, u32x4, u32x2>::type;

    U v[P];
#pragma unroll
    for (int j = 0; j < R; ++j) {
        W w{};
        if (first + j * scan_row_elems<T, P>() < total)
            w = *reinterpret_cast<const W *>(src + j * scan_row_elems<T, P>());
        __builtin_memcpy(&v[j * V], &w, sizeof w);
    }
    scan_values<T, P, ALGO, EXCL>(v, log2n, wave_tot, tx);
#pragma unroll
    for (int j = 0; j < R; ++j) {
        W w;
        __builtin_memcpy(&w, &v[j * V], sizeof w);
        if (first + j * scan_row_elems<T, P>() < total)
            scan_store_word(reinterpret_cast<W *>(dst + j * scan_row_elems<T, P>()), w);
    }
}

template <typename T, int P, int ALGO, bool EXCL>
__global__ __launch_bounds__(1024) void k_scan(const T *in, T *out, int log2n, long long batch,
                                               int gb) {
    __shared__ T wave_tot[kMaxThreadsPerBlock / kWave];
    const long long p0 = (long long)blockIdx.x * gb;
    scan_block<T, P, ALGO, EXCL>(in, out, log2n, p0, (int)min((long long)gb, batch - p0), wave_tot, threadIdx.x);
}

// A thread's rows through a group's buffer descriptor (voff: the byte offset
// of its first vector).  The rows' offsets go in the vector offset (a 16-byte
// store must not take one from a scalar register, see buf_store).
template <typename T, int P, typename U>
__device__ __forceinline__ void scan_load_rows(U (&v)[P], __amdgpu_buffer_rsrc_t r, int voff) {
    constexpr int V = scan_vec<T, P>(), B = scan_row_elems<T, P>() * (int)sizeof(T);
#pragma unroll
    for (int j = 0; j < scan_rows<T, P>(); ++j) {
        if constexpr (V * sizeof(T) == 16) {
            const u32x4 w = __builtin_amdgcn_raw_buffer_load_b128(r, voff + j * B, 0, 0);
            __builtin_memcpy(&v[j * V], &w, sizeof w);
        } else {
            const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(r, voff + j * B, 0, 0);
            __builtin_memcpy(&v[j * V], &w, sizeof w);
        }
    }
}
template <typename T, int P, typename U>
__device__ __forceinline__ void scan_store_rows(const U (&v)[P], __amdgpu_buffer_rsrc_t r, int voff) {
    constexpr int V = scan_vec<T, P>(), B = scan_row_elems<T, P>() * (int)sizeof(T);
#pragma unroll
    for (int j = 0; j < scan_rows<T, P>(); ++j) {
        if constexpr (V * sizeof(T) == 16) {
            u32x4 w;
            __builtin_memcpy(&w, &v[j * V], sizeof w);
            __builtin_amdgcn_raw_buffer_store_b128(w, r, voff + j * B, 0, kStoreNT);
        } else {
            u32x2 w;
            __builtin_memcpy(&w, &v[j * V], sizeof w);
            __builtin_amdgcn_raw_buffer_store_b64(w, r, voff + j * B, 0, 0);
        }
    }
}

// Persistent variant: a grid of resident workgroups (at most one per group)
// walks the groups of gb problems (g, g + gridDim.x, ...) and loads the next
// group's values into a second register set while it scans the current one,
// so the loads overlap the barrier-bound steps of workgroups that span many
// waves.  Loads and stores go through per-group buffer descriptors (lanes
// past the batch read zeros and store nothing, without a branch); the first
// iteration is peeled and the loop unrolled twice with the two register sets
// swapping roles, so the wait for the prefetched group never also covers the
// stores issued after it.  The wave totals alternate between two buffers: a
// wave may start the next group before a slower one has read this group's
// totals, and the barrier of every group keeps the waves within one group of
// each other.
template <typename T, int P, int ALGO, bool EXCL>
__global__ __launch_bounds__(1024) void k_scan_pipe(const T *in, T *out, int log2n, long long batch,
                                                    int gb) {
    using U = ScanArith<T>;
    __shared__ T wave_tot[2][kMaxThreadsPerBlock / kWave];
    const long long n = 1LL << log2n;
    const int voff = scan_first<T, P>((int)threadIdx.x) * (int)sizeof(T);  // byte offset within a group
    const long long ngroups = (batch + gb - 1) / gb;
    const long long G = gridDim.x;
    U v0[P], v1[P];
    auto iteration = [&](long long grp, int parity, U (&cur)[P], U (&nxt)[P]) {
        scan_load_rows<T, P>(nxt, group_rsrc(in, grp + G, gb, n, sizeof(T), batch), voff);
        __builtin_amdgcn_sched_barrier(0);
        scan_values<T, P, ALGO, EXCL>(cur, log2n, wave_tot[parity], threadIdx.x);
        scan_store_rows<T, P>(cur, group_rsrc(out, grp, gb, n, sizeof(T), batch), voff);
    };
    long long g = blockIdx.x;  // < ngroups: the grid never exceeds the groups
    scan_load_rows<T, P>(v0, group_rsrc(in, g, gb, n, sizeof(T), batch), voff);
    iteration(g, 0, v0, v1);
    for (g += G; g < ngroups; g += 2 * G) {
        iteration(g, 1, v1, v0);
        if (g + G >= ngroups) break;
        iteration(g + G, 0, v0, v1);
    }
}

}  // namespace ppx
