// Device code shared by the one-launch tail V-cycles (gfx950, wave64): a
// workgroup per system with the vectors of all covered levels in LDS.
#pragma once

#include "cs_internal.h"

namespace cs {
namespace {

constexpr int TAIL_WG = 1024;

// The level table's pointers are generic to the compiler, which would load through
// them with flat instructions: those count as LDS operations too, so that every
// wait for LDS would wait for them (a step of 216 rows of 8x8 blocks took 4 us).
template <typename T>
using gptr = const __attribute__((address_space(1))) T *;
template <typename T>
__device__ __forceinline__ gptr<T> gp(const T *p) { return (gptr<T>)p; }

// Workgroups beside the n <= 8 that run the cycle, which read what these will
// read: workgroup 8 h + k of the launch, h >= 1, k < n (the dispatcher deals
// workgroups to the 8 XCDs in turn, so that it shares an L2 with workgroup k;
// elsewhere it only does no good).  After the fine levels' sweeps the L2 holds
// nothing of the small levels, and one CU alone fetches 20 to 40 B/ns.
constexpr int TAIL_HELPERS = 8;
__device__ __forceinline__ void tail_warm(const TailLevel *tab, int nlev, int n) {
    if ((int)(blockIdx.x & 7) >= n) return;
    const int64_t step = (int64_t)TAIL_HELPERS * TAIL_WG * 128;
    int v = 0;
    for (int l = 0; l < nlev; ++l) {
#pragma unroll 1
        for (const auto &w : tab[l].warm) {
            const int64_t at = ((int64_t)(blockIdx.x / 8 - 1) * TAIL_WG + threadIdx.x) * 128;
            const gptr<unsigned char> p = gp(static_cast<const unsigned char *>(w.p));
            for (int64_t o = at; o < w.bytes; o += step) v ^= p[o];
        }
    }
    asm volatile("" ::"v"(v));   // the loads are wanted, not their values
}

// LDS elements of a vector of m rows (16-byte ranges)
template <typename T>
__host__ __device__ __forceinline__ int tail_range(int m) { return (m + 3) & ~3; }

// Dot products of SELL rows against a vector, streamed U entries at a time:
// acc += sum_k val_k x[col_k - lo], k in order (as the per-level kernels).  The
// loads of the next U beside the products of these measured 5 to 10% slower.
template <typename T, int U = 8>
__device__ __forceinline__ T tail_row(const int32_t *col, const T *val, int64_t off, int len, int lo, const T *x, T acc) {
    const gptr<int32_t> scol = gp(col);
    const gptr<T> sval = gp(val);
    for (int e0 = 0; e0 < len; e0 += U) {
        int cc[U];
        T aa[U], xv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            cc[u] = lo;
            aa[u] = T(0);
            if (e0 + u < len) {
                cc[u] = scol[off + (int64_t)(e0 + u) * 64];
                aa[u] = sval[off + (int64_t)(e0 + u) * 64];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) xv[u] = x[cc[u] - lo];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (e0 + u < len) acc += aa[u] * xv[u];
    }
    return acc;
}

// Butterfly sum over the wavefront in lane distances 32, 16, 8, 4, 2, 1 (the
// order of direct_row's shuffles, and every lane the same bits) without the LDS
// pipe that __shfl_xor goes through: 16 wavefronts' shuffles took most of a
// direct solve.  From distance 8 on the values repeat with that period, so that
// rotating a row of 16 lanes pairs the same values.
template <int CTRL>
__device__ __forceinline__ double tail_dpp(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const int lo = __builtin_amdgcn_mov_dpp((int)(uint32_t)u, CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_mov_dpp((int)(u >> 32), CTRL, 0xf, 0xf, false);
    return __builtin_bit_cast(double, (uint64_t)(uint32_t)hi << 32 | (uint32_t)lo);
}
__device__ __forceinline__ double tail_wave_sum(double v) {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    // permlane32_swap of (v, v): both halves' values side by side in every lane
    u2 lo = __builtin_amdgcn_permlane32_swap((uint32_t)u, (uint32_t)u, false, false);
    u2 hi = __builtin_amdgcn_permlane32_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
    v = __builtin_bit_cast(double, (uint64_t)hi[0] << 32 | lo[0]) + __builtin_bit_cast(double, (uint64_t)hi[1] << 32 | lo[1]);
    const uint64_t w = __builtin_bit_cast(uint64_t, v);
    lo = __builtin_amdgcn_permlane16_swap((uint32_t)w, (uint32_t)w, false, false);
    hi = __builtin_amdgcn_permlane16_swap((uint32_t)(w >> 32), (uint32_t)(w >> 32), false, false);
    v = __builtin_bit_cast(double, (uint64_t)hi[0] << 32 | lo[0]) + __builtin_bit_cast(double, (uint64_t)hi[1] << 32 | lo[1]);
    v += tail_dpp<0x128>(v);   // row_ror:8
    v += tail_dpp<0x124>(v);
    v += tail_dpp<0x122>(v);
    v += tail_dpp<0x121>(v);
    return v;
}

// Rows [a, m) of the system's direct segments: x = A_seg^{-1} b with FP64
// accumulation, a wavefront per row (as direct_row), up to four rows of a
// segment at a time.  Segment, rows and bounds are uniform, and b is read once
// for the four: with a search and a test per row and entry, a segment of 144
// rows took 10 us on a workgroup's 16 wavefronts.
template <typename T>
__device__ __forceinline__ void tail_direct(const TailLevel &L, int lo, int a, int m, const T *b, T *x) {
    constexpr int NW = TAIL_WG / 64, U = 4, J = 2;
    const int lane = threadIdx.x & 63;
    for (int i = a + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); i < m;) {
        int p = 0, h = L.nseg - 1;   // segment p with dseg[p] <= lo + i < dseg[p + 1]
        while (p < h) {
            const int mid = (p + h + 1) >> 1;
            if (gp(L.dseg)[mid] <= lo + i) p = mid;
            else h = mid - 1;
        }
        const int s = (int)(gp(L.dseg)[p] - lo), n = (int)(gp(L.dseg)[p + 1] - gp(L.dseg)[p]);
        const gptr<double> inv = gp(L.dinv) + gp(L.dinv_off)[p];
        while (i < s + n) {
            gptr<double> row[U];
            double acc[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {   // beyond the segment: the last row again
                acc[u] = 0.0;
                row[u] = inv + (int64_t)(min(i + u * NW, s + n - 1) - s) * n;
            }
            for (int j0 = 0; j0 < n; j0 += 64 * J) {
                double av[J][U], bj[J];
#pragma unroll
                for (int q = 0; q < J; ++q) {
                    const int j = min(j0 + q * 64 + lane, n - 1);
#pragma unroll
                    for (int u = 0; u < U; ++u) av[q][u] = row[u][j];
                    bj[q] = (double)b[s + j];
                }
#pragma unroll
                for (int q = 0; q < J; ++q)
                    if (j0 + q * 64 + lane < n) {
#pragma unroll
                        for (int u = 0; u < U; ++u) acc[u] += av[q][u] * bj[q];
                    }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) acc[u] = tail_wave_sum(acc[u]);
            if (lane == 0) {
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (i + u * NW < s + n) x[i + u * NW] = (T)acc[u];
            }
            i += NW * min(U, (s + n - i + NW - 1) / NW);   // the next of this wavefront, in this segment or beyond
        }
    }
}

}  // namespace
}  // namespace cs
