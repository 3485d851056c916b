// Tail V-cycle (gfx950, wave64): the small levels of a V-cycle in one launch.
#include <algorithm>
#include <type_traits>

#include <hip/hip_ext.h>

#include "cs_internal.h"
#include "tail_device.h"

namespace cs {

namespace {

// ---------------------------------------------------------------------------
// Tail V-cycle: the small levels are bound by latency (a kernel launch and
// three dependent trips to the L2 per sweep, transfer and direct solve, for a
// few KB of data), so Alg. 1 on all of them is one launch.  A workgroup of
// 1024 threads runs the whole cycle for one right-hand side of one independent
// system, with every level's x and b in LDS, a workgroup barrier where the
// per-level path has a kernel boundary, and A, x and b of a thread's rows in
// registers over all sweeps of a visit where a row has at most tail_ml entries
// (longer rows stream from the L2).  The right-hand sides and the systems of a
// batch do not see each other, so they go to different CUs.  Every row's
// arithmetic is the per-level kernels' own, in the same order: identical
// results.
// What bounds it is one CU: about 0.4 us per sweep up to 1024 point rows and 2 us
// at 4096 (a per-level launch takes 3.5-4 us), but as much as a launch for 1728
// rows of 8x8 FP64 blocks (110 KB of Lambda per sweep), so cs_autotune picks the
// first level by timing.  One V(2,2) of the 64^2 FP64 problem: 142 us with a
// launch per step, 93 us in the form with all vectors in the L2 and one
// workgroup for all right-hand sides and systems, 49 us now; V-cycle of 16
// systems of 64^2 to 176^2 with 4 right-hand sides: 118 us per level, 82 now.
// Behind large levels (96^3 FP64, from 1728 rows of 8x8 blocks on) the workgroups
// of tail_warm are worth 18 us of a 375 us V-cycle.
// ---------------------------------------------------------------------------
// Entries per row and rows per thread held in registers, what 128 VGPRs (1024
// threads) take without spilling: the 5-point stencil of point levels, the
// 7-point stencil of block levels; 4 rows (4096-row levels) but for FP64 blocks.
template <int NB>
constexpr int tail_ml() { return NB == 1 ? 5 : 7; }
template <typename T, int NB>
constexpr int tail_tpt() { return sizeof(T) == 8 && NB > 1 ? 2 : 4; }

// The rows of A that a thread owns on a level (row = thread + i * TAIL_WG of
// the system's m active rows), in registers: values and byte offsets of the
// columns in x.  Shorter rows are filled up with zeros at the row's own column,
// threads beyond row m - 1 repeat it.
template <typename T, int TPT, int ML>
struct TailRows {
    T v[TPT][ML];
    uint32_t c[TPT][ML];   // byte offsets
    __device__ __forceinline__ void load(const TailLevel &L, int lo, int m) {
        int64_t off[TPT];
        int len[TPT];
#pragma unroll
        for (int i = 0; i < TPT; ++i) {
            const int q = lo + min((int)threadIdx.x + i * TAIL_WG, m - 1);
            // a wavefront's 64 rows lie in at most two slices: scalar loads
            const int s0 = __builtin_amdgcn_readfirstlane(q >> 6);
            const int s1 = min(s0 + 1, (lo + m - 1) >> 6);
            const bool first = (q >> 6) == s0;
            len[i] = first ? gp(L.slen)[s0] : gp(L.slen)[s1];
            off[i] = (first ? gp(L.sptr)[s0] : gp(L.sptr)[s1]) + (q & 63);
        }
        const gptr<T> sval = gp(static_cast<const T *>(L.sval));
        const gptr<int32_t> scol = gp(L.scol);
#pragma unroll
        for (int i = 0; i < TPT; ++i) {
            const int own = min((int)threadIdx.x + i * TAIL_WG, m - 1);
#pragma unroll
            for (int u = 0; u < ML; ++u) {
                int cc = own;
                v[i][u] = T(0);
                if (u < len[i]) {
                    cc = scol[off[i] + (int64_t)u * 64] - lo;
                    v[i][u] = sval[off[i] + (int64_t)u * 64];
                }
                c[i][u] = (uint32_t)cc * sizeof(T);
            }
        }
    }
    __device__ __forceinline__ T dot(int i, const T *x, T acc) const {
        T xv[ML];
#pragma unroll
        for (int u = 0; u < ML; ++u) xv[u] = *reinterpret_cast<const T *>(reinterpret_cast<const unsigned char *>(x) + c[i][u]);
#pragma unroll
        for (int u = 0; u < ML; ++u) acc += v[i][u] * xv[u];
        return acc;
    }
};

// x_out = x_in - Lambda res for one row (local index row, NB consecutive lanes
// per block), res exchanged inside the wavefront through the row's own slot of
// xout: LDS operations of a wavefront complete in order, and xout is not read
// as an x by anybody before the next barrier.
template <typename T, int NB>
__device__ __forceinline__ void tail_relax(bool valid, int row, T res, T &xo, const T (&lr)[NB], T *xout) {
    if constexpr (NB == 1) {
        xo -= lr[0] * res;
    } else {
        if (valid) xout[row] = res;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        T rb[NB];
        const int base = row - row % NB;
#pragma unroll
        for (int cc = 0; cc < NB; ++cc) rb[cc] = valid ? xout[base + cc] : T(0);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int cc = 0; cc < NB; ++cc) xo -= lr[cc] * rb[cc];
    }
    if (valid) xout[row] = xo;
}

// The row's entries of Lambda (16-byte loads where a row has as many).
template <typename T, int NB>
__device__ __forceinline__ void tail_lam(const T *lam, int lo, int row, int m, T (&lr)[NB]) {
    const int q = lo + min(row, m - 1);
    const gptr<T> p = gp(lam) + (int64_t)(q / NB) * (NB * NB) + (q % NB) * NB;
    if constexpr (NB * sizeof(T) >= 16) {
        typedef uint32_t u4 __attribute__((ext_vector_type(4)));
        const auto v = (const __attribute__((address_space(1))) u4 *)p;
#pragma unroll
        for (int k = 0; k < (int)(NB * sizeof(T) / 16); ++k) {
            const u4 u = v[k];
            __builtin_memcpy(&lr[k * (16 / sizeof(T))], &u, 16);
        }
    } else {
#pragma unroll
        for (int c = 0; c < NB; ++c) lr[c] = p[c];
    }
}

// Lambda of sweep q of a visit: the cascade's steps in order, or (rf) in
// reverse order and transposed.
template <typename T>
__device__ __forceinline__ const T *tail_step(const TailLevel &L, int q, int rf) {
    const int st = q % L.depth, ell = rf ? L.depth - 1 - st : st;
    return static_cast<const T *>(rf ? L.lamT : L.lam) + (int64_t)ell * L.nbl;
}

// ns sweeps x_out = x_in - Lambda (A x_in - b) over the rows [0, m) of one
// level's system, the first reading cur (or from a zero guess) and writing
// nxt, which then alternate with x and alt; every sweep ends with a barrier.
// With `res` the residual A x - b of the result is left in alt (no barrier).
// The thread's rows of A, x and b stay in registers, and the Lambda of a sweep
// is loaded before the barrier that ends the one before it.
template <typename T, int NB, int TPT>
__device__ __forceinline__ void tail_smooth(const TailLevel &L, int lo, int m, const T *b, T *x, T *alt, T *cur, T *nxt,
                                            int ns, int rf, bool zero, bool res) {
    TailRows<T, TPT, tail_ml<NB>()> A;
    A.load(L, lo, m);
    T lr[TPT][NB], xo[TPT], bv[TPT];
#pragma unroll
    for (int i = 0; i < TPT; ++i) {
        const int row = min((int)threadIdx.x + i * TAIL_WG, m - 1);
        tail_lam<T, NB>(tail_step<T>(L, 0, rf), lo, row, m, lr[i]);
        bv[i] = b[row];
        xo[i] = zero ? T(0) : cur[row];
    }
    for (int q = 0; q < ns; ++q) {
        const T *lam = tail_step<T>(L, q + 1 < ns ? q + 1 : q, rf);
#pragma unroll
        for (int i = 0; i < TPT; ++i) {
            if (i * TAIL_WG < m) {   // uniform
                const int row = threadIdx.x + i * TAIL_WG;
                const T r = zero && q == 0 ? -bv[i] : A.dot(i, cur, -bv[i]);
                tail_relax<T, NB>(row < m, row, r, xo[i], lr[i], nxt);
                tail_lam<T, NB>(lam, lo, row, m, lr[i]);
            }
        }
        __syncthreads();
        cur = nxt;
        nxt = cur == x ? alt : x;
    }
    if (res) {
#pragma unroll
        for (int i = 0; i < TPT; ++i) {
            const int row = threadIdx.x + i * TAIL_WG;
            if (i * TAIL_WG < m && row < m) alt[row] = A.dot(i, x, -bv[i]);
        }
    }
}

// The same sweeps with A streamed from memory.
template <typename T, int NB>
__device__ __forceinline__ void tail_smooth_stream(const TailLevel &L, int lo, int m, const T *b, T *x, T *alt, T *cur,
                                                   T *nxt, int ns, int rf, bool zero, bool res) {
    const T *sval = static_cast<const T *>(L.sval);
    for (int q = 0; q < ns; ++q) {
        const T *lam = tail_step<T>(L, q, rf);
        for (int r0 = 0; r0 < m; r0 += TAIL_WG) {
            const int row = r0 + threadIdx.x, g = lo + row;
            const bool valid = row < m;
            T lr[NB], r = T(0), xo = T(0);
            tail_lam<T, NB>(lam, lo, row, m, lr);
            if (valid) {
                r = -b[row];
                if (!(zero && q == 0)) {
                    r = tail_row<T>(L.scol, sval, gp(L.sptr)[g >> 6] + (g & 63), gp(L.slen)[g >> 6], lo, cur, r);
                    xo = cur[row];
                }
            }
            tail_relax<T, NB>(valid, row, r, xo, lr, nxt);
        }
        __syncthreads();
        cur = nxt;
        nxt = cur == x ? alt : x;
    }
    if (res)
        for (int row = threadIdx.x; row < m; row += TAIL_WG) {
            const int g = lo + row;
            alt[row] = tail_row<T>(L.scol, sval, gp(L.sptr)[g >> 6] + (g & 63), gp(L.slen)[g >> 6], lo, x, -b[row]);
        }
}

// One visit's sweeps in the form that the level's rows allow.
template <typename T, int NB>
__device__ __forceinline__ void tail_visit(const TailLevel &L, int lo, int m, const T *b, T *x, T *alt, T *cur, T *nxt,
                                           int ns, int rf, bool zero, bool res) {
    constexpr int TPT = tail_tpt<T, NB>();
    if (L.max_len > tail_ml<NB>() || m > TPT * TAIL_WG)
        tail_smooth_stream<T, NB>(L, lo, m, b, x, alt, cur, nxt, ns, rf, zero, res);
    else if (m > TAIL_WG)
        tail_smooth<T, NB, TPT>(L, lo, m, b, x, alt, cur, nxt, ns, rf, zero, res);
    else
        tail_smooth<T, NB, 1>(L, lo, m, b, x, alt, cur, nxt, ns, rf, zero, res);
}

// Alg. 1 from tab[0] (its right-hand side in global memory, [n][R]: tab[0].bb,
// or the FP64 vector b64) to the last entry; the result in tab[0].xb, or x64.  Workgroup (system, right-hand side).
// sys: [nlev][nsys + 1] row offsets of the systems on every level.  LDS: x and
// b of every level, then one buffer of the largest level's rows (`alt`): a
// sweep writes the other one of x and alt, started so that the last one of
// a visit ends in x.
template <typename T, int NB>
__global__ __launch_bounds__(TAIL_WG) void k_tail_vcycle(const TailLevel *__restrict__ tab, int nlev, int nsys,
                                                         const int32_t *__restrict__ sys, int R, int n_pre,
                                                         int n_post, int rf, int alt_off,
                                                         const double *__restrict__ b64, double *x64, int add) {
    extern __shared__ __align__(16) unsigned char tail_lds[];
    T *const base = reinterpret_cast<T *>(tail_lds);
    T *const alt = base + alt_off;
    if ((int)blockIdx.x >= nsys * R) {
        tail_warm(tab, nlev, nsys * R);
        return;
    }
    const int s = blockIdx.x % nsys, k = blockIdx.x / nsys;
    // x_l at x, b_l at x + m (m rows on the level, up to 16-byte ranges)
    int last = 0;   // the system's last level: nothing of it is smoothed there
    T *x = base;
    {
        const TailLevel &L = tab[0];
        const int lo = sys[s], m = sys[s + 1] - lo;
        T *b = x + tail_range<T>(m);
        const gptr<T> gb = gp(static_cast<const T *>(L.bb));
        for (int r = threadIdx.x; r < m; r += TAIL_WG) {
            const int64_t e = (int64_t)(lo + r) * R + k;
            b[r] = b64 ? (T)b64[e] : gb[e];
        }
        __syncthreads();
    }
    for (int l = 0;; ++l) {
        const TailLevel &L = tab[l];
        const int lo = sys[l * (nsys + 1) + s], m = sys[l * (nsys + 1) + s + 1] - lo;
        const int act = max(0, min((int)L.n_active - lo, m));
        T *b = x + tail_range<T>(m);
        tail_direct<T>(L, lo, act, m, b, x);   // reads b only
        if (l + 1 == nlev || act == 0) {
            last = l;
            __syncthreads();
            break;
        }
        const int ns = n_pre * L.depth;
        tail_visit<T, NB>(L, lo, act, b, x, alt, x, (ns & 1) ? x : alt, ns, rf, true, true);   // ends in x
        __syncthreads();
        const int mc = sys[(l + 1) * (nsys + 1) + s + 1] - sys[(l + 1) * (nsys + 1) + s];
        T *xn = b + tail_range<T>(m), *bn = xn + tail_range<T>(mc);
        const T rs = (T)L.r_scale;
        for (int I = threadIdx.x; I < mc; I += TAIL_WG) {
            T v = T(0);
            if (L.agg_k > 0) {
                for (int u = 0; u < L.agg_k; ++u) v += alt[I * L.agg_k + u];
            } else {
                v = tail_row<T>(L.tcol, static_cast<const T *>(L.tval), gp(L.tptr)[I >> 6] + (I & 63), gp(L.tlen)[I >> 6], 0,
                                alt, v);
            }
            bn[I] = v * rs;
        }
        __syncthreads();
        x = xn;
    }
    for (int l = last - 1; l >= 0; --l) {
        const TailLevel &L = tab[l];
        const int lo = sys[l * (nsys + 1) + s], m = sys[l * (nsys + 1) + s + 1] - lo;
        const int act = max(0, min((int)L.n_active - lo, m));
        const T *xc = x;
        T *b = x - tail_range<T>(m);
        x = b - tail_range<T>(m);
        const int ns = n_post * L.depth;
        T *cur = (ns & 1) ? alt : x;
        const int sh = L.agg_k > 0 ? __builtin_ctz((unsigned)L.agg_k) : 0;   // agg_k divides 64
        for (int row = threadIdx.x; row < act; row += TAIL_WG) {
            T v = x[row];
            if (L.agg_k > 0) v -= xc[row >> sh];
            else
                v -= tail_row<T>(L.pcol, static_cast<const T *>(L.pval), gp(L.pptr)[row >> 6] + (row & 63),
                                 gp(L.plen)[row >> 6], 0, xc, T(0));
            cur[row] = v;
        }
        __syncthreads();
        tail_visit<T, NB>(L, lo, act, b, x, alt, cur, cur == x ? alt : x, ns, 0, false, false);
    }
    const int lo = sys[s], m = sys[s + 1] - lo;
    auto gx = (__attribute__((address_space(1))) T *)static_cast<T *>(tab[0].xb);
    for (int r = threadIdx.x; r < m; r += TAIL_WG) {
        const int64_t e = (int64_t)(lo + r) * R + k;
        if (x64) x64[e] = add ? x64[e] + (double)x[r] : (double)x[r];
        else gx[e] = x[r];
    }
}

template <class F>
void tail_dispatch(int nb, F &&f) {
    switch (nb) {
        case 1: f(std::integral_constant<int, 1>{}); break;
        case 2: f(std::integral_constant<int, 2>{}); break;
        case 4: f(std::integral_constant<int, 4>{}); break;
        case 8: f(std::integral_constant<int, 8>{}); break;
        default: fail(CS_EINVAL, "tail block size must be 1, 2, 4 or 8");
    }
}

template <typename T>
const T *pick(const DBuf<double> &d, const DBuf<float> &f) {
    if constexpr (std::is_same<T, double>::value) return d.get();
    else return f.get();
}

template <typename T>
size_t pick_n(const DBuf<double> &d, const DBuf<float> &f) {
    if constexpr (std::is_same<T, double>::value) return d.n;
    else return f.n;
}

}  // namespace

namespace {

// Dynamic LDS that a workgroup may use (160 KB per CU on gfx950).
int64_t tail_lds_limit(const Ctx &c) {
    int v = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, c.device) != hipSuccess) return 65536;
    return v;
}

// Row offsets of the independent systems on every level, [level][nsys + 1]: a
// batch under aggregation splits as its finest level does, provided that no
// row of levels >= from couples two systems; anything else is one system.
std::vector<std::vector<int32_t>> tail_systems(const Ctx &c, int from) {
    const int nl = (int)c.lv.size();
    std::vector<std::vector<int32_t>> rng(nl);
    bool split = c.sys_ptr.size() > 2;
    if (split) rng[0].assign(c.sys_ptr.begin(), c.sys_ptr.end());
    for (int l = 0; split && l + 1 < nl; ++l) {
        const Level &L = c.lv[l];
        split = c.fuse_transfers && L.agg_k > 0;
        for (size_t q = 0; split && q < rng[l].size(); ++q) {
            const int64_t r = std::min<int64_t>(rng[l][q], L.n_active);
            split = r % L.agg_k == 0;
            rng[l + 1].push_back((int32_t)(r / std::max(L.agg_k, 1)));
        }
        split = split && rng[l + 1].back() == c.lv[l + 1].n;
    }
    for (int l = from; split && l < nl; ++l) {
        const Level &L = c.lv[l];
        for (size_t q = 0; split && q + 1 < rng[l].size(); ++q) {
            const int32_t r0 = rng[l][q], r1 = rng[l][q + 1];
            split = r0 % L.nb == 0;
            for (int64_t e = L.h_ptr[r0]; split && e < L.h_ptr[r1]; ++e) split = L.h_col[e] >= r0 && L.h_col[e] < r1;
            for (size_t t = 0; split && t + 1 < L.dseg.size(); ++t)   // a segment belongs to one system
                split = !(L.dseg[t] < r1 && L.dseg[t + 1] > r0) || (L.dseg[t] >= r0 && L.dseg[t + 1] <= r1);
        }
    }
    if (!split)
        for (int l = 0; l < nl; ++l) rng[l] = {0, (int32_t)c.lv[l].n};
    return rng;
}

// LDS elements of the tail from level `from` for its largest system: x and b
// of every level (in *alt), and the buffer of the largest level after them.
int64_t tail_elements(const std::vector<std::vector<int32_t>> &rng, int from, int64_t *alt) {
    int64_t xb = 0, top = 0;
    for (size_t s = 0; s + 1 < rng[0].size(); ++s) {
        int64_t t = 0;
        for (size_t l = from; l < rng.size(); ++l) {
            const int64_t m = tail_range<float>(rng[l][s + 1] - rng[l][s]);
            t += 2 * m;
            top = std::max(top, m);
        }
        xb = std::max(xb, t);
    }
    if (alt) *alt = xb;
    return xb + top;
}

}  // namespace

static bool tail_b16(const Ctx &c) { return c.opt.mode == CS_MULTIPLICATIVE && c.precision == CS_BF16; }

// LDS bytes of the BF16 tail beside the vectors: a block of zeros and the schedules.
static int64_t tail16_extra(const Ctx &c, bool b16, int from) {
    int64_t n = 0;
    for (size_t l = from; b16 && l + 1 < c.lv.size(); ++l) n += tail16_schedule_words(c.lv[l]) * 4;
    return b16 ? n + 64 : 0;
}

// A level of general transfers whose rows are too long for registers streams A
// from the L2 through one CU in every sweep, 12 us for 39,300 entries in FP64 and
// 9 in FP32, which a launch per step does on all of them: such a level is covered
// up to STREAM_MAX bytes of A, or STREAM_MAX0 where the tail is the whole V-cycle
// (its A stays in the L2, and no conversions are launched).  One V-cycle of the
// 27-point problem, per-level launches / tail, one right-hand side: 24^3 from 1,728
// rows in FP32 (307 KB) 101 / 90 us and in FP64 (460 KB) 103 / 108, 48^3 from there
// 125 / 128 and 132 / 163; 32^3 from 4,096 rows (760 KB, 1,140 KB) 125 / 129 and
// 126 / 184; from level 0 12^3 in FP64 (460 KB) 76 / 71, 16^3 in FP32 (760 KB)
// 102 / 87 and in FP64 (1,140 KB) 102 / 135.
constexpr int64_t STREAM_MAX = 320 << 10, STREAM_MAX0 = 800 << 10;

static bool tail_streams_well(const Ctx &c, int l) {
    const Level &L = c.lv[l];
    if ((c.fuse_transfers && L.agg_k > 0) || L.act_row <= (L.nb == 1 ? tail_ml<1>() : tail_ml<8>())) return true;
    return L.act_nnz * (c.precision == CS_FP64 ? 12 : 8) <= (l == 0 ? STREAM_MAX0 : STREAM_MAX);
}

// The levels the tail kernel covers: the first level l (the finest included)
// from which every level has at most c.tail_rows rows, every smoothed one is
// additive (no overlapping blocks) with one common block size of 1, 2, 4 or 8,
// none streams more than it may, the cycle pre- and post-smooths, and a system's vectors on all covered levels
// fit a workgroup's LDS; -1 when there is none.  Multicoloured levels are
// covered where the sweeps run in BF16 (16x16 blocks, one right-hand side, no
// direct segments above the last level).
int tail_start(const Ctx &c, int nrhs) {
    const int nl = (int)c.lv.size();
    if (c.tail_rows <= 0 || nl < 2 || c.opt.n_pre < 1 || c.opt.n_post < 1) return -1;
    const int64_t nb = c.lv[nl - 2].nb;
    const bool b16 = tail_b16(c);
    if (b16 ? nrhs != 1 : (c.opt.mode != CS_ADDITIVE || (nb != 1 && nb != 2 && nb != 4 && nb != 8))) return -1;
    int from = -1;
    for (int l = nl - 1; l >= 0; --l) {
        const Level &V = c.lv[l];
        bool ok = V.n <= c.tail_rows && !V.ovl_m;
        if (l + 1 < nl) ok = ok && V.depth >= 1 && V.nb == nb && V.n_active > 0;
        if (l + 1 < nl && b16)
            ok = ok && use_bf16(c, V) && !V.h_bmeta.empty() && V.lam16.get() && V.n_active == V.n;
        else if (l + 1 < nl)
            ok = ok && tail_streams_well(c, l);
        if (!ok) break;
        from = l;
    }
    if (from < 0 || from >= nl - 1) return -1;
    const auto rng = tail_systems(c, from);
    if (b16 && rng[0].size() != 2) return -1;   // one system
    const int64_t es = c.precision == CS_FP64 ? 8 : 4, lim = tail_lds_limit(c);
    while (from < nl - 1 && tail_elements(rng, from, nullptr) * es + tail16_extra(c, b16, from) > lim) ++from;
    return from < nl - 1 ? from : -1;
}

namespace {

template <typename T>
void tail_table(Ctx &c, int nrhs) {
    if (c.tail_gen == c.gen && c.tail_prec == c.precision && c.tail_nrhs == nrhs) return;
    const int from = tail_start(c, nrhs);
    c.tail_from = from;
    if (from < 0) return;
    c.tail_b16 = tail_b16(c);
    const auto rng = tail_systems(c, from);
    c.tail_sched_host.clear();
    int64_t alt = 0;
    const int64_t el = tail_elements(rng, from, &alt);   // vectors of the levels, then (from alt on) one more
    if (c.tail_b16) {
        for (size_t l = from; l + 1 < c.lv.size(); ++l)
            tail16_schedule(c.lv[l], (uint32_t)(el - alt) * 4, c.tail_sched_host);
        c.tail_sched.upload(c.tail_sched_host.data(), c.tail_sched_host.size(), c.stream);
    }
    int64_t soff = 0;
    int64_t aoff = 0;
    if (c.tail_b16) {
        for (size_t l = from; l + 1 < c.lv.size(); ++l) aoff += tail16_pack(c, c.lv[l], nullptr);
        c.tail_a16.alloc(aoff);
        aoff = 0;
    }
    std::vector<TailLevel> tab;
    std::vector<int32_t> sys;
    const double es = sizeof(T), vr = (double)nrhs * es;
    double bytes = 0.0;
    for (size_t l = from; l < c.lv.size(); ++l) {
        const Level &L = c.lv[l];
        const bool agg = c.fuse_transfers && L.agg_k > 0;
        sys.insert(sys.end(), rng[l].begin(), rng[l].end());
        bytes += (double)L.dinv.n * 8.0 + 2.0 * (L.n - L.n_active) * vr;
        TailLevel t{};
        int nw = 0;
        auto warm = [&](const void *p, int64_t n) {
            if (p && n > 0) t.warm[nw++] = {p, n};
        };
        if (l + 1 < c.lv.size()) {
            const double A = L.act_nnz * (es + 4.0), lamb = (double)L.n_active * L.nb * (c.tail_b16 ? 2.0 : es);
            const double As = c.tail_b16 ? (double)L.bsr_nnzb * 512.0 : A;   // what the sweeps read
            const double v = (double)L.n_active * vr, sweeps = (double)(c.opt.n_pre + c.opt.n_post) * L.depth;
            bytes += (lamb + 2.0 * v) + (sweeps - 1.0) * (As + lamb + 3.0 * v);   // the first from zero
            bytes += A + 2.0 * v + 2.0 * (double)L.nc * vr + (agg ? 0.0 : 2.0 * L.p_nnz * (es + 4.0));   // transfers
            t.lam = pick<T>(L.lam64, L.lam32);
            t.lamT = pick<T>(L.lam64T, L.lam32T);
            t.max_len = L.act_row;
            if (c.tail_b16) {
                t.nitems = tail16_rounds(L);
                t.sched = (int)(soff / 4);
                soff += tail16_schedule_words(L);
                t.bmeta = L.bmeta.get();
                t.bcol = L.bsr_col.get();
                t.a16 = L.a16.get();
                t.ar16 = c.tail_a16.get() + aoff;
                const int64_t na = tail16_pack(c, L, c.tail_a16.get() + aoff);
                aoff += na;
                warm(t.ar16, na * 2);
                warm(L.lam16.get(), (int64_t)L.lam16.n * 2);
                if (c.opt.order == CS_RF) warm(L.lam16T.get(), (int64_t)L.lam16T.n * 2);
                t.lam16 = L.lam16.get();
                t.lam16T = L.lam16T.get();
            }
            if (!agg || c.tail_b16) {
                t.pptr = L.psell.slice_ptr.get();
                t.plen = L.psell.slice_len.get();
                t.pcol = L.psell.col.get();
                t.pval = pick<T>(L.psell.val64, L.psell.val32);
                t.tptr = L.ptsell.slice_ptr.get();
                t.tlen = L.ptsell.slice_len.get();
                t.tcol = L.ptsell.col.get();
                t.tval = pick<T>(L.ptsell.val64, L.ptsell.val32);
            }
        }
        t.n_active = L.n_active;
        t.nbl = L.B * L.nb * L.nb;
        t.sptr = L.sell.slice_ptr.get();
        t.slen = L.sell.slice_len.get();
        t.scol = L.sell.col.get();
        t.sval = pick<T>(L.sell.val64, L.sell.val32);
        t.bb = L.w_bb;
        t.xb = L.w_xb;
        t.depth = L.depth;
        t.agg_k = agg ? L.agg_k : 0;
        t.r_scale = L.r_scale;
        if (l + 1 < c.lv.size()) {
            warm(t.sval, (int64_t)pick_n<T>(L.sell.val64, L.sell.val32) * sizeof(T));
            warm(t.scol, (int64_t)L.sell.col.n * 4);
            if (!c.tail_b16) {
                warm(t.lam, t.nbl * L.depth * (int64_t)sizeof(T));
                if (c.opt.order == CS_RF) warm(t.lamT, t.nbl * L.depth * (int64_t)sizeof(T));
            }
            if (t.pptr) {
                warm(t.tval, (int64_t)pick_n<T>(L.ptsell.val64, L.ptsell.val32) * sizeof(T));
                warm(t.tcol, (int64_t)L.ptsell.col.n * 4);
                warm(t.pval, (int64_t)pick_n<T>(L.psell.val64, L.psell.val32) * sizeof(T));
                warm(t.pcol, (int64_t)L.psell.col.n * 4);
            }
        }
        warm(L.dinv.get(), (int64_t)L.dinv.n * 8);
        t.nseg = L.dseg.size() > 1 ? (int)L.dseg.size() - 1 : 0;
        t.dseg = L.dseg_d.get();
        t.dinv_off = L.dinv_off.get();
        t.dinv = L.dinv.get();
        tab.push_back(t);
    }
    c.tail_lds = el * sizeof(T) + tail16_extra(c, c.tail_b16, from);
    c.tail_zero = (int)el;
    c.tail_alt = (int)alt;
    c.tail_nsys = (int)rng[from].size() - 1;
    c.tail_host = tab;
    c.tail_sys_host = sys;
    c.tail_bytes = bytes;
    c.tail_tab.upload(c.tail_host.data(), c.tail_host.size(), c.stream);
    c.tail_sys.upload(c.tail_sys_host.data(), c.tail_sys_host.size(), c.stream);
    if (c.tail_b16) tail16_prepare(tail_lds_limit(c));
    else tail_dispatch((int)c.lv[from].nb, [&](auto nbc) {
        constexpr int NB = decltype(nbc)::value;
        allow_lds(reinterpret_cast<const void *>(&k_tail_vcycle<T, NB>), tail_lds_limit(c));
    });
    c.tail_gen = c.gen;
    c.tail_prec = c.precision;
    c.tail_nrhs = nrhs;
}

template <typename T>
void launch(Ctx &c, int nrhs, const double *b64, double *x64, bool add) {
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    (void)trace_begin_launch(c, CS_TRACE_TAIL, c.tail_bytes, &ev0, &ev1);
    if (c.tail_b16) {
        tail16_launch(c, ev0, ev1, b64, x64, add);
        return;
    }
    // workgroups that warm the L2 where the cycle's own few come after other levels
    const unsigned n = (unsigned)(c.tail_nsys * nrhs);
    tail_dispatch((int)c.lv[c.tail_from].nb, [&](auto nbc) {
        constexpr int NB = decltype(nbc)::value;
        hipExtLaunchKernelGGL((k_tail_vcycle<T, NB>), dim3(n <= 8 && c.tail_from > 0 ? 8 * (1 + TAIL_HELPERS) : n), dim3(TAIL_WG), (unsigned)c.tail_lds,
                              c.stream, ev0, ev1, 0, (const TailLevel *)c.tail_tab.get(),
                              (int)c.lv.size() - c.tail_from, c.tail_nsys, (const int32_t *)c.tail_sys.get(), nrhs,
                              c.opt.n_pre, c.opt.n_post, c.opt.order == CS_RF ? 1 : 0, c.tail_alt, b64, x64, add ? 1 : 0);
    });
    CS_LAUNCH_CHECK();
}

}  // namespace

// Build the table of the covered levels for the current workspace (kept until
// the buffers, the precision, the right-hand sides or the limit change).
void tail_prepare(Ctx &c, int nrhs) {
    if (c.precision == CS_FP64) tail_table<double>(c, nrhs);
    else tail_table<float>(c, nrhs);
}

// The V-cycle from level c.tail_from down, in one launch; with b64 and x64 from
// and into those FP64 vectors instead of the level's workspace; with `add` the
// result is added to x64.
void tail_launch(Ctx &c, int nrhs, const double *b64, double *x64, bool add) {
    if (c.precision == CS_FP64) launch<double>(c, nrhs, b64, x64, add);
    else launch<float>(c, nrhs, b64, x64, add);
}

}  // namespace cs
