// Tail V-cycle of the BF16 multicoloured cascade (gfx950, wave64): the small
// levels of 16x16 blocks in one launch.
#include <algorithm>

#include <hip/hip_ext.h>

#include "bf16_device.h"
#include "cs_internal.h"
#include "tail_device.h"

namespace cs {

namespace {

// ---------------------------------------------------------------------------
// A multicoloured visit is a chain of depth x colours dependent steps, each a
// launch of about 4 us for a microsecond's work on the small levels.  Here one
// workgroup of 16 wavefronts runs Alg. 1 on all of them: x, b and the residual
// of every level in LDS (FP32), a wavefront per block row, a barrier where the
// per-level path has a kernel boundary.  The step's operands do not depend on
// x, so a wavefront loads the blocks of its next row, and the entry of the one
// after, while it computes its current row: the loads cross the barriers.
// The arithmetic is k_bsr16_sweep's (and the SELL kernels' for the residual and
// the transfers), in the same order: identical results.
// What bounds it is the instructions and LDS turns of a round of 16 rows, one
// row deep per wavefront: 0.6 us, 0.7 where a step is one round.  The levels of
// 12^2 and 6^2 elements and the direct solve of 3^2 take 85 us (213 us with a
// launch per step): V-cycle of the 96^2 SIPG problem 484 -> 410 us.  At 24^2 a
// step is 9 rounds, no faster than a launch, and its vectors and schedule do
// not fit the LDS beside the others'.
// ---------------------------------------------------------------------------
constexpr int NW = TAIL_WG / 64;

// A level's schedule (tail16_schedule): the steps in forward order, each in
// rounds of a row per wavefront, between SCHED_PAD rounds without rows; an entry
// is {Lambda block | flags, row of A, x of the row, x of its first five block
// columns} as byte offsets, ready to be added, with a block of zeros of x as
// the column of missing blocks.  Wavefronts without a row in a round have
// entries too, so that every load is issued unconditionally: behind a branch
// the compiler cannot count loads in flight and waits for all of them.
constexpr uint32_t S_FIRST = 1, S_LAST = 2, S_IDLE = 4, S_LONG = 8;   // first, last round of its step; more blocks
constexpr int SCHED_PAD = 4;

typedef short bf16x8 __attribute__((ext_vector_type(8)));
struct BRow {
    bf16x8 a01, a23;
    bf16x4 a4, l;
};
static_assert(META_COLS == 5, "two pairs of blocks and one");
constexpr int ROW16 = META_COLS * 256;   // a row of the tail's copy of A

// The tail's copy of A: the first five blocks of the active rows in colour
// order, zeros where a row has fewer, in pairs whose lanes' operands are
// neighbours: one 16-byte load per lane brings two blocks (a load of 8 bytes
// takes the vector cache as long: 0.8 -> 0.6 us per round).
__global__ __launch_bounds__(64) void k_pack_tail16(const int32_t *__restrict__ meta,
                                                    const unsigned short *__restrict__ a16,
                                                    unsigned short *__restrict__ out) {
    const int lane = threadIdx.x;
    const int32_t *m = meta + 8 * (int64_t)blockIdx.x;
    const int e0 = m[1], ne = m[2] - e0;
    unsigned short *o = out + (int64_t)blockIdx.x * ROW16;
    for (int c = 0; c < META_COLS; ++c) {
        bf16x4 v = {0, 0, 0, 0};
        if (c < ne) v = *reinterpret_cast<const bf16x4 *>(a16 + (int64_t)(e0 + c) * 256 + lane * 4);
        unsigned short *d = c < 4 ? o + (c >> 1) * 512 + lane * 8 + (c & 1) * 4 : o + 1024 + lane * 4;
        *reinterpret_cast<bf16x4 *>(d) = v;
    }
}

// hi and lo of an FP32 vector's blocks of four, interleaved: 16 bytes that a
// lane reads as its operands
struct HiLo {
    bf16x4 hi, lo;
};

__device__ __forceinline__ void split4(const float4 &x, HiLo &o) {
    const float v[4] = {x.x, x.y, x.z, x.w};
    split(v, o.hi, o.lo);
}

__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

// All steps over x (in place): x_i -= Lambda_i (sum_j A_ij x_j - b_i).  xs: x as
// BF16 pairs, kept with x (split once per update instead of by every
// neighbour); sched: the level's schedule in LDS.  The operands of the next row
// are in flight while a row is computed, and the entry of the one after.  A
// round costs its instructions (four wavefronts share a SIMD), hence the
// ready-made offsets: with entries unpacked by scalar code a round took 0.8 us.
// Ends with a barrier.
__device__ __forceinline__ void bsr16_visit(const TailLevel &L, const uint4 *sched, const float *b, float *x, HiLo *xs,
                                            int rf) {
    const int lane = threadIdx.x & 63, wv = uni(threadIdx.x >> 6), kg = lane >> 4;
    constexpr int NB = 2, NREC = 4;
    typedef const __attribute__((address_space(1))) bf16x4 *gv;
    typedef const __attribute__((address_space(1))) bf16x8 *gv8;
    const int n = L.nitems, step = rf ? -2 * NW : 2 * NW;
    const uint32_t end = rf ? S_FIRST : S_LAST, kb = kg * 16;
    const gptr<char> ar16 = gp((const char *)L.ar16), lam16 = gp((const char *)(rf ? L.lam16T : L.lam16));
    const uint4 *sp = sched + ((SCHED_PAD + (rf ? n - 1 : 0)) * NW + wv) * 2;
    struct Entry {
        uint32_t lam, a, row, c[META_COLS];
    };
    auto record = [&](Entry &E) {
        const uint4 p = sp[0], q = sp[1];
        sp += step;
        E = Entry{p.x, p.y, p.z, {p.w, q.x, q.y, q.z, q.w}};
    };
    auto fetch = [&](BRow &B, const Entry &E) {
        const gptr<char> a = ar16 + (E.a + lane * 16);
        B.a01 = *(gv8)a;
        B.a23 = *(gv8)(a + 1024);
        B.a4 = *(gv)(ar16 + (E.a + lane * 8) + 2048);
        B.l = *(gv)(lam16 + ((E.lam & ~511u) | (uint32_t)(lane * 8)));
    };
    auto relax = [&](const BRow &B, const Entry &E, BRow &N, const Entry &EN, Entry &E2) {
        if (uni(E.lam) & S_IDLE) {
            fetch(N, EN);
            record(E2);
            return;
        }
        const uint32_t own = E.row + kb;
        HiLo v[META_COLS];
#pragma unroll
        for (int c = 0; c < META_COLS; ++c) v[c] = *reinterpret_cast<const HiLo *>(reinterpret_cast<const char *>(xs) + (E.c[c] + kb));
        const float4 bv = *reinterpret_cast<const float4 *>(reinterpret_cast<const char *>(b) + own);
        float4 *const xp = reinterpret_cast<float4 *>(reinterpret_cast<char *>(x) + own);
        float4 xo = *xp;
        fetch(N, EN);   // while the LDS returns x
        record(E2);
        __builtin_amdgcn_sched_barrier(0);
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        const bf16x4 a[META_COLS] = {B.a01.lo, B.a01.hi, B.a23.lo, B.a23.hi, B.a4};
#pragma unroll
        for (int c = 0; c < META_COLS; ++c) {
            acc = mfma(a[c], v[c].hi, acc);
            acc = mfma(a[c], v[c].lo, acc);
        }
        if (uni(E.lam) & S_LONG) {   // the blocks beyond the fifth
            const gptr<int32_t> meta = gp(L.bmeta) + (int64_t)(uni(E.a) / (ROW16 * 2)) * 8, bcol = gp(L.bcol);
            const gptr<unsigned short> a16 = gp(L.a16);
            const int e1 = uni(meta[2]);
            for (int e = uni(meta[1]) + META_COLS; e < e1; ++e) {
                const bf16x4 ae = ((gv)(a16 + (int64_t)e * 256))[lane];
                const HiLo ve = xs[uni(bcol[e]) * 4 + kg];
                acc = mfma(ae, ve.hi, acc);
                acc = mfma(ae, ve.lo, acc);
            }
        }
        const float r[4] = {acc[0] - bv.x, acc[1] - bv.y, acc[2] - bv.z, acc[3] - bv.w};
        bf16x4 hi, lo;
        split(r, hi, lo);
        f32x4 y = {0.f, 0.f, 0.f, 0.f};
        y = mfma(B.l, hi, y);
        y = mfma(B.l, lo, y);
        xo.x -= y[0];
        xo.y -= y[1];
        xo.z -= y[2];
        xo.w -= y[3];
        HiLo s;
        split4(xo, s);
        // 16 lanes write the same four values: cheaper than a branch
        *xp = xo;
        *reinterpret_cast<HiLo *>(reinterpret_cast<char *>(xs) + own) = s;
    };

    BRow B[NB];
    Entry E[NREC];
    record(E[0]);
    record(E[1]);
    record(E[2]);
    fetch(B[0], E[0]);
    for (int it = 0; it < n; it += NREC) {   // static ring indices: no copies
#pragma unroll
        for (int d = 0; d < NREC; ++d) {
            if (it + d >= n) break;
            relax(B[d % NB], E[d], B[(d + 1) % NB], E[(d + 1) % NREC], E[(d + 3) % NREC]);
            if (uni(E[d].lam) & end) __syncthreads();   // the step's last round
        }
    }
}

// A SELL row of the wavefront's slice: acc + sum_k val_k x[col_k], k in order.
// The slice's length is uniform, and whole groups of 16 entries have no test.
__device__ __forceinline__ float slice_row(const int64_t *ptr, const int32_t *len_, const int32_t *col,
                                           const void *val, int slice, int lane, const float *x, float acc) {
    constexpr int U = 16;
    const int len = uni(gp(len_)[slice]);
    const int64_t off = gp(ptr)[slice];
    gptr<int32_t> c = gp(col) + (((int64_t)uni((int)(off >> 32)) << 32) | (uint32_t)uni((int)off));
    gptr<float> a = gp(static_cast<const float *>(val)) + (((int64_t)uni((int)(off >> 32)) << 32) | (uint32_t)uni((int)off));
    int k = 0;
    for (; k + U <= len; k += U, c += U * 64, a += U * 64) {
        int cc[U];
        float aa[U];
#pragma unroll
        for (int u = 0; u < U; ++u) cc[u] = c[u * 64 + lane];
#pragma unroll
        for (int u = 0; u < U; ++u) aa[u] = a[u * 64 + lane];
#pragma unroll
        for (int u = 0; u < U; ++u) acc += aa[u] * x[cc[u]];
    }
    for (; k < len; ++k, c += 64, a += 64) acc += a[lane] * x[c[lane]];
    return acc;
}

// Alg. 1 from tab[0] (right-hand side tab[0].bb, result tab[0].xb, or the FP64
// vectors b64 and x64) to the last entry.  rows: [level][2] = {0, rows}.  LDS:
// x and b of every level, then one residual of the largest, a block of
// zeros (zero_off) and the schedules.  Way down and way up share their code (a turn per visit): what a
// workgroup runs once it fetches from the L2, a cache line at a time.
__global__ __launch_bounds__(TAIL_WG) void k_tail_bsr16(const TailLevel *__restrict__ tab, int nlev,
                                                        const int32_t *__restrict__ rows, int n_pre, int n_post,
                                                        int rf, int alt_off, int zero_off,
                                                        const int32_t *__restrict__ sched, int sched_words, const double *__restrict__ b64,
                                                        double *x64, int add) {
    extern __shared__ __align__(16) unsigned char tail16_lds[];
    if (blockIdx.x) {
        tail_warm(tab, nlev, 1);
        return;
    }
    float *const base = reinterpret_cast<float *>(tail16_lds);
    float *const res = base + alt_off;   // outside the visits; inside, x as BF16 pairs
    HiLo *const xs = reinterpret_cast<HiLo *>(res);
    uint4 *const lsched = reinterpret_cast<uint4 *>(base + zero_off + 16);
    const int t = threadIdx.x, lane = t & 63, wv = uni(t >> 6);
    int m = uni(rows[1]);
    float *x = base;
    {
        const gptr<float> gb = gp(static_cast<const float *>(tab[0].bb));
        float *b = x + tail_range<float>(m);
        for (int r = t; r < m; r += TAIL_WG) b[r] = b64 ? (float)b64[r] : gb[r];
        if (t < 16) base[zero_off + t] = 0.f;
        for (int e = t; e < sched_words / 4; e += TAIL_WG) lsched[e] = reinterpret_cast<const uint4 *>(sched)[e];
    }
    const int nv = nlev - 1;   // smoothed levels
    for (int q = 0; q < 2 * nv; ++q) {
        const bool down = q < nv;
        const TailLevel &L = tab[down ? q : 2 * nv - 1 - q];
        if (down) {
            for (int r = t; r < m; r += TAIL_WG) x[r] = res[r] = 0.f;
        } else {
            const float *xc = x;   // the level below is done: interpolate from it
            m = uni(rows[2 * (2 * nv - 1 - q) + 1]);
            x -= 2 * tail_range<float>(m);
            for (int r0 = wv * 64; r0 < m; r0 += TAIL_WG) {
                const int r = r0 + lane;
                if (r < m) x[r] -= slice_row(L.pptr, L.plen, L.pcol, L.pval, r0 >> 6, lane, xc, 0.f);
            }
            __syncthreads();
            for (int r = t; r < m / 4; r += TAIL_WG) split4(reinterpret_cast<const float4 *>(x)[r], xs[r]);
        }
        __syncthreads();
        const float *b = x + tail_range<float>(m);
        for (int a = 0; a < (down ? n_pre : n_post); ++a) bsr16_visit(L, lsched + L.sched, b, x, xs, down ? rf : 0);
        if (!down) continue;
        for (int r0 = wv * 64; r0 < m; r0 += TAIL_WG) {
            const int r = r0 + lane;
            if (r < m) res[r] = slice_row(L.sptr, L.slen, L.scol, L.sval, r0 >> 6, lane, x, -b[r]);
        }
        __syncthreads();
        const int mc = uni(rows[2 * (q + 1) + 1]);
        float *xn = x + 2 * tail_range<float>(m), *bn = xn + tail_range<float>(mc);
        const float rs = (float)L.r_scale;
        for (int I0 = wv * 64; I0 < mc; I0 += TAIL_WG) {
            const int I = I0 + lane;
            if (I >= mc) continue;
            float v = 0.f;
            if (L.agg_k > 0) {
                for (int u = 0; u < L.agg_k; ++u) v += res[I * L.agg_k + u];
            } else {
                v = slice_row(L.tptr, L.tlen, L.tcol, L.tval, I0 >> 6, lane, res, v);
            }
            bn[I] = v * rs;
        }
        __syncthreads();
        x = xn;
        m = mc;
        if (q + 1 == nv) {
            tail_direct<float>(tab[nv], 0, min((int)tab[nv].n_active, m), m, bn, x);
            __syncthreads();
        }
    }
    auto gx = (__attribute__((address_space(1))) float *)static_cast<float *>(tab[0].xb);
    for (int r = t; r < m; r += TAIL_WG) {
        if (x64) x64[r] = add ? x64[r] + (double)x[r] : (double)x[r];
        else gx[r] = x[r];
    }
}

}  // namespace

// Rounds of a level's schedule.
int tail16_rounds(const Level &L) {
    int r = 0;
    for (int k = 0; k < L.chi; ++k) r += (int)((L.cblk_ptr[k + 1] - L.cblk_ptr[k] + NW - 1) / NW);
    return r * L.depth;
}

// Words of a level's schedule with its padding.
int64_t tail16_schedule_words(const Level &L) { return (int64_t)(tail16_rounds(L) + 2 * SCHED_PAD) * NW * 8; }

// The schedule of one level for the wavefronts of a workgroup; zero: byte offset
// of the block of zeros from the covered levels' vector of BF16 pairs.
void tail16_schedule(const Level &L, uint32_t zero, std::vector<int32_t> &out) {
    auto idle_round = [&](int w0, uint32_t flags) {
        for (int w = w0; w < NW; ++w)
            for (int k = 0; k < 8; ++k) out.push_back(k ? 0 : (int32_t)(flags | S_IDLE));
    };
    for (int q = 0; q < SCHED_PAD; ++q) idle_round(0, 0);
    for (int s = 0; s < L.depth * L.chi; ++s) {
        const int ell = s / L.chi, k = s % L.chi;
        const int64_t q1 = L.cblk_ptr[k + 1];
        for (int64_t q0 = L.cblk_ptr[k]; q0 < q1; q0 += NW) {
            const uint32_t flags = (q0 == L.cblk_ptr[k] ? S_FIRST : 0) | (q0 + NW >= q1 ? S_LAST : 0);
            for (int64_t q = q0; q < std::min(q0 + NW, q1); ++q) {
                const int32_t *m = &L.h_bmeta[8 * q];
                const bool more = m[2] - m[1] > META_COLS;
                out.push_back((int32_t)((uint32_t)(ell * L.B + m[0]) * 512u | flags | (more ? S_LONG : 0)));
                out.push_back((int32_t)(q * ROW16 * 2));
                out.push_back(m[0] * 64);
                for (int u = 0; u < META_COLS; ++u) out.push_back(m[3 + u] < 0 ? (int32_t)zero : m[3 + u] * 64);
            }
            idle_round((int)(std::min(q0 + NW, q1) - q0), flags);
        }
    }
    for (int q = 0; q < SCHED_PAD; ++q) idle_round(0, 0);
}

// The tail's copy of a level's A (elements), packed into out when given.
int64_t tail16_pack(Ctx &c, const Level &L, unsigned short *out) {
    const int64_t rows = L.cblk_ptr.back();
    if (out && rows > 0) {
        hipLaunchKernelGGL(k_pack_tail16, dim3((unsigned)rows), dim3(64), 0, c.stream, L.bmeta.get(), L.a16.get(), out);
        CS_LAUNCH_CHECK();
    }
    return rows * ROW16;
}

void tail16_prepare(int64_t lds) { allow_lds(reinterpret_cast<const void *>(&k_tail_bsr16), lds); }

void tail16_launch(Ctx &c, hipEvent_t ev0, hipEvent_t ev1, const double *b64, double *x64, bool add) {
    hipExtLaunchKernelGGL(k_tail_bsr16, dim3(8 * (1 + TAIL_HELPERS)), dim3(TAIL_WG), (unsigned)c.tail_lds, c.stream, ev0, ev1, 0,
                          (const TailLevel *)c.tail_tab.get(), (int)c.lv.size() - c.tail_from,
                          (const int32_t *)c.tail_sys.get(), c.opt.n_pre, c.opt.n_post, c.opt.order == CS_RF ? 1 : 0,
                          c.tail_alt, c.tail_zero, (const int32_t *)c.tail_sched.get(),
                          (int)c.tail_sched_host.size(), b64, x64, add ? 1 : 0);
    CS_LAUNCH_CHECK();
}

}  // namespace cs
