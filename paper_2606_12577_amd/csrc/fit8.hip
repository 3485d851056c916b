// Fused fit step for 8x8 blocks (gfx950, wave64): Alg. 2's least-squares step
// and residual update of one block row in one workgroup, the row of M = A~ E in
// LDS.  See Fit8 (fit_device.h).
//
// What the step has to move is E (read by a row's neighbours, which run on the
// same XCD and partly find it in the L2) and the new E; M, at the last step of a
// depth-4 cascade on a 7-point stencil twice the size of E, was written once and
// read back by the normal equations and by the update.  Row product, normal
// equations and update as kernels of their own (rows that do not fit still take
// them) were 15 of the 22 ms of kernel time of the 96^3 setup; the four steps of
// the finest level (110,592 rows) now take 0.44, 1.2, 2.5 and 4.2 ms, setup
// 24.6 -> 17.0 ms.  The updates run at the memory rate (3.6 GB written by step 3 in
// 0.9 ms); the product is bound by latency with the two workgroups per CU that the
// LDS allows (step 4: 2.5 ms against 0.65 of FP64 FMAs and 1.7 of loads from beyond
// the L2).
//
//   product    scatter form: the blocks of E_j of one neighbour after the other
//              are multiplied by A~_ij, which sits in scalar registers, and added
//              into the columns of M that they belong to (a barrier per neighbour).
//              A gather over M's blocks would leave half of the lanes without a
//              match, and A~ from LDS would need twice the LDS bandwidth there is.
//              Entry by entry the sum runs over the neighbours, then the inner
//              index, as in the row product kernel.  E = I: M is the row of A~.
//   Gram       FP64 MFMA 16x16x4, the row's columns in two halves: operand rows
//              0-7 hold the first half's columns of M (or E_i), rows 8-15 the
//              second's, and the two diagonal 8x8 blocks of the result are added.
//   solve      one wavefront, [G + tau I | I] in registers; rows that meet a small
//              pivot are left to a second launch with the minimum-norm solve.
//   update     E_new = E_i - Lambda~_i M on the matrix cores, from LDS.
//
// M's rows are padded to 4 mod 32 doubles, so that eight rows of four doubles
// fall into 64 different banks.
#include <algorithm>

#include "fit_device.h"

namespace cs {
namespace {

constexpr int64_t FIT8_LDS = 80 * 1024;   // two workgroups per CU

__host__ __device__ inline int fit8_stride(int maxk) { return (8 * maxk + 31) / 32 * 32 + 4; }

int64_t fit8_bytes(const Fit8 &f, int waves) {
    return (int64_t)sizeof(double) * (8 * fit8_stride(f.maxk) + 128 * waves + 192) +
           (int64_t)sizeof(int32_t) * f.maxk + (int64_t)sizeof(uint16_t) * (f.pcap + 3) / 4 * 4;
}

// Per list row, laid out for the step's kernel, which then waits for one load
// instead of a chain of five (list, pointers, neighbours, their E rows, their
// columns): a record of fit8_rec(maxdeg) ints
//   {i, neighbours, k, blocks of E_i, first A~ block, first block of E_i, first of
//    the new E_i, position list's offset of E_i's blocks}, then per neighbour
//   {first block of E_j, offset of its blocks in the position list}, and the
//    list's length as a last offset;
// and the position list: where in row M_i every block of the neighbours' E rows
// goes.  A wavefront per row; with ncol the row's columns are copied there too.
constexpr int REC_HEAD = 8;
__host__ __device__ inline int fit8_rec(int maxdeg) { return REC_HEAD + 2 * (maxdeg + 1); }

__global__ __launch_bounds__(WG) void k_fit8_rows(int nl, const int32_t *__restrict__ list,
                                                  const int32_t *__restrict__ abptr, const int32_t *__restrict__ abcol,
                                                  const int32_t *__restrict__ eptr, const int32_t *__restrict__ ecol,
                                                  const int32_t *__restrict__ mptr, const int32_t *__restrict__ mcol,
                                                  const int32_t *__restrict__ nptr, int32_t *__restrict__ ncol,
                                                  int maxk, int pcap, int maxdeg, int32_t *__restrict__ rec,
                                                  uint16_t *__restrict__ pos) {
    extern __shared__ __align__(16) int32_t rows_lds[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int li = (int)xcd_tile(blockIdx.x, gridDim.x) * (WG / 64) + wave;
    const bool live = li < nl;
    int32_t *const mc = rows_lds + wave * (maxk + 2 * (maxdeg + 1)), *const elo = mc + maxk, *const eoff = elo + maxdeg + 1;
    int deg = 0, k = 0, tot = 0;
    if (live) {
        const int i = list[li], alo = abptr[i], mlo = mptr[li];
        deg = abptr[i + 1] - alo;
        k = mptr[li + 1] - mlo;
        const int nlo = nptr ? nptr[i] : 0;
        int32_t *const r = rec + (int64_t)li * fit8_rec(maxdeg);
        for (int p = lane; p < k; p += 64) {
            const int32_t c = mcol[mlo + p];
            mc[p] = c;
            if (ncol) ncol[nlo + p] = c;
        }
        int len = 0, e0 = 0, j = -1;
        if (lane < deg) {   // deg <= 64
            j = abcol[alo + lane];
            e0 = eptr[j];
            len = eptr[j + 1] - e0;
        }
        int inc = len;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(inc, o, 64);
            if (lane >= o) inc += y;
        }
        tot = __shfl(inc, 63, 64);
        if (lane < deg) {
            elo[lane] = e0;
            eoff[lane + 1] = inc;
            r[REC_HEAD + 2 * lane] = e0;
            r[REC_HEAD + 2 * lane + 1] = inc - len;
            if (j == i) {
                r[3] = len;
                r[5] = e0;
                r[7] = inc - len;
            }
        }
        if (lane == 0) {
            eoff[0] = 0;
            r[0] = i;
            r[1] = deg;
            r[2] = k;
            r[4] = alo;
            r[6] = nlo;
            r[REC_HEAD + 2 * deg + 1] = tot;
        }
    }
    __syncthreads();
    for (int e = lane; e < tot; e += 64) {
        int a = 0, b = deg;   // eoff[a] <= e < eoff[b]
        while (b - a > 1) {
            const int m = (a + b) >> 1;
            if (eoff[m] <= e) a = m;
            else b = m;
        }
        pos[(int64_t)li * pcap + e] = (uint16_t)bsearch_i32(mc, 0, k, ecol[elo[a] + (e - eoff[a])]);
    }
}

// WGS threads per row in two groups; a thread takes two columns of a block of
// E_j and its group's four rows of M.
template <int WGS, bool REDO>
__global__ __launch_bounds__(WGS, REDO ? 2 : 4) void k_fit8(const int32_t *__restrict__ rec,
                                              const uint16_t *__restrict__ gpos, const double *__restrict__ abval,
                                              const double *__restrict__ eval, double *__restrict__ lamt,
                                              int32_t *__restrict__ sing, int32_t *__restrict__ redo, double ridge,
                                              double *__restrict__ nval, int nl, int ahead, int identity, int maxk,
                                              int pcap, int maxdeg) {
    constexpr int NW = WGS / 64, TW = WGS / 2, RPT = 4;
    extern __shared__ __align__(16) double lds[];
    const int sc = fit8_stride(maxk);
    double *const M = lds, *const part = M + 8 * sc, *const GH = part + 128 * NW, *const Lm = GH + 128;
    int32_t *const inv = reinterpret_cast<int32_t *>(Lm + 64);
    uint16_t *const pos = reinterpret_cast<uint16_t *>(inv + maxk);
    __shared__ int32_t s_bad;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int r16 = lane & 15, kq = lane >> 4, half = r16 >> 3, rr = r16 & 7;
    const int nrows = REDO ? redo[0] : 1;
    for (int idx = REDO ? (int)blockIdx.x : 0; idx < nrows; idx += REDO ? (int)gridDim.x : 1) {
        const int li = REDO ? redo[1 + idx] : (int)xcd_tile(blockIdx.x, gridDim.x);
        const int32_t *const r = rec + (int64_t)li * fit8_rec(maxdeg);   // uniform: scalar loads
        const int i = r[0], deg = r[1], k = r[2], ek = r[3], alo = r[4], ei = r[5], nlo = r[6], epos = r[7];
        const int tot = r[REC_HEAD + 2 * deg + 1];
        // the row of A~ comes into the L2 meanwhile: the scalar loads of the product
        // would wait for its lines one after the other (step 4 of the 96^3 level 4.2
        // ms; without this, and eight rows per thread in three batches, 6.4)
        double2 warm = make_double2(0.0, 0.0);
        for (int e = t; e < deg * 32; e += WGS) warm = reinterpret_cast<const double2 *>(abval)[(int64_t)alo * 32 + e];
        for (int e = t; e < tot; e += WGS) pos[e] = gpos[(int64_t)li * pcap + e];
        for (int p = t; p < k; p += WGS) inv[p] = -1;
        for (int c = t; c < 4 * k; c += WGS)
#pragma unroll
            for (int q = 0; q < 8; ++q) *reinterpret_cast<double2 *>(M + q * sc + 2 * c) = make_double2(0.0, 0.0);
        asm volatile("" ::"v"(warm.x), "v"(warm.y));
        __syncthreads();
        for (int e = t; e < ek; e += WGS) inv[pos[epos + e]] = e;
        // product
        auto load = [&](int e0, int w, double2 (&d)[8]) {
            const double *ev = eval + ((int64_t)e0 + (w >> 2)) * 64 + 2 * (w & 3);
#pragma unroll
            for (int u = 0; u < 8; ++u) d[u] = *reinterpret_cast<const double2 *>(ev + u * 8);
        };
        const int tt = t % TW, rh = __builtin_amdgcn_readfirstlane(t / TW);
        auto accumulate = [&](int jj, int o, int w, const double2 (&d)[8]) {
            const double *a = abval + ((int64_t)alo + jj) * 64 + rh * RPT * 8;   // uniform: scalar loads
            double *mp = M + rh * RPT * sc + pos[o + (w >> 2)] * 8 + 2 * (w & 3);
#pragma unroll
            for (int q = 0; q < RPT; ++q) {
                double2 m = *reinterpret_cast<double2 *>(mp + q * sc);
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    m.x += a[q * 8 + u] * d[u].x;
                    m.y += a[q * 8 + u] * d[u].y;
                }
                *reinterpret_cast<double2 *>(mp + q * sc) = m;
            }
        };
        // the row that follows on this XCD: its record, positions and (below) A~ come
        // into the L2 while this one is worked on
        const int ln = li + ahead;
        const bool touch = !REDO && ln < nl;
        int32_t t_rec = 0;
        uint16_t t_pos = 0;
        if (touch) {
            if (t < fit8_rec(maxdeg)) t_rec = rec[(int64_t)ln * fit8_rec(maxdeg) + t];
            if (t * 64 < pcap) t_pos = gpos[(int64_t)ln * pcap + t * 64];
        }
        // every thread loads (the last block again where it has none), so that the
        // loads in flight over a neighbour are known and only the older ones waited for
        const int32_t *const nbr = r + REC_HEAD;   // {first block, offset} per neighbour
        if (identity) {   // E = I: M_i is the row of A~
            for (int e = t; e < deg * 64; e += WGS)
                M[((e >> 3) & 7) * sc + pos[e >> 6] * 8 + (e & 7)] = abval[(int64_t)alo * 64 + e];
            __syncthreads();
        } else {
            // the next neighbour in flight, in two register buffers used in turn (a
            // copy between buffers would wait for its loads)
            double2 d0[8], d1[8];
            auto request = [&](int jj, double2 (&d)[8]) {
                const int j = min(jj, deg - 1);
                load(nbr[2 * j], min(tt, 4 * (nbr[2 * j + 3] - nbr[2 * j + 1]) - 1), d);
            };
            auto neighbour = [&](int jj, const double2 (&d)[8], double2 (&ahead)[8]) {
                request(jj + 1, ahead);
                const int o = nbr[2 * jj + 1], items = 4 * (nbr[2 * jj + 3] - o);
                if (tt < items) accumulate(jj, o, tt, d);
                for (int w = tt + TW; w < items; w += TW) {
                    double2 more[8];
                    load(nbr[2 * jj], w, more);
                    accumulate(jj, o, w, more);
                }
                __syncthreads();   // the next neighbour's blocks may add into the same columns
            };
            request(0, d0);
            for (int jj = 0;; jj += 2) {
                neighbour(jj, d0, d1);
                if (jj + 1 >= deg) break;
                neighbour(jj + 1, d1, d0);
                if (jj + 2 >= deg) break;
            }
        }
        double t_a = 0.0;
        if (touch) {   // t_rec of lanes 1 and 4: its neighbours and first A~ block
            const int dn = __shfl(t_rec, 1, 64), an = __shfl(t_rec, 4, 64);
            if (wave == 0 && lane < dn * 4) t_a = abval[(int64_t)an * 64 + lane * 16];
        }
        // G = M M^T, H = E_i M^T: lane group kq holds columns 2 kq and 2 kq + 1 of a block
        d4_t dg = {0.0, 0.0, 0.0, 0.0}, dh = {0.0, 0.0, 0.0, 0.0};
        {
            const int kh = (k + 1) / 2, eh = (ek + 1) / 2;
            const double *mr = M + rr * sc + 2 * kq;
            // (blocks off the end: the last one, times zero)
            auto e_block = [&](int e) {
                const int ee = e + half * eh;
                double2 v = *reinterpret_cast<const double2 *>(eval + ((int64_t)ei + min(ee, ek - 1)) * 64 + rr * 8 + 2 * kq);
                const bool ok = e < eh && ee < ek;
                v.x = ok ? v.x : 0.0;
                v.y = ok ? v.y : 0.0;
                return v;
            };
            auto h_step = [&](int e, double2 ev) {
                const double2 mv = *reinterpret_cast<const double2 *>(mr + pos[epos + min(e + half * eh, ek - 1)] * 8);
                dh = __builtin_amdgcn_mfma_f64_16x16x4f64(ev.x, mv.x, dh, 0, 0, 0);
                dh = __builtin_amdgcn_mfma_f64_16x16x4f64(ev.y, mv.y, dh, 0, 0, 0);
            };
            double2 e4[4];   // E_i's first blocks are requested before G's products
#pragma unroll
            for (int u = 0; u < 4; ++u) e4[u] = e_block(wave + u * NW);
#pragma unroll 2
            for (int p = wave; p < kh; p += NW) {
                const int pp = p + half * kh;
                double2 mv = *reinterpret_cast<const double2 *>(mr + min(pp, k - 1) * 8);
                mv.x = pp < k ? mv.x : 0.0;
                mv.y = pp < k ? mv.y : 0.0;
                dg = __builtin_amdgcn_mfma_f64_16x16x4f64(mv.x, mv.x, dg, 0, 0, 0);
                dg = __builtin_amdgcn_mfma_f64_16x16x4f64(mv.y, mv.y, dg, 0, 0, 0);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (wave + u * NW < eh) h_step(wave + u * NW, e4[u]);
            for (int e = wave + 4 * NW; e < eh; e += NW) h_step(e, e_block(e));
        }
        // result lane l, register x = D[4x + l/16][l%16]
        {
            double g0 = half ? dg[2] : dg[0], g1 = half ? dg[3] : dg[1];
            double h0 = half ? dh[2] : dh[0], h1 = half ? dh[3] : dh[1];
            g0 += __shfl_xor(g0, 8, 64);
            g1 += __shfl_xor(g1, 8, 64);
            h0 += __shfl_xor(h0, 8, 64);
            h1 += __shfl_xor(h1, 8, 64);
            if (half == 0) {
                double *pw = part + wave * 128 + kq * 8 + rr;
                pw[0] = g0;
                pw[32] = g1;
                pw[64] = h0;
                pw[96] = h1;
            }
        }
        __syncthreads();
        for (int e = t; e < 128; e += WGS) {
            double v = part[e];
#pragma unroll
            for (int w = 1; w < NW; ++w) v += part[w * 128 + e];
            GH[e] = v;
        }
        __syncthreads();
        if constexpr (REDO) {
            __shared__ double Lc[MAXNB * MAXNB], V[MAXNB * MAXNB];
            normal_solve(GH, GH + 64, Lc, V, 8, lamt + (int64_t)i * 64, sing + li, ridge);
            __syncthreads();
            if (t < 64) Lm[t] = lamt[(int64_t)i * 64 + t];
            if (t == 0) s_bad = 0;
        } else if (wave == 0) {
            // Gauss-Jordan on [G + tau I | I]: entry lane + 64 m of the 8 x 16 array
            // in register m (k_gram_mfma8's elimination, cut-off and products)
            const double *G = GH, *H = GH + 64;
            double trace = 0.0, dmax = 0.0;
#pragma unroll
            for (int q = 0; q < 8; ++q) trace += G[q * 9];
            const double tau = ridge > 0.0 ? ridge * trace / 8 : 0.0;
#pragma unroll
            for (int q = 0; q < 8; ++q) dmax = fmax(dmax, G[q * 9] + tau);
            bool bad = !(dmax > 0.0);
            double v[2];
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const int r = kq + 4 * m;
                v[m] = r16 < 8 ? G[r * 8 + r16] + (r == r16 ? tau : 0.0) : (r16 - 8 == r ? 1.0 : 0.0);
            }
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const double piv = __shfl(v[q >> 2], (q & 3) * 16 + q, 64);
                const double g = __shfl(v[q >> 2], (q & 3) * 16 + r16, 64);
                const double f0 = __shfl(v[0], (lane & 48) + q, 64), f1 = __shfl(v[1], (lane & 48) + q, 64);
                if (!(piv > PIVOT_TOL * dmax)) bad = true;
                const double n0 = kq == q ? g / piv : v[0] - f0 * g / piv;
                const double n1 = kq + 4 == q ? g / piv : v[1] - f1 * g / piv;
                if (!bad) {
                    v[0] = n0;
                    v[1] = n1;
                }
            }
            double acc = 0.0;
#pragma unroll
            for (int u = 0; u < 8; ++u)
                acc += H[(lane >> 3) * 8 + u] * __shfl(v[u >> 2], (u & 3) * 16 + 8 + (lane & 7), 64);
            if (!bad) {
                lamt[(int64_t)i * 64 + lane] = acc;
                Lm[lane] = acc;
            }
            if (lane == 0) {
                sing[li] = bad ? 1 : 0;
                if (bad) redo[1 + atomicAdd(redo, 1)] = li;
                s_bad = bad ? 1 : 0;
            }
        }
        asm volatile("" ::"v"(t_rec), "v"((uint32_t)t_pos), "v"(t_a));
        __syncthreads();
        if (nval && !s_bad) {   // uniform
            // Lambda~ M on the matrix cores, two blocks (16 columns) per pair of
            // MFMAs; operand rows 8-15 are zero, lane l receives rows l/16 and
            // 4 + l/16 of column l%16.  UP pairs at a time: their E rows are requested
            // first.
            constexpr int UP = 4;
            const double a0 = half ? 0.0 : Lm[rr * 8 + kq], a1 = half ? 0.0 : Lm[rr * 8 + 4 + kq];
            const int pairs = (k + 1) / 2;
            for (int g0 = wave; g0 < pairs; g0 += NW * UP) {
                double v0[UP], v1[UP];
                int pb[UP], ok[UP];
#pragma unroll
                for (int u = 0; u < UP; ++u) {
                    const int p = 2 * (g0 + u * NW) + half;
                    ok[u] = p < k;
                    pb[u] = min(p, k - 1);
                    const int q = inv[pb[u]];
                    const double *eo = eval + ((int64_t)ei + max(q, 0)) * 64 + kq * 8 + rr;
                    v0[u] = eo[0];
                    v1[u] = eo[32];
                    v0[u] = q >= 0 ? v0[u] : 0.0;
                    v1[u] = q >= 0 ? v1[u] : 0.0;
                }
#pragma unroll
                for (int u = 0; u < UP; ++u) {
                    const double *mp = M + kq * sc + pb[u] * 8 + rr;
                    d4_t d = {0.0, 0.0, 0.0, 0.0};
                    d = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, mp[0], d, 0, 0, 0);
                    d = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, mp[4 * sc], d, 0, 0, 0);
                    if (ok[u]) {
                        double *no = nval + ((int64_t)nlo + pb[u]) * 64 + kq * 8 + rr;
                        no[0] = v0[u] - d[0];
                        no[32] = v1[u] - d[1];
                    }
                }
            }
        }
        if constexpr (REDO) __syncthreads();   // the buffers are rewritten by the next row
    }
}

template <int WGS, bool REDO>
void go(hipStream_t s, const Fit8 &f) {
    const int64_t bytes = fit8_bytes(f, WGS / 64);
    allow_lds(reinterpret_cast<const void *>(&k_fit8<WGS, REDO>), FIT8_LDS);
    const unsigned grid = REDO ? 256u : (unsigned)f.nl;
    // rows in flight on an XCD (32 CUs): LDS, five wavefronts per SIMD
    const int ahead = 32 * (int)std::max<int64_t>(std::min<int64_t>(2 * FIT8_LDS / bytes, 20 * 64 / WGS), 1);
    hipLaunchKernelGGL((k_fit8<WGS, REDO>), dim3(grid), dim3(WGS), (unsigned)bytes, s, f.rec, f.pos, f.abval,
                       f.eval, f.lamt, f.sing, f.redo, f.ridge, f.nval, f.nl, ahead, f.identity ? 1 : 0, f.maxk, f.pcap, f.maxdeg);
    CS_LAUNCH_CHECK();
}

}  // namespace

size_t fit8_rec_ints(const Fit8 &f) { return (size_t)f.nl * fit8_rec(f.maxdeg); }

// Rows fit when two workgroups' LDS do: up to 150 blocks in a row of M (a
// depth-4 cascade on a 7-point stencil of 2x2x2 blocks has 129, depth 2 on a
// 27-point stencil 125).
bool fit8_fits(const Fit8 &f) {
    return f.maxdeg <= 64 && f.pcap <= 4096 && fit8_bytes(f, 8) <= FIT8_LDS;
}

void launch_fit8(hipStream_t s, const Fit8 &f) {
    if (f.nl <= 0) return;
    const size_t lds = (size_t)(WG / 64) * (f.maxk + 2 * (f.maxdeg + 1)) * sizeof(int32_t);
    hipLaunchKernelGGL(k_fit8_rows, dim3((unsigned)ceil_div(f.nl, WG / 64)), dim3(WG), (unsigned)lds, s, f.nl, f.list,
                       f.abptr, f.abcol, f.eptr, f.ecol, f.mptr, f.mcol, f.nptr, f.ncol, f.maxk, f.pcap, f.maxdeg, f.rec,
                       f.pos);
    CS_LAUNCH_CHECK();
    // threads per row by the blocks of a neighbour's E row, four threads each
    const int items = 4 * (f.pcap / std::max(f.maxdeg, 1));
    if (items <= 64) go<128, false>(s, f);
    else if (items <= 128) go<256, false>(s, f);
    else go<512, false>(s, f);
    go<256, true>(s, f);
}

}  // namespace cs
