// Device functions shared by the setup's normal-equation kernels.
#pragma once

#include "cs_internal.h"

namespace cs {
namespace {

constexpr int WG = 256;
constexpr int MAXNB = 16;
constexpr double PIVOT_TOL = 1e-13;
typedef double d4_t __attribute__((ext_vector_type(4)));

__device__ inline int bsearch_i32(const int32_t *a, int lo, int hi, int32_t key) {
    // index of key in the sorted range a[lo, hi), or -1
    while (lo < hi) {
        int mid = (lo + hi) >> 1;
        int32_t v = a[mid];
        if (v == key) return mid;
        if (v < key) lo = mid + 1;
        else hi = mid;
    }
    return -1;
}

// Lambda~ (G + tau I) = H for one block (G, H: nb x nb in LDS, row-major), by
// the whole workgroup, tau = ridge tr(G) / nb (ridge = 0: the plain normal
// equations; ridge > 0: the Tikhonov-regularised fit).  Lc and V are LDS
// scratch of MAXNB^2 doubles.  Writes Lambda~ to out and, from thread 0,
// whether the matrix was (numerically) singular to *singular.
__device__ void normal_solve(const double *G, const double *H, double *Lc, double *V, int nb,
                             double *__restrict__ out, int32_t *__restrict__ singular, double ridge) {
    const int t = threadIdx.x;
    const int nb2 = nb * nb;
    double trace = 0.0;
    for (int q = 0; q < nb; ++q) trace += G[q * nb + q];
    const double tau = ridge > 0.0 ? ridge * trace / nb : 0.0;
    // Lambda~ G = H.  Regular G: Gauss-Jordan inverse of [G | I] (G is SPD:
    // no pivoting; the pivots are the Cholesky pivots squared, with the same
    // cut-off), one thread per entry, two barriers per step.  A pivot below
    // PIVOT_TOL max diag(G) marks G as (numerically) singular: then the
    // minimum-norm solution through a parallel cyclic Jacobi eigen-decomposition.
    __shared__ double Aug[MAXNB * 2 * MAXNB];
    const int w2 = 2 * nb;
    double dmax = 0.0;
    for (int q = 0; q < nb; ++q) dmax = fmax(dmax, G[q * nb + q] + tau);
    bool bad = !(dmax > 0.0);
    for (int e = t; e < nb * w2; e += WG) {
        const int r = e / w2, c = e % w2;
        Aug[e] = c < nb ? G[r * nb + c] + (r == c ? tau : 0.0) : (c - nb == r ? 1.0 : 0.0);
    }
    __syncthreads();
    constexpr int PER = (MAXNB * 2 * MAXNB + WG - 1) / WG;
    for (int q = 0; q < nb && !bad; ++q) {
        const double piv = Aug[q * w2 + q];
        if (!(piv > PIVOT_TOL * dmax)) {   // same value in every thread: uniform
            bad = true;
            break;
        }
        double f[PER], g[PER];
#pragma unroll
        for (int k2 = 0; k2 < PER; ++k2) {
            const int e = t + k2 * WG;
            if (e < nb * w2) {
                f[k2] = Aug[(e / w2) * w2 + q];
                g[k2] = Aug[q * w2 + e % w2];
            }
        }
        __syncthreads();
#pragma unroll
        for (int k2 = 0; k2 < PER; ++k2) {
            const int e = t + k2 * WG;
            if (e < nb * w2) Aug[e] = (e / w2 == q) ? g[k2] / piv : Aug[e] - f[k2] * g[k2] / piv;
        }
        __syncthreads();
    }
    if (t == 0) *singular = bad ? 1 : 0;
    if (!bad) {
        if (t < nb2) {
            const int r = t / nb, c = t % nb;
            double acc = 0.0;
            for (int u = 0; u < nb; ++u) acc += H[r * nb + u] * Aug[u * w2 + nb + c];
            out[t] = acc;
        }
        return;
    }
    // ---- (near-)singular G: Lambda~ = H V diag(1/ev, ev kept) V^T
    const int m = nb + (nb & 1);   // even order for the round-robin pairing (zero padding)
    __shared__ int pp_s[MAXNB / 2], pq_s[MAXNB / 2], pair_of[MAXNB], side_of[MAXNB];
    __shared__ double rc_s[MAXNB / 2], rs_s[MAXNB / 2], off_s[WG], dia_s[WG];
    for (int e = t; e < m * m; e += WG) {
        const int r = e / m, c = e % m;
        Lc[e] = (r < nb && c < nb) ? G[r * nb + c] + (r == c ? tau : 0.0) : 0.0;
        V[e] = r == c ? 1.0 : 0.0;
    }
    __syncthreads();
    for (int sweep = 0; sweep < 40; ++sweep) {
        double off = 0.0, dia = 0.0;
        for (int e = t; e < m * m; e += WG) {
            const double v = Lc[e];
            if (e / m == e % m) dia += v * v;
            else off += v * v;
        }
        off_s[t] = off;
        dia_s[t] = dia;
        __syncthreads();
        for (int h = WG / 2; h > 0; h >>= 1) {
            if (t < h) {
                off_s[t] += off_s[t + h];
                dia_s[t] += dia_s[t + h];
            }
            __syncthreads();
        }
        const double offt = off_s[0], diat = dia_s[0];
        __syncthreads();
        if (offt <= 1e-30 * diat || offt == 0.0) break;   // uniform
        for (int k = 0; k < m - 1; ++k) {
            // circle-method pairing: (m-1, k) and ((k+j) mod (m-1), (k-j) mod (m-1))
            if (t < m / 2) {
                int a1, b1;
                if (t == 0) {
                    a1 = m - 1;
                    b1 = k;
                } else {
                    a1 = (k + t) % (m - 1);
                    b1 = (k - t + (m - 1)) % (m - 1);
                }
                const int pp = min(a1, b1), qq = max(a1, b1);
                pp_s[t] = pp;
                pq_s[t] = qq;
                pair_of[pp] = t;
                side_of[pp] = 0;
                pair_of[qq] = t;
                side_of[qq] = 1;
                const double apq = Lc[pp * m + qq];
                double c = 1.0, sn = 0.0;
                if (apq != 0.0) {
                    const double tau = (Lc[qq * m + qq] - Lc[pp * m + pp]) / (2.0 * apq);
                    const double tt = (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
                    c = 1.0 / sqrt(1.0 + tt * tt);
                    sn = tt * c;
                }
                rc_s[t] = c;
                rs_s[t] = sn;
            }
            __syncthreads();
            // rows: Lc <- J^T Lc
            double nv[(MAXNB * MAXNB + WG - 1) / WG];
            for (int e = t, k2 = 0; e < m * m; e += WG, ++k2) {
                const int r = e / m, c2 = e % m, pr = pair_of[r];
                const double c = rc_s[pr], sn = rs_s[pr];
                const double vp = Lc[pp_s[pr] * m + c2], vq = Lc[pq_s[pr] * m + c2];
                nv[k2] = side_of[r] == 0 ? c * vp - sn * vq : sn * vp + c * vq;
            }
            __syncthreads();
            for (int e = t, k2 = 0; e < m * m; e += WG, ++k2) Lc[e] = nv[k2];
            __syncthreads();
            // columns: Lc <- Lc J, V <- V J
            double nw[(MAXNB * MAXNB + WG - 1) / WG];
            for (int e = t, k2 = 0; e < m * m; e += WG, ++k2) {
                const int r = e / m, c2 = e % m, pr = pair_of[c2];
                const double c = rc_s[pr], sn = rs_s[pr];
                const int p0 = pp_s[pr], q0 = pq_s[pr];
                const double lp = Lc[r * m + p0], lq = Lc[r * m + q0];
                const double vp = V[r * m + p0], vq = V[r * m + q0];
                nv[k2] = side_of[c2] == 0 ? c * lp - sn * lq : sn * lp + c * lq;
                nw[k2] = side_of[c2] == 0 ? c * vp - sn * vq : sn * vp + c * vq;
            }
            __syncthreads();
            for (int e = t, k2 = 0; e < m * m; e += WG, ++k2) {
                Lc[e] = nv[k2];
                V[e] = nw[k2];
            }
            __syncthreads();
        }
    }
    double emax = 0.0;
    for (int q = 0; q < nb; ++q) emax = fmax(emax, fabs(Lc[q * m + q]));
    // HV[r][a] = sum_u H[r][u] V[u][a] (into Aug)
    if (t < nb2) {
        const int r = t / nb, a2 = t % nb;
        double acc = 0.0;
        for (int u = 0; u < nb; ++u) acc += H[r * nb + u] * V[u * m + a2];
        Aug[t] = acc;
    }
    __syncthreads();
    if (t < nb2) {
        const int r = t / nb, c = t % nb;
        double acc = 0.0;
        for (int a2 = 0; a2 < nb; ++a2) {
            const double ev = Lc[a2 * m + a2];
            if (ev > PIVOT_TOL * emax) acc += Aug[r * nb + a2] * V[c * m + a2] / ev;
        }
        out[t] = acc;
    }
}

}  // namespace

// Fused fit step of a level of 8x8 blocks (fit8.hip): per list row M_i = sum_j
// A~_ij E_j, the normal equations, Lambda~_i and, with nval, the updated row of
// E on pattern(M_i).  Every list row has to store its diagonal block in A~.
struct Fit8 {
    int nl = 0;                           // list rows
    const int32_t *list = nullptr, *abptr = nullptr, *abcol = nullptr;
    const double *abval = nullptr;        // A~ blocks
    const int32_t *eptr = nullptr, *ecol = nullptr;
    const double *eval = nullptr;
    const int32_t *mptr = nullptr, *mcol = nullptr;   // pattern(M), by list position
    double *lamt = nullptr;               // [B][8][8]
    int32_t *sing = nullptr, *redo = nullptr;   // [nl]; count and list of rows for the minimum-norm pass
    double ridge = 0.0;
    bool identity = false;                // E = I
    const int32_t *nptr = nullptr;        // new E (null: not wanted)
    int32_t *ncol = nullptr;
    double *nval = nullptr;
    int32_t *rec = nullptr;               // scratch: fit8_rec_ints ints
    uint16_t *pos = nullptr;              // scratch: nl * pcap
    int maxk = 0, pcap = 0, maxdeg = 0;   // longest row of M; bound of a row's neighbours' blocks; most neighbours
};
bool fit8_fits(const Fit8 &f);
size_t fit8_rec_ints(const Fit8 &f);
void launch_fit8(hipStream_t s, const Fit8 &f);

}  // namespace cs
