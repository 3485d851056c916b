// Block-smoother network, row-tile path (gfx950, wave64): hidden and output
// widths of at most 128.  Everything after the first product is local to a
// tile of rows, so a training step is four launches and a prediction two:
//   k_l1     part_z = X W1^T over slice z of the inputs            (GEMM)
//   k_rows   sum of the slices, both hidden layers, the output, and in
//            training the loss and the three layers' deltas          (row tiles)
//   k_wgrad  partial weight gradients delta^T input over row slices  (GEMM)
//   k_adam_rows / k_grad_rows  sum of the partials, Adam update
// All products on the FP32 matrix cores (16x16x4: lane l supplies A[l%16][k]
// and B[k][l%16] for its k group l/16 and receives D[4(l/16) + r][l%16]).
// k runs in groups of 16: lane group q = l/16 holds k = 4q .. 4q + 3 (one
// 16-byte load) and step j multiplies k = 4q + j, so a sum over k is taken in
// that order.
#include <algorithm>

#include "mlp_internal.h"

namespace cs {
namespace {

constexpr int WG = 256;
constexpr int NP = 128;        // padded width of the hidden and output layers
constexpr int BM = 64, BK = 16;
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x4 mfma(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 ld4(const float *p) { return *reinterpret_cast<const f32x4 *>(p); }
__device__ __forceinline__ void st4(float *p, f32x4 v) { *reinterpret_cast<f32x4 *>(p) = v; }
__device__ __forceinline__ float sigmoid(float z) { return 1.0f / (1.0f + expf(-z)); }

// part[z][m][0..NP) = sum over the inputs [z kchunk, (z + 1) kchunk) of
// X[row(m)][k] W1[n][k], rows of W1 beyond `width` taken as zero.  A tile of 64
// rows by the whole width per workgroup, 32 x 64 per wavefront (8 MFMA tiles):
// a 16-deep slice of both operands sits in LDS (rows padded to 20 words: the
// 16-byte reads of 16 rows hit 64 different banks) while the next one is in
// flight in registers.  Bound by the matrix cores: 32 MFMAs of 32 cycles per
// slice and wavefront against 6 LDS reads.  110,592 x 1464 x 128: 444 us, 93
// TFLOP/s (scalar loads into 64 x 64 tiles: 1,782 us with the second layer).
__global__ __launch_bounds__(WG) void k_l1(int M, int K, const float *__restrict__ X, const int32_t *__restrict__ rows,
                                           const float *__restrict__ W1, int width, int kchunk,
                                           float *__restrict__ part) {
    __shared__ __align__(16) float As[2][BM][BK + 4], Bs[2][NP][BK + 4];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6, r16 = lane & 15, q = lane >> 4;
    const int wm = (w >> 1) * 32, wn = (w & 1) * 64;
    const int m0 = blockIdx.x * BM;
    const int kb = blockIdx.y * kchunk, ke = min(K, kb + kchunk);
    const int lr = t >> 2, lk = (t & 3) * 4;   // this thread's row and column of a slice
    const int gm = m0 + lr;
    const float *xa = X + (gm < M ? (rows ? (int64_t)rows[gm] : (int64_t)gm) : 0) * K + lk;
    const float *wb0 = W1 + (int64_t)min(lr, width - 1) * K + lk, *wb1 = W1 + (int64_t)min(lr + 64, width - 1) * K + lk;
    const bool okm = gm < M, ok0 = lr < width, ok1 = lr + 64 < width;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 acc[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int n = 0; n < 4; ++n) acc[i][n] = zero;
    auto fetch = [&](int k0, f32x4 &a, f32x4 &b0, f32x4 &b1) {   // K and kb are multiples of 4
        const bool in = k0 + lk < ke;
        a = in && okm ? ld4(xa + k0) : zero;
        b0 = in && ok0 ? ld4(wb0 + k0) : zero;
        b1 = in && ok1 ? ld4(wb1 + k0) : zero;
    };
    f32x4 ra, rb0, rb1;
    fetch(kb, ra, rb0, rb1);
    int cur = 0;
    for (int k0 = kb; k0 < ke; k0 += BK, cur ^= 1) {
        st4(&As[cur][lr][lk], ra);
        st4(&Bs[cur][lr][lk], rb0);
        st4(&Bs[cur][lr + 64][lk], rb1);
        __syncthreads();
        if (k0 + BK < ke) fetch(k0 + BK, ra, rb0, rb1);
        f32x4 a[2], b[4];
#pragma unroll
        for (int i = 0; i < 2; ++i) a[i] = ld4(&As[cur][wm + 16 * i + r16][4 * q]);
#pragma unroll
        for (int n = 0; n < 4; ++n) b[n] = ld4(&Bs[cur][wn + 16 * n + r16][4 * q]);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int n = 0; n < 4; ++n) acc[i][n] = mfma(a[i][j], b[n][j], acc[i][n]);
    }
    float *out = part + (int64_t)blockIdx.y * M * NP;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int n = 0; n < 4; ++n)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = m0 + wm + 16 * i + 4 * q + r;
                if (row < M) out[(int64_t)row * NP + wn + 16 * n + r16] = acc[i][n][r];
            }
}

enum RowMode { ROWS_PREDICT = 0, ROWS_LOSS = 1, ROWS_TRAIN = 2 };

struct RowArgs {
    int M, S, W, O;                                  // rows, slices of part, hidden and output width
    const float *part;                               // [S][M][NP]
    const float *b1, *W2, *b2, *W3, *b3, *mean, *std;
    const float *T;                                  // targets [.][O]
    const int32_t *rows;                             // row of every tile row in T (null: itself)
    float *Y;                                        // predictions [M][O]
    float *h1, *h2, *dy, *d2, *d1;                   // [M][NP], training
    float *bpart;                                    // [workgroups][3][NP] column sums of d1, d2, dy
    double *lpart;                                   // [workgroups] sums of squares
    float gscale;
};

// One tile of 16 RT rows; wavefront w of eight owns columns [16 w, 16 w + 16) of
// every layer as RT MFMA tiles, its elements (i, r) = row 16 i + 4 q + r, column
// 16 w + l%16 of all of them, so pre-activations stay in registers from the
// forward to the backward pass and only the left operand of the next product
// goes through LDS.  A wavefront's share of the weights (8 KB a product) comes
// from the L2 into registers, all of it requested before the first wait: what
// bounds a batch's 64 workgroups is the latency of a chain of dependent loads
// and barriers: 1,024 rows of training take 18.7 us, 45 us with four wavefronts
// that load each product's weights after the one before it, and the separate
// products, bias sums and loss before them took 150.  110,592 rows of prediction
// take 125 us (152 with four wavefronts; 47 at the matrix rate).  16-row tiles
// for batches, larger ones above 16,384 rows, where re-reading the weights
// costs more than it spreads.
constexpr int RW = 512;        // threads of k_rows

template <int RT, int MODE>
__global__ __launch_bounds__(RW) void k_rows(RowArgs a) {
    __shared__ __align__(16) float At[16 * RT][NP + 4];
    __shared__ double sred[RW / 64];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6, r16 = lane & 15, q = lane >> 4;
    const int m0 = blockIdx.x * 16 * RT, col = 16 * w + r16;
    struct Frag {
        f32x4 k[8];
    };
    // B fragments of V[n][k] (ld, n < N, k < K; K a multiple of 4), or of V[k][n]
    auto load_b = [&](const float *V, int ld, int N, int K) {
        Frag B;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            const int k = 16 * kk + 4 * q;
            B.k[kk] = col < N && k < K ? ld4(V + (int64_t)col * ld + k) : f32x4{0.f, 0.f, 0.f, 0.f};
        }
        return B;
    };
    auto load_bt = [&](const float *V, int ld, int N, int K) {
        Frag B;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int k = 16 * kk + 4 * q + j;
                B.k[kk][j] = col < N && k < K ? V[(int64_t)k * ld + col] : 0.f;
            }
        return B;
    };
    f32x4 acc[RT];
    // acc = At B; small tiles (batches) in four sums of 32 products each, which
    // rounds half as much as one chain of 128
    constexpr int NS = RT == 1 ? 4 : 1;
    auto product = [&](const Frag &B) {
        f32x4 part[NS][RT];
#pragma unroll
        for (int p = 0; p < NS; ++p)
#pragma unroll
            for (int i = 0; i < RT; ++i) part[p][i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            f32x4 av[RT];
#pragma unroll
            for (int i = 0; i < RT; ++i) av[i] = ld4(&At[16 * i + r16][16 * kk + 4 * q]);
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int i = 0; i < RT; ++i) part[kk % NS][i] = mfma(av[i][j], B.k[kk][j], part[kk % NS][i]);
        }
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            if constexpr (NS == 4) acc[i] = (part[0][i] + part[1][i]) + (part[2][i] + part[3][i]);
            else acc[i] = part[0][i];
        }
    };
    // every element of the tile: f(i, r, tile row, global row)
    auto each = [&](auto &&f) {
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) f(i, r, 16 * i + 4 * q + r, m0 + 16 * i + 4 * q + r);
    };
    // column sums of this tile's deltas (in acc): rows in order per lane group,
    // then the four groups
    auto bias = [&](int slot) {
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) s += acc[i][r];
        s += __shfl_xor(s, 16, 64);
        s += __shfl_xor(s, 32, 64);
        if (q == 0) a.bpart[((int64_t)blockIdx.x * 3 + slot) * NP + col] = s;
    };
    const Frag B2 = load_b(a.W2, a.W, a.W, a.W), B3 = load_b(a.W3, a.W, a.O, a.W);
    Frag T3, T2;
    if constexpr (MODE == ROWS_TRAIN) {
        T3 = load_bt(a.W3, a.W, a.W, a.O);
        T2 = load_bt(a.W2, a.W, a.W, a.W);
    }
    // The padded columns of a layer stay zero: an infinity in the row times a
    // padded zero weight is a NaN there, which the next product would spread over
    // the row.
    const bool inW = col < a.W, inO = col < a.O;
    const uint32_t keep = inW ? ~0u : 0u;
    auto pad = [&](float v) { return __uint_as_float(__float_as_uint(v) & keep); };
    const float b1 = inW ? a.b1[col] : 0.f, b2 = inW ? a.b2[col] : 0.f, b3 = inO ? a.b3[col] : 0.f;
    const float mean = inO ? a.mean[col] : 0.f, sd = inO ? a.std[col] : 1.f;
    float z1[RT][4], z2[RT][4], tt[RT][4];
    if constexpr (MODE != ROWS_PREDICT)
        each([&](int i, int r, int row, int gm) {
            tt[i][r] = 0.f;
            if (gm < a.M && inO) tt[i][r] = a.T[(a.rows ? (int64_t)a.rows[gm] : (int64_t)gm) * a.O + col];
        });
    each([&](int i, int r, int row, int gm) { z1[i][r] = 0.f; });
    for (int s0 = 0; s0 < a.S; s0 += 4) {   // slices in order, the loads of four at a time
        float pv[4][RT][4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            each([&](int i, int r, int row, int gm) {
                pv[u][i][r] = 0.f;
                if (gm < a.M && s0 + u < a.S) pv[u][i][r] = a.part[((int64_t)(s0 + u) * a.M + gm) * NP + col];
            });
#pragma unroll
        for (int u = 0; u < 4; ++u) each([&](int i, int r, int row, int gm) { z1[i][r] += pv[u][i][r]; });
    }
    each([&](int i, int r, int row, int gm) {
        const float v = z1[i][r] + b1, h = pad(v * sigmoid(v));
        z1[i][r] = v;
        At[row][col] = h;
        if constexpr (MODE == ROWS_TRAIN)
            if (gm < a.M) a.h1[(int64_t)gm * NP + col] = h;
    });
    __syncthreads();
    product(B2);
    __syncthreads();
    each([&](int i, int r, int row, int gm) {
        const float v = acc[i][r] + b2, h = pad(v * sigmoid(v));
        z2[i][r] = v;
        At[row][col] = h;
        if constexpr (MODE == ROWS_TRAIN)
            if (gm < a.M) a.h2[(int64_t)gm * NP + col] = h;
    });
    __syncthreads();
    product(B3);
    if constexpr (MODE == ROWS_PREDICT) {
        each([&](int i, int r, int row, int gm) {
            if (gm < a.M && inO) a.Y[(int64_t)gm * a.O + col] = (acc[i][r] + b3) * sd + mean;
        });
        return;
    }
    if constexpr (MODE == ROWS_TRAIN) __syncthreads();
    double sq = 0.0;
    each([&](int i, int r, int row, int gm) {
        float d = 0.f;
        if (gm < a.M && inO) {
            d = acc[i][r] + b3 - (tt[i][r] - mean) / sd;
            sq += (double)d * (double)d;
        }
        if constexpr (MODE == ROWS_TRAIN) {
            d *= a.gscale;
            acc[i][r] = d;
            At[row][col] = d;
            if (gm < a.M) a.dy[(int64_t)gm * NP + col] = d;
        }
    });
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sq += __shfl_xor(sq, o, 64);
    if (lane == 0) sred[w] = sq;
    if constexpr (MODE == ROWS_TRAIN) bias(2);
    __syncthreads();
    if (t == 0) {
        double v = 0.0;
#pragma unroll
        for (int u = 0; u < RW / 64; ++u) v += sred[u];
        a.lpart[blockIdx.x] = v;
    }
    if constexpr (MODE == ROWS_TRAIN) {
        auto dsilu = [](float z) {
            const float s = sigmoid(z);
            return s * (1.0f + z * (1.0f - s));
        };
        product(T3);   // dy W3
        __syncthreads();
        each([&](int i, int r, int row, int gm) {
            const float d = pad(acc[i][r] * dsilu(z2[i][r]));
            acc[i][r] = d;
            At[row][col] = d;
            if (gm < a.M) a.d2[(int64_t)gm * NP + col] = d;
        });
        bias(1);
        __syncthreads();
        product(T2);   // d2 W2
        each([&](int i, int r, int row, int gm) {
            const float d = acc[i][r] * dsilu(z1[i][r]);
            acc[i][r] = d;
            if (gm < a.M) a.d1[(int64_t)gm * NP + col] = d;
        });
        bias(0);
    }
}

// Partial weight gradients of slice y of the rows: workgroup x computes 128 x 64
// entries of one of gW1 = d1^T X, gW2 = d2^T h1, gW3 = dy^T h2 (tiles of gW1
// first) into wpart[y][parameter].  Both operands are staged as they lie in
// memory, a row of 16 k-slices per LDS row, padded so that the four k groups of a
// wavefront read 64 different banks.
struct GradArgs {
    int M, W, O, I, kchunk, ntile1;
    const float *X, *h1, *h2, *dy, *d2, *d1;
    const int32_t *rows;
    float *wpart;
    int64_t np, off1, off2, off3;
};

__global__ __launch_bounds__(WG) void k_wgrad(GradArgs g) {
    constexpr int LA = NP + 16, LB = 64 + 16;
    __shared__ __align__(16) float As[2][BK][LA], Bs[2][BK][LB];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6, r16 = lane & 15, q = lane >> 4;
    const float *A, *Bp;
    const int32_t *rows = nullptr;
    int nA, nB, n0, ldb;
    int64_t off;
    int x = blockIdx.x;
    if (x < g.ntile1) {
        A = g.d1, Bp = g.X, rows = g.rows, nA = g.W, nB = g.I, ldb = g.I, off = g.off1;
    } else if (x < g.ntile1 + 2) {
        x -= g.ntile1;
        A = g.d2, Bp = g.h1, nA = g.W, nB = g.W, ldb = NP, off = g.off2;
    } else {
        x -= g.ntile1 + 2;
        A = g.dy, Bp = g.h2, nA = g.O, nB = g.W, ldb = NP, off = g.off3;
    }
    n0 = x * 64;
    if (n0 >= nB) return;   // (a hidden width of at most 64 has one tile)
    const int kb = blockIdx.y * g.kchunk, ke = min(g.M, kb + g.kchunk);
    const int ar = t >> 5, ac = (t & 31) * 4;        // A: rows ar and ar + 8 of a slice
    const int br = t >> 4, bc = (t & 15) * 4;        // B: one row, 4 columns
    const bool okb = n0 + bc < nB;                   // nB is a multiple of 4
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 acc[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int n = 0; n < 4; ++n) acc[i][n] = zero;
    auto brow = [&](int k) -> int64_t { return k < ke ? (rows ? (int64_t)rows[k] : (int64_t)k) : 0; };
    auto fetch = [&](int k0, int64_t kr, f32x4 &a0, f32x4 &a1, f32x4 &b) {
        a0 = k0 + ar < ke ? ld4(A + (int64_t)(k0 + ar) * NP + ac) : zero;
        a1 = k0 + ar + 8 < ke ? ld4(A + (int64_t)(k0 + ar + 8) * NP + ac) : zero;
        b = k0 + br < ke && okb ? ld4(Bp + kr * ldb + n0 + bc) : zero;
    };
    f32x4 ra0, ra1, rb;
    fetch(kb, brow(kb + br), ra0, ra1, rb);
    int64_t rnext = brow(kb + BK + br);   // the gathered row of the next slice, one slice ahead
    int cur = 0;
    for (int k0 = kb; k0 < ke; k0 += BK, cur ^= 1) {
        st4(&As[cur][ar][ac], ra0);
        st4(&As[cur][ar + 8][ac], ra1);
        st4(&Bs[cur][br][bc], rb);
        __syncthreads();
        if (k0 + BK < ke) {
            fetch(k0 + BK, rnext, ra0, ra1, rb);
            rnext = brow(k0 + 2 * BK + br);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float a[2], b[4];
#pragma unroll
            for (int i = 0; i < 2; ++i) a[i] = As[cur][4 * j + q][32 * w + 16 * i + r16];
#pragma unroll
            for (int n = 0; n < 4; ++n) b[n] = Bs[cur][4 * j + q][16 * n + r16];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int n = 0; n < 4; ++n) acc[i][n] = mfma(a[i], b[n], acc[i][n]);
        }
    }
    float *out = g.wpart + (int64_t)blockIdx.y * g.np + off;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int n = 0; n < 4; ++n)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int o = 32 * w + 16 * i + 4 * q + r, c = n0 + 16 * n + r16;
                if (o < nA && c < nB) out[(int64_t)o * nB + c] = acc[i][n][r];
            }
}

// Gradient of parameter e: the row slices' partial products in order, or (a
// bias) the row tiles' column sums in order.
struct SumArgs {
    int64_t np, off[7];
    int SW, G;              // row slices of wpart, row tiles of bpart
    const float *wpart, *bpart;
};

__device__ __forceinline__ float grad_sum(const SumArgs &s, int64_t e) {
    int slot = -1;
    int64_t c = 0;
#pragma unroll
    for (int l = 0; l < 3; ++l)
        if (e >= s.off[2 * l + 1] && e < s.off[2 * l + 2]) {
            slot = l;
            c = e - s.off[2 * l + 1];
        }
    double v = 0.0;   // rounded once
    if (slot >= 0) {
        const float *p = s.bpart + slot * NP + c;
#pragma unroll 8
        for (int b = 0; b < s.G; ++b) v += (double)p[(int64_t)b * 3 * NP];
    } else {
#pragma unroll 4
        for (int z = 0; z < s.SW; ++z) v += (double)s.wpart[z * s.np + e];
    }
    return (float)v;
}

__global__ __launch_bounds__(WG) void k_grad_rows(SumArgs s, float *__restrict__ g) {
    const int64_t e = blockIdx.x * (int64_t)WG + threadIdx.x;
    if (e < s.np) g[e] = grad_sum(s, e);
}

__global__ __launch_bounds__(WG) void k_adam_rows(SumArgs s, float *__restrict__ p, float *__restrict__ m,
                                                  float *__restrict__ v, float lr, float b1, float b2, float eps,
                                                  float c1, float c2) {
    const int64_t e = blockIdx.x * (int64_t)WG + threadIdx.x;
    if (e >= s.np) return;
    const float me0 = m[e], ve0 = v[e], pe = p[e];
    const float ge = grad_sum(s, e);
    const float me = b1 * me0 + (1.0f - b1) * ge;
    const float ve = b2 * ve0 + (1.0f - b2) * ge * ge;
    m[e] = me;
    v[e] = ve;
    p[e] = pe - lr * (me * c1) / (sqrtf(ve * c2) + eps);
}

// acc[st] (+)= sum of the row tiles' squares of step st, in a fixed order;
// every step holds G tiles, the last one Glast, `stride` apart
__global__ __launch_bounds__(WG) void k_loss_rows(int steps, int G, int Glast, int stride,
                                                  const double *__restrict__ lpart, double *__restrict__ acc,
                                                  int accumulate) {
    __shared__ double red[WG];
    const int st = blockIdx.x, n = st + 1 == steps ? Glast : G;
    double s = 0.0;
    for (int e = threadIdx.x; e < n; e += WG) s += lpart[(int64_t)st * stride + e];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int h = WG / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) acc[st] = accumulate ? acc[st] + red[0] : red[0];
}

// Rows per tile of k_rows (training keeps four sets of weights in registers,
// which leaves room for two MFMA tiles instead of four)
inline int tile_rows(int64_t n, bool train) { return n > 16384 ? (train ? 32 : 64) : 16; }

// Slices of the first layer's inputs: enough workgroups (two per CU) for few
// rows, at least 64 inputs each
int l1_slices(const Mlp &m, int64_t n, int *kchunk) {
    const int64_t tiles = ceil_div(n, BM);
    const int64_t S = std::max<int64_t>(std::min<int64_t>({16, ceil_div(512, tiles), m.n_in / 64}), 1);
    *kchunk = (int)ceil_div(ceil_div(m.n_in, S), BK) * BK;
    return (int)ceil_div(m.n_in, *kchunk);
}

// Slices of the rows in the weight gradients: about one workgroup per CU
int grad_slices(const Mlp &m, int64_t n, int *kchunk) {
    const int64_t tiles = ceil_div(m.n_in, 64) + 4;
    const int64_t S = std::max<int64_t>(std::min<int64_t>(ceil_div(256, tiles), n / 64), 1);
    *kchunk = (int)ceil_div(ceil_div(n, S), BK) * BK;
    return (int)ceil_div(n, *kchunk);
}

void ensure(Mlp &m, int64_t n, bool train) {
    int kc = 0;
    const size_t part = (size_t)l1_slices(m, n, &kc) * n * NP;
    if (m.r_part.n < part) m.r_part.alloc(part);
    if (!train) return;
    for (DBuf<float> *d : {&m.r_h1, &m.r_h2, &m.r_dy, &m.r_d2, &m.r_d1})
        if (d->n < (size_t)n * NP) d->alloc((size_t)n * NP);
    const size_t wp = (size_t)grad_slices(m, n, &kc) * m.np, bp = (size_t)ceil_div(n, tile_rows(n, true)) * 3 * NP;
    if (m.r_wpart.n < wp) m.r_wpart.alloc(wp);
    if (m.r_bpart.n < bp) m.r_bpart.alloc(bp);
}

template <int MODE>
void launch_rows(Mlp &m, hipStream_t s, const float *X, const float *T, const int32_t *rows, int64_t n, float *Y,
                 double *lpart) {
    int kc = 0;
    const int S = l1_slices(m, n, &kc);
    const float *p = m.p.get();
    hipLaunchKernelGGL(k_l1, dim3((unsigned)ceil_div(n, BM), S), dim3(WG), 0, s, (int)n, m.n_in, X, rows, p + m.off[0],
                       m.width, kc, m.r_part.get());
    RowArgs a{};
    a.M = (int)n, a.S = S, a.W = m.width, a.O = m.n_out;
    a.part = m.r_part.get();
    a.b1 = p + m.off[1], a.W2 = p + m.off[2], a.b2 = p + m.off[3], a.W3 = p + m.off[4], a.b3 = p + m.off[5];
    a.mean = m.mean.get(), a.std = m.std.get();
    a.T = T, a.rows = rows, a.Y = Y;
    a.h1 = m.r_h1.get(), a.h2 = m.r_h2.get(), a.dy = m.r_dy.get(), a.d2 = m.r_d2.get(), a.d1 = m.r_d1.get();
    a.bpart = m.r_bpart.get(), a.lpart = lpart;
    a.gscale = (float)(2.0 / (double)(n * m.n_out));
    const int tr = tile_rows(n, MODE == ROWS_TRAIN);
    const dim3 g((unsigned)ceil_div(n, tr));
    if (tr > 16) hipLaunchKernelGGL((k_rows<MODE == ROWS_TRAIN ? 2 : 4, MODE>), g, dim3(RW), 0, s, a);
    else hipLaunchKernelGGL((k_rows<1, MODE>), g, dim3(RW), 0, s, a);
    CS_LAUNCH_CHECK();
}

SumArgs weight_grads(Mlp &m, hipStream_t s, const float *X, const int32_t *rows, int64_t n) {
    GradArgs g{};
    const int S = grad_slices(m, n, &g.kchunk);
    g.M = (int)n, g.W = m.width, g.O = m.n_out, g.I = m.n_in;
    g.ntile1 = (int)ceil_div(m.n_in, 64);
    g.X = X, g.rows = rows;
    g.h1 = m.r_h1.get(), g.h2 = m.r_h2.get(), g.dy = m.r_dy.get(), g.d2 = m.r_d2.get(), g.d1 = m.r_d1.get();
    g.wpart = m.r_wpart.get();
    g.np = m.np, g.off1 = m.off[0], g.off2 = m.off[2], g.off3 = m.off[4];
    hipLaunchKernelGGL(k_wgrad, dim3(g.ntile1 + 4, S), dim3(WG), 0, s, g);
    CS_LAUNCH_CHECK();
    SumArgs a{};
    a.np = m.np, a.SW = S, a.G = (int)ceil_div(n, tile_rows(n, true));
    std::copy(m.off, m.off + 7, a.off);
    a.wpart = m.r_wpart.get(), a.bpart = m.r_bpart.get();
    return a;
}

constexpr int64_t PREDICT_ROWS = 131072;   // rows per pass of predictions and losses (67 MB of products)

}  // namespace

// The row-tile path: widths of at most 128 (one column of workgroups covers a
// layer; wider networks would need several passes over X) and 16-byte rows of
// X and of every weight matrix.
bool rows_path(const Mlp &m, const float *X) {
    return m.width <= NP && m.n_out <= NP && m.n_in % 4 == 0 && m.width % 4 == 0 &&
           reinterpret_cast<uintptr_t>(X) % 16 == 0;
}

void rows_predict(Mlp &m, hipStream_t s, const float *X, int64_t n, float *Y) {
    ensure(m, std::min(n, PREDICT_ROWS), false);
    for (int64_t r0 = 0; r0 < n; r0 += PREDICT_ROWS) {
        const int64_t nr = std::min(PREDICT_ROWS, n - r0);
        ensure(m, nr, false);   // a short last pass is cut into more slices
        launch_rows<ROWS_PREDICT>(m, s, X + r0 * m.n_in, nullptr, nullptr, nr, Y + r0 * m.n_out, nullptr);
    }
}

// acc[0] = sum of squared errors over the rows
void rows_loss(Mlp &m, hipStream_t s, const float *X, const float *T, const int32_t *rows, int64_t n) {
    for (int64_t r0 = 0; r0 < n; r0 += PREDICT_ROWS) {
        const int64_t nr = std::min(PREDICT_ROWS, n - r0);
        const int G = (int)ceil_div(nr, tile_rows(nr, false));
        ensure(m, nr, false);
        if (m.r_lpart.n < (size_t)G) m.r_lpart.alloc(G);
        launch_rows<ROWS_LOSS>(m, s, rows ? X : X + r0 * m.n_in, rows ? T : T + r0 * m.n_out,
                               rows ? rows + r0 : nullptr, nr, nullptr, m.r_lpart.get());
        hipLaunchKernelGGL(k_loss_rows, dim3(1), dim3(WG), 0, s, 1, G, G, G, m.r_lpart.get(), m.acc.get(), r0 > 0 ? 1 : 0);
        CS_LAUNCH_CHECK();
    }
}

// gradient into m.g, sum of squared errors into acc[0]
void rows_gradient(Mlp &m, hipStream_t s, const float *X, const float *T, const int32_t *rows, int64_t n) {
    const int G = (int)ceil_div(n, tile_rows(n, true));
    ensure(m, n, true);
    if (m.r_lpart.n < (size_t)G) m.r_lpart.alloc(G);
    launch_rows<ROWS_TRAIN>(m, s, X, T, rows, n, nullptr, m.r_lpart.get());
    hipLaunchKernelGGL(k_loss_rows, dim3(1), dim3(WG), 0, s, 1, G, G, G, m.r_lpart.get(), m.acc.get(), 0);
    const SumArgs a = weight_grads(m, s, X, rows, n);
    hipLaunchKernelGGL(k_grad_rows, dim3((unsigned)ceil_div(m.np, WG)), dim3(WG), 0, s, a, m.g.get());
    CS_LAUNCH_CHECK();
}

// One pass over the rows `order` in batches; acc[st] = sum of squared errors
// of step st.  rate(k): learning rate and bias corrections of the k-th step.
void rows_epoch(Mlp &m, hipStream_t s, const float *X, const float *T, const int32_t *order, int64_t n_train,
                int64_t batch, const std::function<AdamRate()> &rate) {
    const int64_t steps = ceil_div(n_train, batch), b = std::min(batch, n_train), last = n_train - (steps - 1) * batch;
    const int G = (int)ceil_div(b, tile_rows(b, true)), Glast = (int)ceil_div(last, tile_rows(last, true));
    ensure(m, b, true);
    ensure(m, last, true);   // a short last batch is cut into more slices
    const int stride = std::max(G, Glast);
    if (m.r_lpart.n < (size_t)(steps * stride)) m.r_lpart.alloc(steps * stride);
    for (int64_t st = 0; st < steps; ++st) {
        const int64_t r0 = st * batch, nr = std::min(batch, n_train - r0);
        launch_rows<ROWS_TRAIN>(m, s, X, T, order + r0, nr, nullptr, m.r_lpart.get() + st * stride);
        const SumArgs a = weight_grads(m, s, X, order + r0, nr);
        const AdamRate r = rate();
        hipLaunchKernelGGL(k_adam_rows, dim3((unsigned)ceil_div(m.np, WG)), dim3(WG), 0, s, a, m.p.get(), m.m.get(),
                           m.v.get(), r.lr, r.b1, r.b2, r.eps, r.c1, r.c2);
        CS_LAUNCH_CHECK();
    }
    hipLaunchKernelGGL(k_loss_rows, dim3((unsigned)steps), dim3(WG), 0, s, (int)steps, G, Glast, stride, m.r_lpart.get(),
                       m.acc.get(), 0);
    CS_LAUNCH_CHECK();
}

}  // namespace cs
