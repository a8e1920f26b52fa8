// The coarsest level's l1-Jacobi sweeps by powers of the sweep matrix, gfx950.
// A coarsest level too large for a dense operator and no star ran one launch per
// sweep (20 by default), each a chain of dependent loads on a level of a few
// megabytes: launch latency, not bandwidth.  With M = I - D A, formed once at
// setup as M^p (p = 2 or 4), p sweeps are one:
//   x_(t+p) = M^p x_t + c_p,   c_p = p sweeps from zero,
// so 20 sweeps take 10 or 6 launches.  Rows are kept at a fixed stride (no row
// pointer to wait for) and padded with zeros.
#include <type_traits>

#include "device.h"
#include "internal.h"

#pragma clang fp contract(off)

namespace bcm {

namespace {

constexpr int kCand = 4096;    // most products that form one row of a square
constexpr int kCandWave = 512; // rows of up to this many take one wave, longer ones four
constexpr int kRowMax = 512;   // most entries of a row that is squared
constexpr int kPad = 64;       // row strides, a multiple of every lane count

inline int blocks_for(long long threads) { return (int)((threads + kBlock - 1) / kBlock); }

// M = I - D A at stride W >= the longest row
__global__ void __launch_bounds__(kBlock)
k_power_first(int n, int W, const int *__restrict__ rp, const int *__restrict__ ci, const double *__restrict__ a,
              const double *__restrict__ dinv, int *__restrict__ len, int *__restrict__ col, double *__restrict__ val) {
    constexpr int G = 16;
    const int i = (blockIdx.x * kBlock + threadIdx.x) / G, lane = threadIdx.x % G;
    if (i >= n) return;
    const int s = rp[i], l = rp[i + 1] - s;
    const double d = dinv[i];
    const size_t o = (size_t)i * W;
    for (int k = lane; k < W; k += G) {
        const int j = k < l ? ci[s + k] : i;
        col[o + k] = j;
        val[o + k] = k < l ? (j == i ? 1.0 - d * a[s + k] : -(d * a[s + k])) : 0.0;
    }
    if (lane == 0) len[i] = l;
}

// Rows of a CSR matrix, and of a power
struct RowsCsr {
    const int *rp;
    __device__ size_t begin(int i) const { return rp[i]; }
    __device__ int length(int i) const { return rp[i + 1] - rp[i]; }
};
struct RowsPadded {
    const int *len;
    int W;
    __device__ size_t begin(int i) const { return (size_t)i * W; }
    __device__ int length(int i) const { return len[i]; }
};

// products that form row i of the square
template <typename Rows>
__global__ void __launch_bounds__(kBlock)
k_power_products(int n, Rows R, const int *__restrict__ col, int *__restrict__ cnt) {
    constexpr int G = 16;
    const int i = (blockIdx.x * kBlock + threadIdx.x) / G, lane = threadIdx.x % G;
    if (i >= n) return;
    const int l = R.length(i);
    const size_t o = R.begin(i);
    int c = 0;
    for (int k = lane; k < l; k += G) c += R.length(col[o + k]);
    c = group_sum<G>(c);
    if (lane == 0) cnt[i] = c;
}

// One row of M M per workgroup: its products (j, k) -> m_ij m_jk, in that order,
// sorted by column in LDS; each column's are then summed in order (the result
// depends on nothing else).  Pass 0 counts the row's columns, pass 1 writes them.
// Rows of more than Lo and at most Cap products by T threads: one wave needs no
// barrier between the stages of the sort and 12 KB of LDS instead of 66 (9,628 rows
// of 110 products on average and at most 2,200: 198 -> 116 us a pass).
template <int Lo, int Cap, int T>
__global__ void __launch_bounds__(T)
k_power_square(int pass, int n, int W, const int *__restrict__ len, const int *__restrict__ col,
               const double *__restrict__ val, int W2, int *__restrict__ len2, int *__restrict__ col2,
               double *__restrict__ val2, const int *__restrict__ products) {
    __shared__ unsigned long long keys[Cap];
    __shared__ double terms[Cap];
    __shared__ int off[kRowMax + 1];
    __shared__ int wsum[T / 64];
    const int i = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int l = len[i], C = products[i];
    if (C <= Lo || C > Cap) return;
    auto sync = [] {
        if (T == 64) wave_sync();
        else __syncthreads();
    };
    const size_t o = (size_t)i * W;
    for (int k = tid; k < l; k += T) off[k + 1] = len[col[o + k]];
    if (tid == 0) off[0] = 0;
    sync();
    if (wv == 0) {  // prefix sums of the row lengths, 64 at a time
        int run = 0;
        for (int k0 = 0; k0 < l; k0 += 64) {
            int x = k0 + lane < l ? off[k0 + lane + 1] : 0;
            for (int s = 1; s < 64; s <<= 1) {
                const int t = __shfl_up(x, s, 64);
                if (lane >= s) x += t;
            }
            if (k0 + lane < l) off[k0 + lane + 1] = run + x;
            run += __shfl(x, 63, 64);
        }
    }
    sync();
    int P = 64;
    while (P < C) P <<= 1;
    for (int c = tid; c < P; c += T) {
        unsigned long long key = ~0ull;
        if (c < C) {
            int lo = 0, hi = l - 1;  // the entry whose products hold c
            while (lo < hi) {
                const int m = (lo + hi + 1) >> 1;
                if (off[m] <= c) lo = m; else hi = m - 1;
            }
            const size_t q = (size_t)col[o + lo] * W + (c - off[lo]);
            key = ((unsigned long long)(unsigned)col[q] << 32) | (unsigned)c;
            if (pass) terms[c] = val[o + lo] * val[q];
        }
        keys[c] = key;
    }
    sync();
    for (int size = 2; size <= P; size <<= 1)
        for (int st = size >> 1; st > 0; st >>= 1) {
            for (int t = tid; t < (P >> 1); t += T) {
                const int a = 2 * t - (t & (st - 1)), b = a + st;
                const bool up = (a & size) == 0;
                const unsigned long long x = keys[a], y = keys[b];
                if ((x > y) == up) {
                    keys[a] = y;
                    keys[b] = x;
                }
            }
            sync();
        }
    // the starts of the columns' runs, numbered
    const int per = (P + T - 1) / T, k0 = min(tid * per, C), k1 = min(k0 + per, C);
    auto starts = [&](int k) { return k == 0 || (int)(keys[k] >> 32) != (int)(keys[k - 1] >> 32); };
    int mine = 0;
    for (int k = k0; k < k1; ++k) mine += starts(k) ? 1 : 0;
    int inc = mine;
    for (int s = 1; s < 64; s <<= 1) {
        const int t = __shfl_up(inc, s, 64);
        if (lane >= s) inc += t;
    }
    if (lane == 63) wsum[wv] = inc;
    sync();
    int rank = inc - mine, tot = 0;
    for (int w = 0; w < T / 64; ++w) {
        if (w < wv) rank += wsum[w];
        tot += wsum[w];
    }
    if (pass == 0) {
        if (tid == 0) len2[i] = tot;
        return;
    }
    const size_t o2 = (size_t)i * W2;
    for (int k = k0; k < k1; ++k) {
        if (!starts(k)) continue;
        const int f = (int)(keys[k] >> 32);
        double s = terms[(int)(keys[k] & 0xffffffffull)];
        for (int e = k + 1; e < C && (int)(keys[e] >> 32) == f; ++e) s += terms[(int)(keys[e] & 0xffffffffull)];
        col2[o2 + rank] = f;
        val2[o2 + rank] = s;
        ++rank;
    }
    for (int k = tot + tid; k < W2; k += T) {
        col2[o2 + k] = i;
        val2[o2 + k] = 0.0;
    }
}

// Two sweeps from zero: c_2 = 2 D b - D A D b = M D b + D b
template <typename VB>
struct Scaled {
    const double *dinv;
    const VB *b;
    __device__ double operator()(int j) const { return dinv[j] * (double)b[j]; }
};
struct Vector {
    const double *x;
    __device__ double operator()(int j) const { return x[j]; }
};

// Entries k, k + G, ..., k + (U - 1) G of a row of l entries (k: the lane's first
// of them less its lane), all loaded before any is used.
template <int G, int U, typename F>
__device__ __forceinline__ double power_batch(const int *__restrict__ col, const double *__restrict__ val, size_t o,
                                              int k, int l, double s, F f) {
    int j[U];
    double v[U], x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const size_t q = k + u * G < l ? o + k + u * G : o;  // (the padding makes the last chunk whole)
        j[u] = col[q];
        v[u] = val[q];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) x[u] = f(j[u]);
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (k + u * G < l) s += v[u] * x[u];
    return s;
}

// xo_i = sum_k m_ik f(k) + g(i), G lanes per row.  The first G entries of every
// row are loaded beside its length (rows are padded), and the rest in as few
// batches as its length asks for: a launch is two to four dependent loads and a
// reduction, set by its longest rows.
template <int G, typename VX, typename F, typename C>
__global__ void __launch_bounds__(kBlock)
k_power_apply(int n, int W, const int *__restrict__ len, const int *__restrict__ col, const double *__restrict__ val,
              F f, C g, VX *__restrict__ xo, const double *__restrict__ done) {
    const int i = (xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x) / G, lane = threadIdx.x % G;
    if (i >= n) return;
    const size_t o = (size_t)i * W + lane;
    const int l = len[i];
    const double c = g(i);
    double s = val[o] * f(col[o]);
    for (int k = G; k < l;) {
        const int rest = (l - k + G - 1) / G;
        if (rest == 1) {
            s = power_batch<G, 1>(col, val, o, k, l, s, f);
            k += G;
        } else if (rest <= 3) {
            s = power_batch<G, 3>(col, val, o, k, l, s, f);
            k += 3 * G;
        } else {
            s = power_batch<G, 8>(col, val, o, k, l, s, f);
            k += 8 * G;
        }
    }
    s = group_sum<G>(s);
    // (the solve-ended flag is tested before the store only)
    if (lane == 0 && !(done && *done != 0.0)) xo[i] = (VX)(s + c);
}

template <typename VX, typename F, typename C>
void apply(hipStream_t s, int n, const PowerMat &M, F f, C g, VX *x, const double *done) {
    const int lanes = power_lanes(M.nnz, n);
    auto go = [&](auto gc) {
        constexpr int G = decltype(gc)::value;
        hipLaunchKernelGGL((k_power_apply<G, VX, F, C>), dim3(blocks_for((long long)n * G)), dim3(kBlock), 0, s, n, M.W,
                           M.len, M.col, M.val, f, g, x, done);
    };
    if (lanes == 16) go(std::integral_constant<int, 16>{});
    else if (lanes == 32) go(std::integral_constant<int, 32>{});
    else go(std::integral_constant<int, 64>{});
}

// sweeps = p k, k >= 2: c_p, then k - 1 times x <- M^p x + c_p
template <typename VB, typename VX>
void power_t(hipStream_t s, const PowerOp &P, int n, int sweeps, const double *dinv, const VB *b, VX *x,
             const double *done) {
    const Scaled<VB> db{dinv, b};
    double *c = P.buf[0], *xa = P.buf[1], *xb = P.buf[2];
    const int steps = sweeps / P.p;
    apply(s, n, P.m[0], db, db, c, done);  // c_2
    if (P.p == 4) {
        apply(s, n, P.m[1], Vector{c}, Vector{c}, xa, done);  // c_4 = M^2 c_2 + c_2
        std::swap(c, xa);
    }
    const PowerMat &M = P.m[P.p == 4 ? 2 : 1];
    const double *in = c;
    for (int t = 1; t < steps; ++t) {
        if (t == steps - 1) {
            apply(s, n, M, Vector{in}, Vector{c}, x, done);
        } else {
            double *out = in == xa ? xb : xa;
            apply(s, n, M, Vector{in}, Vector{c}, out, done);
            in = out;
        }
    }
}

}  // namespace

int power_row_limit() { return kRowMax; }
int power_cand_limit() { return kCand; }
int power_lanes(long long nnz, int n) {
    const double avg = (double)nnz / n;
    return avg <= 12.0 ? 16 : (avg <= 40.0 ? 32 : 64);
}
int power_stride(int longest) { return (longest + kPad - 1) / kPad * kPad; }

void launch_power_first(hipStream_t s, const Level &L, const PowerMat &M) {
    hipLaunchKernelGGL(k_power_first, dim3(blocks_for(16LL * L.A.n)), dim3(kBlock), 0, s, L.A.n, M.W, L.A.rp, L.A.ci,
                       L.A.v, L.dinv, M.len, M.col, M.val);
}

void launch_power_products(hipStream_t s, const Csr &A, int *cnt) {
    hipLaunchKernelGGL(k_power_products<RowsCsr>, dim3(blocks_for(16LL * A.n)), dim3(kBlock), 0, s, A.n,
                       RowsCsr{A.rp}, A.ci, cnt);
}

void launch_power_products(hipStream_t s, int n, const PowerMat &M, int *cnt) {
    hipLaunchKernelGGL(k_power_products<RowsPadded>, dim3(blocks_for(16LL * n)), dim3(kBlock), 0, s, n,
                       RowsPadded{M.len, M.W}, M.col, cnt);
}

void launch_power_square(hipStream_t s, int pass, int n, const PowerMat &M, const PowerMat &Q, const int *products,
                         int most) {
    hipLaunchKernelGGL((k_power_square<0, kCandWave, 64>), dim3(n), dim3(64), 0, s, pass, n, M.W, M.len, M.col, M.val,
                       Q.W, Q.len, Q.col, Q.val, products);
    if (most > kCandWave)
        hipLaunchKernelGGL((k_power_square<kCandWave, kCand, kBlock>), dim3(n), dim3(kBlock), 0, s, pass, n, M.W, M.len,
                           M.col, M.val, Q.W, Q.len, Q.col, Q.val, products);
}

void launch_power(hipStream_t s, const PowerOp &P, int n, int sweeps, const double *dinv, const void *b, void *x,
                  int b_f64, int x_f64, const double *done) {
    if (b_f64 && x_f64) power_t(s, P, n, sweeps, dinv, (const double *)b, (double *)x, done);
    else power_t(s, P, n, sweeps, dinv, (const float *)b, (float *)x, done);
}

}  // namespace bcm
