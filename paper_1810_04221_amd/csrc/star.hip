// Star levels for gfx950.  On strongly heterogeneous problems the coarsening
// of Section 2.2 stalls: one row (the hub) ends up coupled to every other row,
// and each of those (the leaves) holds only its diagonal and the hub entry.  A
// pairwise sweep then matches the hub with one leaf and leaves a star with one
// row less, so the rule of Section 5 (stop at 40 n^(1/3) rows or 40 levels)
// appends dozens of such levels.  Two things are special to them:
//
//  * Setup.  Matching, Algorithm 2, the prolongator and P^T A P of one sweep
//    are one launch (k_star_sweep): the suitor of the hub is the leaf of largest
//    weight, and every row of the coarse star follows from one fine row.
//  * Solve.  Every leaf's value along the whole descent, the coarsest level's
//    sweeps and the ascent is a scalar recurrence driven by the leaf's own
//    right-hand side and by the hub's values alone.  The V-cycle from the first
//    star level down is therefore diag(delta) + V A^T with a few dozen columns
//    (one per sum over the leaves that the hub takes), formed once at setup and
//    applied as two passes (k_chain_sums, k_chain_apply) instead of three
//    launches per level.  The coarsest level's l1-Jacobi sweeps alone are the
//    same with no level above it.
#include "device.h"
#include "internal.h"

#pragma clang fp contract(off)

namespace bcm {

namespace {

inline int blocks_for(long long threads) { return (int)((threads + kBlock - 1) / kBlock); }

// ----------------------------------------------------------------------------
// Recognising a star
// ----------------------------------------------------------------------------
// out[0] += rows of more than two entries, out[1] = max of their indices
// (start both at 0); out[2] is raised to 1 where a row of at most two entries
// is not {diagonal} or {diagonal, one other column}.
__global__ void __launch_bounds__(kBlock)
k_star_find(int n, const int *__restrict__ rp, const int *__restrict__ ci, int *__restrict__ out) {
    const int i = blockIdx.x * kBlock + threadIdx.x;
    bool lng = false, odd = false;
    if (i < n) {
        const int s = rp[i], len = rp[i + 1] - s;
        lng = len > 2;
        if (!lng) odd = len < 1 || !(ci[s] == i || (len == 2 && ci[s + 1] == i));
    }
    if (lng) {
        atomicAdd(&out[0], 1);
        atomicMax(&out[1], i);
    }
    if (odd) atomicMax(&out[2], 1);
}

// out[2] is raised where a leaf's other column is not the hub; out[3] where a leaf
// has no hub entry, the hub row has no entry for it, or the two differ.
__global__ void __launch_bounds__(kBlock)
k_star_verify(int n, const int *__restrict__ rp, const int *__restrict__ ci, const double *__restrict__ v, int hub,
              int *__restrict__ out) {
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n || i == hub) return;
    const int s = rp[i], len = rp[i + 1] - s;
    if (len != 2) {
        atomicMax(&out[3], 1);
        return;
    }
    const int q = ci[s] == i ? s + 1 : s;
    if (ci[q] != hub) {
        atomicMax(&out[2], 1);
        return;
    }
    const int hs = rp[hub], hl = rp[hub + 1] - hs;
    const bool same = hl == n && ci[hs + i] == i && __double_as_longlong(v[hs + i]) == __double_as_longlong(v[q]);
    if (!same) atomicMax(&out[3], 1);
}

// ----------------------------------------------------------------------------
// Setup sweeps.  A star whose hub is coupled to all its n rows has an analytic
// layout: row j < hub holds {j, hub} from entry 2j, the hub row all n columns
// from 2 hub, row j > hub {hub, j} from 2 (j - 1) + n.
// ----------------------------------------------------------------------------
__device__ __forceinline__ int star_row(int j, int hub, int n) { return j <= hub ? 2 * j : 2 * (j - 1) + n; }

// better of two candidate leaves: larger weight, then larger index (the order
// of the matching among edges that share the hub); -1: none
__device__ __forceinline__ void star_better(double &c, int &i, double c2, int i2) {
    if (i2 >= 0 && (i < 0 || c2 > c || (c2 == c && i2 > i))) {
        c = c2;
        i = i2;
    }
}

// best candidate of the workgroup (valid in every thread)
__device__ __forceinline__ void star_block_best(double &c, int &i) {
    __shared__ double sc[kBlock / 64];
    __shared__ int si[kBlock / 64];
    for (int o = 32; o > 0; o >>= 1) {
        const double c2 = __shfl_xor(c, o, 64);
        const int i2 = __shfl_xor(i, o, 64);
        star_better(c, i, c2, i2);
    }
    if ((threadIdx.x & 63) == 0) {
        sc[threadIdx.x >> 6] = c;
        si[threadIdx.x >> 6] = i;
    }
    __syncthreads();
    c = sc[0];
    i = si[0];
    for (int w = 1; w < kBlock / 64; ++w) star_better(c, i, sc[w], si[w]);
    __syncthreads();
}

// weight of the edge between rows i and h (Section 2.2, in the operand order
// every end of an edge uses), or no candidate when it cannot be matched
__device__ __forceinline__ void star_weight(int i, int h, double a, double aii, double wi, double ahh, double wh,
                                            double &c, int &idx) {
    const bool lo = i < h;
    const double wm = lo ? wi : wh, wM = lo ? wh : wi, dm = lo ? aii : ahh, dM = lo ? ahh : aii;
    const double num = ((2.0 * a) * wm) * wM;
    const double den = (dm * wm) * wm + (dM * wM) * wM;
    c = 1.0 - num / den;
    idx = (c > 0.0 && c < INFINITY) ? i : -1;
}

// the first star's best leaf, one candidate per workgroup; *hub_out = hub
__global__ void __launch_bounds__(kBlock)
k_star_best(int n, const double *__restrict__ v, const double *__restrict__ w, int hub, int *__restrict__ hub_out,
            double *__restrict__ pc, int *__restrict__ pi) {
    const int i = blockIdx.x * kBlock + threadIdx.x;
    double c = 0.0;
    int idx = -1;
    if (i < n && i != hub) {
        const int q = star_row(i, hub, n);
        const bool lo = i < hub;
        star_weight(i, hub, v[q + (lo ? 1 : 0)], v[q + (lo ? 0 : 1)], w[i], v[3 * (size_t)hub], w[hub], c, idx);
    }
    star_block_best(c, idx);
    if (threadIdx.x == 0) {
        pc[blockIdx.x] = c;
        pi[blockIdx.x] = idx;
        if (blockIdx.x == 0) *hub_out = hub;
    }
}

// One pairwise sweep on a star of n rows: the leaf l of largest weight joins
// the hub (the workgroups' candidates come from the launch before); aggregates
// numbered by their smallest member are then the rows with max(hub, l) taken
// out; prolongator and coarse entries as the general kernels form them, term
// by term in the same order:
//   p = w / sqrt(w_i w_i + w_j w_j) on the pair, w / |w| elsewhere,
//   a'_jj = (p_j a_jj) p_j,  a'_jh = (p_m a) p_M with m = min, M = max,
//   a'_hh = sum of its four terms in ascending (m, M).
// One thread per fine row of the level (nf >= n when earlier sweeps' aggregates
// are composed with this one's).  The same pass checks the star's values,
// computes the coarse star's weights and leaves one candidate per workgroup
// for the next sweep.  No eligible leaf: *sel = -1, and every later sweep of
// the chain (hub -1) does nothing.  Latency-bound: a few thousand to some ten
// thousand rows, one launch of about 5 us where the general sweep with its
// segmented sorts took about 20 launches and 0.4 ms.
__global__ void __launch_bounds__(kBlock) k_star_sweep(StarSweep S) {
    const int hub = *S.hub;
    double bc = 0.0;
    int l = -1;
    for (int t = threadIdx.x; t < S.np; t += kBlock) star_better(bc, l, S.pc[t], S.pi[t]);
    star_block_best(bc, l);
    if (hub < 0) l = -1;
    if (l < 0) {
        if (threadIdx.x == 0) {
            S.pi_out[blockIdx.x] = -1;
            S.pc_out[blockIdx.x] = 0.0;
            if (blockIdx.x == 0) {
                *S.sel = -1;
                *S.hub_out = -1;
            }
        }
        return;
    }
    const int n = S.n, n1 = n - 1;
    const int lo = min(hub, l), hi = max(hub, l);
    const int ql = star_row(l, hub, n);
    const double ahh = S.v[3 * (size_t)hub], all = S.v[ql + (l < hub ? 0 : 1)], ahl = S.v[ql + (l < hub ? 1 : 0)];
    const double wh = S.w[hub], wl = S.w[l];
    const double wlo = lo == hub ? wh : wl, whi = lo == hub ? wl : wh;
    const double sp = sqrt(wlo * wlo + whi * whi);
    const double ph = wh / sp, pl = wl / sp;
    const double thh = (ph * ahh) * ph, tll = (pl * all) * pl;
    const double tx = ((lo == hub ? ph : pl) * ahl) * (lo == hub ? pl : ph);
    const double first = lo == hub ? thh : tll, last = lo == hub ? tll : thh;
    const double ahh1 = ((first + tx) + tx) + last;
    const int t = blockIdx.x * kBlock + threadIdx.x;
    double cc = 0.0;
    int ci1 = -1;
    if (t < n) {  // row t of the star
        const int q = star_row(t, hub, n);
        const double wt = S.w[t];
        int f = 0;
        if (t == hub) {
            if (!isfinite(ahh)) f |= kErrNonFinite;
            if (!(ahh > 0.0)) f |= kErrDiagNonPos;
        } else {
            const double ajj = S.v[q + (t < hub ? 0 : 1)], ajh = S.v[q + (t < hub ? 1 : 0)];
            if (!isfinite(ajj) || !isfinite(ajh)) f |= kErrNonFinite;
            if (!(ajj > 0.0)) f |= kErrDiagNonPos;
            if (t != l) {
                const double w1 = fabs(wt), pt = wt / w1;
                const double d1 = (pt * ajj) * pt;
                const double o1 = ((t < hub ? pt : ph) * ajh) * (t < hub ? ph : pt);
                const int j = t < hi ? t : t - 1;
                const int q1 = star_row(j, lo, n1);
                const bool low = j < lo;
                S.rp[j] = q1;
                S.ci[q1] = low ? j : lo;
                S.ci[q1 + 1] = low ? lo : j;
                S.cv[q1] = low ? d1 : o1;
                S.cv[q1 + 1] = low ? o1 : d1;
                S.ci[2 * (size_t)lo + j] = j;
                S.cv[2 * (size_t)lo + j] = o1;
                S.cw[j] = w1;
                star_weight(j, lo, o1, d1, w1, ahh1, sp, cc, ci1);
            }
        }
        if (!(isfinite(wt) && wt != 0.0)) f |= kErrW;
        if (f) atomicOr(S.flags, f);
        if (t == hub) {
            S.rp[lo] = 2 * lo;
            S.rp[n1] = 3 * n1 - 2;
            S.rp[n1 + 1] = n1;  // the longest row, as the general sweep leaves it
            S.ci[3 * (size_t)lo] = lo;
            S.cv[3 * (size_t)lo] = ahh1;
            S.cw[lo] = sp;
            *S.sel = l;
            *S.hub_out = lo;
        }
        // members of the aggregate of row t (the hub's: below, once)
        if (t != hub && t != l) {
            const int j = t < hi ? t : t - 1, st = S.stride_prev;
            for (int u = 0; u < 2 * st; ++u)
                S.mem[(size_t)j * 2 * st + u] = u >= st ? -1 : (S.mem_prev ? S.mem_prev[(size_t)t * st + u] : t);
        } else if (t == hub) {
            const int st = S.stride_prev;
            int buf[16];
            int cnt = 0;
            for (int h = 0; h < 2; ++h) {
                const int F = h == 0 ? lo : hi;
                for (int u = 0; u < st; ++u) {
                    const int i = S.mem_prev ? S.mem_prev[(size_t)F * st + u] : F;
                    if (i < 0) break;
                    int pos = cnt++;
                    while (pos > 0 && buf[pos - 1] > i) { buf[pos] = buf[pos - 1]; --pos; }
                    buf[pos] = i;
                }
            }
            for (int u = 0; u < 2 * st; ++u) S.mem[(size_t)lo * 2 * st + u] = u < cnt ? buf[u] : -1;
        }
    }
    if (t < S.nf) {  // fine row t of the level
        const int a = S.agg_prev ? S.agg_prev[t] : t;
        const double pa = a == hub ? ph : (a == l ? pl : S.w[a] / fabs(S.w[a]));
        S.agg[t] = (a == hub || a == l) ? lo : (a < hi ? a : a - 1);
        S.p[t] = S.agg_prev ? S.p_prev[t] * pa : pa;
    }
    star_block_best(cc, ci1);
    if (threadIdx.x == 0) {
        S.pc_out[blockIdx.x] = cc;
        S.pi_out[blockIdx.x] = ci1;
    }
}

// l1-Jacobi diagonals (Section 3.2) of all the star levels of a chain at once
// (blockIdx.y = level): a leaf's from its two entries; the hub row's |a_hj|
// summed per workgroup, then by k_star_dhub in workgroup order.
__global__ void __launch_bounds__(kBlock)
k_star_dinv(const ChainLevel *__restrict__ tab, double *__restrict__ part) {
    const ChainLevel L = tab[blockIdx.y];
    const int i = blockIdx.x * kBlock + threadIdx.x;
    double s[1] = {0.0};
    if (i < L.n) {
        const double ah = L.v[2 * (size_t)L.hub + i];  // hub row, column i
        s[0] = fabs(ah);
        if (i != L.hub) {
            const int q = star_row(i, L.hub, L.n);
            L.dinv[i] = 1.0 / (fabs(L.v[q]) + fabs(L.v[q + 1]));
        }
    }
    __shared__ double lds[16];
    block_sum<1>(s, lds);
    if (threadIdx.x == 0) part[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = s[0];
}

__global__ void __launch_bounds__(kBlock)
k_star_dhub(const ChainLevel *__restrict__ tab, const double *__restrict__ part, int nb) {
    const ChainLevel L = tab[blockIdx.x];
    double s[1] = {0.0};
    for (int t = threadIdx.x; t < nb; t += kBlock) s[0] += part[(size_t)blockIdx.x * nb + t];
    __shared__ double lds[16];
    block_sum<1>(s, lds);
    if (threadIdx.x == 0) L.dinv[L.hub] = 1.0 / s[0];
}

// ----------------------------------------------------------------------------
// The chain operator.  Star levels t = 0 .. L - 1 and the coarsest star L.
// Hub scalars ("drivers"): H_t = b of the hub at level t; y_k, k = 1 .. S - 1,
// its coarsest iterates; W_t = x of the hub at level t + 1; X_t = d H_t + p W_t
// its prolonged iterate.  A leaf with c = 1 - d a_jj:
//   down    r = c b - a_jh d_h H_t;  b <- p r     (merged at t: p r goes to the hub)
//   sweeps  x <- c x + d b - d a_jh y_k
//   up      x' = d b + p x (merged at t: d b + p W_t);  x <- c x' + d b - d a_jh X_t
// The hub needs sums over the leaves: G_t = sum(-p_h a_hj d b) + sum over the
// merged (p r), P_k = sum a_hj x before sweep k, Q_t = sum a_hj x':
//   H_(t+1) = p c H_t + G_t,   y_(k+1) = y_k + d (H_L - (a_hh y_k + P_k)),
//   x_t = c X_t + d H_t - d Q_t.
// Each sum is linear in the leaves' b (the rows of A) and in the drivers before
// it (the matrix B).  k_chain_sim runs the leaf recurrences for a unit b and
// for each unit driver; k_chain_z solves the hub's recurrence for each sum; the
// product of the two is V.
// ----------------------------------------------------------------------------
struct ChainDims {
    int n, L, S;  // rows of level 0, star levels above the coarsest, sweeps
    __host__ __device__ int M() const { return 2 * L + S - 1; }   // sums over the leaves
    __host__ __device__ int Z() const { return 2 * L + S - 1; }   // drivers H, y, X
    __host__ __device__ int cols() const { return Z() + L; }      // and W
    __host__ __device__ int sum_P(int k) const { return L + k - 1; }           // 1 <= k < S
    __host__ __device__ int sum_Q(int t) const { return L + S - 1 + (L - 1 - t); }
    __host__ __device__ int drv_y(int k) const { return L + k - 1; }
    __host__ __device__ int drv_X(int t) const { return L + S - 1 + t; }
    __host__ __device__ int drv_W(int t) const { return Z() + t; }
};

// Per leaf and level: d, a_jh, a_hj, p; the level a leaf is merged at (L: never;
// -1: the hub).  Per level the hub's a_hh, d, p (hs[4 t ..]).
struct ChainParams {
    double *d, *jh, *hj, *p;  // (L + 1) x n each
    double *c;
    int *mrg;
    double *hs;
};

__device__ __forceinline__ int row_find(const int *ci, int s, int e, int j) {
    while (s < e) {
        const int m = (s + e) >> 1;
        if (ci[m] < j) s = m + 1; else e = m;
    }
    return s;
}

__global__ void __launch_bounds__(kBlock)
k_chain_params(ChainDims D, const ChainLevel *__restrict__ tab, ChainParams P) {
    const int j = blockIdx.x * kBlock + threadIdx.x;
    if (j <= D.L) {  // the hub of level j
        const ChainLevel T = tab[j];
        const int e = T.rp[T.hub + 1], q = row_find(T.ci, T.rp[T.hub], e, T.hub);
        P.hs[4 * j] = q < e && T.ci[q] == T.hub ? T.v[q] : 0.0;
        P.hs[4 * j + 1] = T.dinv[T.hub];
        P.hs[4 * j + 2] = j < D.L ? T.p[T.hub] : 0.0;
    }
    if (j >= D.n) return;
    int r = j, mrg = D.L;
    for (int t = 0; t <= D.L; ++t) {
        const ChainLevel T = tab[t];
        if (r == T.hub) {
            mrg = -1;  // (only at t = 0: a leaf that joins the hub stops below)
            break;
        }
        double ajj = 0.0, ajh = 0.0;
        for (int q = T.rp[r]; q < T.rp[r + 1]; ++q) {
            if (T.ci[q] == r) ajj = T.v[q];
            else ajh = T.v[q];
        }
        const int he = T.rp[T.hub + 1], hq = row_find(T.ci, T.rp[T.hub], he, r);
        const size_t o = (size_t)t * D.n + j;
        const double d = T.dinv[r];
        P.d[o] = d;
        P.c[o] = 1.0 - d * ajj;
        P.jh[o] = ajh;
        P.hj[o] = hq < he && T.ci[hq] == r ? T.v[hq] : 0.0;
        if (t == D.L) break;
        const int a = T.agg[r];
        P.p[o] = T.p[r];
        if (a == tab[t + 1].hub) {
            mrg = t;
            break;
        }
        r = a;
    }
    P.mrg[j] = mrg;
}

// Leaf recurrences for one input (blockIdx.y): 0 = the leaf's own b = 1 (sums
// go to A, the result to delta), 1 + i = driver i = 1 (the sums over the
// workgroup's leaves to Bp, the result to V; W_t: to vw of the leaves merged at
// t).  Own: the inputs that enter on the way down and need every level's b.
template <bool Own>
__global__ void __launch_bounds__(kBlock)
k_chain_sim(ChainDims D, ChainParams P, int col0, double *__restrict__ A, double *__restrict__ delta,
            double *__restrict__ V, double *__restrict__ vw, double *__restrict__ Bp) {
    extern __shared__ double acc[];  // sums of this driver: M x waves
    constexpr int NW = kBlock / 64;
    const int col = col0 + blockIdx.y, drv = col - 1;
    const int j = blockIdx.x * kBlock + threadIdx.x, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int n = D.n, L = D.L, M = D.M();
    const int mrg = j < n ? P.mrg[j] : -1;
    const size_t jj = j < n ? j : 0;
    for (int m = threadIdx.x; m < M * NW; m += kBlock) acc[m] = 0.0;
    __syncthreads();
    auto emit = [&](int m, double v) {
        if (col == 0) {
            if (j < n) A[(size_t)m * n + j] = v;
        } else {
            v = group_sum<64>(v);
            if (lane == 0) acc[m * NW + wv] = v;
        }
    };
    double bt[Own ? kMaxLevels : 1];
    double b = Own && col == 0 && mrg >= 0 ? 1.0 : 0.0, x = 0.0;
    if (Own) {
        for (int t = 0; t < L; ++t) {
            const size_t o = (size_t)t * n + jj;
            bt[t] = b;
            double out = 0.0;
            if (t <= mrg) {
                const double d = P.d[o], hu = drv == t && col > 0 ? P.hs[4 * t + 1] : 0.0;
                const double r = P.c[o] * b - (P.jh[o] * hu);
                const double pr = P.p[o] * r;
                out = -(P.hs[4 * t + 2] * (P.hj[o] * (d * b)));
                if (t == mrg) out += pr;
                b = t == mrg ? 0.0 : pr;
            }
            if (col == 0 || t >= drv) emit(t, out);
        }
        bt[Own ? L : 0] = b;
    }
    {
        const size_t o = (size_t)L * n + jj;
        const bool live = mrg == L;
        const double d = live ? P.d[o] : 0.0, c = live ? P.c[o] : 0.0, jh = live ? P.jh[o] : 0.0,
                     hj = live ? P.hj[o] : 0.0;
        const double db = d * b;
        for (int k = 0; k < D.S; ++k) {
            if (k > 0) emit(D.sum_P(k), hj * x);
            const double y = col > 0 && k > 0 && drv == D.drv_y(k) ? 1.0 : 0.0;
            x = (c * x + db) - d * (jh * y);
        }
        if (!live) x = 0.0;
    }
    for (int t = L - 1; t >= 0; --t) {
        const size_t o = (size_t)t * n + jj;
        double out = 0.0;
        if (t <= mrg) {
            const double d = P.d[o], p = P.p[o], jh = P.jh[o];
            const double db = Own ? d * bt[t] : 0.0;
            const double W = col > 0 && drv == D.drv_W(t) ? 1.0 : 0.0, X = col > 0 && drv == D.drv_X(t) ? 1.0 : 0.0;
            const double xp = db + p * (t == mrg ? W : x);
            out = P.hj[o] * xp;
            x = (P.c[o] * xp + db) - d * (jh * X);
        }
        emit(D.sum_Q(t), out);
    }
    if (j < n) {
        if (col == 0) delta[j] = x;
        else if (drv < D.Z()) V[(size_t)drv * n + j] = x;
        else if (mrg == drv - D.Z()) vw[j] = x;
    }
    if (col == 0) return;
    __syncthreads();
    for (int m = threadIdx.x; m < M; m += kBlock) {
        double s = acc[m * NW];
        for (int w = 1; w < NW; ++w) s += acc[m * NW + w];
        Bp[((size_t)drv * gridDim.x + blockIdx.x) * M + m] = s;
    }
}

// B[drv][m] = sum over the workgroups of k_chain_sim, in order
__global__ void __launch_bounds__(kBlock)
k_chain_bsum(int M, int nb, const double *__restrict__ Bp, double *__restrict__ B) {
    const int drv = blockIdx.x;
    for (int m = threadIdx.x; m < M; m += kBlock) {
        const double *p = Bp + (size_t)drv * nb * M + m;
        double s = 0.0;
#pragma unroll 8
        for (int b = 0; b < nb; ++b) s += p[(size_t)b * M];
        B[(size_t)drv * M + m] = s;
    }
}

// The hub's recurrence for one unit input (blockIdx.x: 0 = H_0 = 1, 1 + m =
// the sum m over the leaves' own right-hand sides = 1), one wave: lane m % 64
// holds the sums m, m + 64, ..., and every driver, once known, is added to
// them at once.  Zm[i][input]: driver i; Zm[cols][input]: x of the hub.
constexpr int kChainLanes = 3;  // sums per lane: M <= 2 * 62 + 31 <= 192
__global__ void __launch_bounds__(64)
k_chain_z(ChainDims D, const double *__restrict__ hs, const double *__restrict__ B, double *__restrict__ Zm) {
    const int in = blockIdx.x, lane = threadIdx.x, M = D.M(), R = M + 1;
    double acc[kChainLanes];
#pragma unroll
    for (int r = 0; r < kChainLanes; ++r) acc[r] = in > 0 && lane + 64 * r == in - 1 ? 1.0 : 0.0;
    auto sum = [&](int m) {
        double v = acc[0];
        if (m >= 64) v = m >= 128 ? acc[2] : acc[1];
        return __shfl(v, m & 63, 64);
    };
    auto drive = [&](int i, double z) {
        if (lane == 0) Zm[(size_t)i * R + in] = z;
#pragma unroll
        for (int r = 0; r < kChainLanes; ++r)
            if (lane + 64 * r < M) acc[r] += B[(size_t)i * M + lane + 64 * r] * z;
    };
    double H[kMaxLevels];
    double h = in == 0 ? 1.0 : 0.0;
    for (int t = 0; t < D.L; ++t) {
        H[t] = h;
        drive(t, h);
        const double c = 1.0 - hs[4 * t + 1] * hs[4 * t];
        h = hs[4 * t + 2] * (c * h) + sum(t);
    }
    double y = 0.0;
    for (int k = 0; k < D.S; ++k) {
        if (k > 0) drive(D.drv_y(k), y);
        const double P = k > 0 ? sum(D.sum_P(k)) : 0.0;
        y = y + hs[4 * D.L + 1] * (h - (hs[4 * D.L] * y + P));
    }
    double x = y;
    for (int t = D.L - 1; t >= 0; --t) {
        const double ahh = hs[4 * t], d = hs[4 * t + 1], p = hs[4 * t + 2];
        drive(D.drv_W(t), x);
        const double X = d * H[t] + p * x;
        const double Q = sum(D.sum_Q(t));  // (the drivers before it: X_t enters after the product)
        drive(D.drv_X(t), X);
        x = X + d * (H[t] - (ahh * X + Q));
    }
    if (lane == 0) Zm[(size_t)D.cols() * R + in] = x;
}

// V[e][j] of the operator: the leaves' responses to the drivers times the
// drivers' responses to input e.  kVB inputs per thread, so each response is
// read once per kVB of them.
constexpr int kVB = 16;
__global__ void __launch_bounds__(kBlock)
k_chain_v(ChainDims D, const int *__restrict__ mrg, const double *__restrict__ V, const double *__restrict__ vw,
          const double *__restrict__ Zm, double *__restrict__ out) {
    const int j = blockIdx.x * kBlock + threadIdx.x, e0 = blockIdx.y * kVB, n = D.n, R = D.M() + 1;
    if (j >= n) return;
    const int mg = mrg[j];
    double s[kVB];
#pragma unroll
    for (int u = 0; u < kVB; ++u) s[u] = 0.0;
    if (mg < 0) {
        for (int u = 0; u < kVB && e0 + u < R; ++u) s[u] = Zm[(size_t)D.cols() * R + e0 + u];
    } else {
        for (int i = 0; i < D.Z(); ++i) {
            const double v = V[(size_t)i * n + j];
#pragma unroll
            for (int u = 0; u < kVB; ++u) s[u] += v * Zm[(size_t)i * R + min(e0 + u, R - 1)];
        }
        if (mg < D.L) {
            const double v = vw[j];
            for (int u = 0; u < kVB && e0 + u < R; ++u) s[u] += v * Zm[(size_t)(D.Z() + mg) * R + e0 + u];
        }
    }
    for (int u = 0; u < kVB && e0 + u < R; ++u) out[(size_t)(e0 + u) * n + j] = s[u];
}

// T = diag(delta) + V A^T as a dense n x n row-major matrix (small chains that
// go into the folded operator); column e = 0 of A is the hub's unit vector.
__global__ void __launch_bounds__(kBlock)
k_chain_dense(int n, int M, int hub, const double *__restrict__ A, const double *__restrict__ V,
              const double *__restrict__ delta, double *__restrict__ T) {
    const long long idx = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (idx >= (long long)n * n) return;
    const int i = (int)(idx / n), j = (int)(idx % n);
    double s = j == hub ? V[i] : 0.0;
    for (int m = 0; m < M; ++m) s += V[(size_t)(m + 1) * n + i] * A[(size_t)m * n + j];
    T[idx] = s + (i == j ? delta[i] : 0.0);
}

// First pass: E_m = sum_j A[m][j] b_j, one sum and kChainChunk rows per
// workgroup (partials in chunk order).  A pass over A once: bandwidth from the
// caches (87 sums over 39,001 rows are 27 MB).  All sums of a chunk go to one XCD,
// one after the other, so that its b comes from beyond the L2 once (3,000,000
// rows, coarsest star alone: cycle 264 -> 232 us).
constexpr int kChainU = kChainChunk / kBlock;
template <typename VB>
__global__ void __launch_bounds__(kBlock)
k_chain_sums(int n, int M, int nch, const double *__restrict__ A, const VB *__restrict__ b, double *__restrict__ E,
             const double *__restrict__ done) {
    const int l = xcd_block(blockIdx.x, gridDim.x), ch = l / M, m = l % M;
    const double *a = A + (size_t)m * n;
    double av[kChainU], bv[kChainU];
#pragma unroll
    for (int u = 0; u < kChainU; ++u) {
        const int j = ch * kChainChunk + u * kBlock + threadIdx.x;
        av[u] = j < n ? a[j] : 0.0;
        bv[u] = j < n ? (double)b[j] : 0.0;
    }
    double s[1] = {0.0};
#pragma unroll
    for (int u = 0; u < kChainU; ++u) s[0] += av[u] * bv[u];
    __shared__ double lds[16];
    block_sum<1>(s, lds);
    // (the solve-ended flag is tested before the store only: its load overlaps the sum)
    if (threadIdx.x == 0 && !(done && *done != 0.0)) E[(size_t)m * nch + ch] = s[0];
}

// The sums from their partials, one wave each (more than kChainFew chunks).  The
// cycle of a coarsest star of 1,000,000 rows: 341 us with every workgroup of the
// second pass adding 19 x 245 partials, 94 with this launch; 40 levels of as many
// rows 1049 -> 430.
__global__ void __launch_bounds__(64)
k_chain_fin(int nch, const double *__restrict__ E, double *__restrict__ Es, const double *__restrict__ done) {
    const int m = blockIdx.x, lane = threadIdx.x;
    double s = 0.0;
#pragma unroll 4
    for (int c = lane; c < nch; c += 64) s += E[(size_t)m * nch + c];
    s = group_sum<64>(s);
    if (lane == 0 && !(done && *done != 0.0)) Es[m] = s;
}

// Second pass: x = delta b + V E.  64 rows per workgroup, its four waves
// taking a quarter of the columns each (one thread per row would leave fewer
// workgroups than CUs); every workgroup first adds the sums' partials.
template <typename VB, typename VX>
__global__ void __launch_bounds__(kBlock)
k_chain_apply(int n, int M, int nch, int hub, const double *__restrict__ V, const double *__restrict__ delta,
              const double *__restrict__ E, const VB *__restrict__ b, VX *__restrict__ x,
              const double *__restrict__ done) {
    constexpr int NW = kBlock / 64;
    __shared__ double e[kChainLanes * 64 + 1];
    __shared__ double red[NW][64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int j = blockIdx.x * 64 + lane, jc = min(j, n - 1);
    if (threadIdx.x <= M) {
        double s = 0.0;
        if (threadIdx.x == 0) {
            s = (double)b[hub];
        } else {
            const double *p = E + (size_t)(threadIdx.x - 1) * nch;
            for (int c = 0; c < nch; ++c) s += p[c];
        }
        e[threadIdx.x] = s;
    }
    __syncthreads();
    double s = 0.0;
#pragma unroll 8
    for (int m = wv; m <= M; m += NW) s += V[(size_t)m * n + jc] * e[m];
    red[wv][lane] = s;
    __syncthreads();
    if (wv == 0 && j < n && !(done && *done != 0.0)) {
        double t = delta[j] * (double)b[j];
#pragma unroll
        for (int w = 0; w < NW; ++w) t += red[w][lane];
        x[j] = (VX)t;
    }
}

}  // namespace

void launch_star_find(hipStream_t s, int n, const int *rp, const int *ci, int *out) {
    hipLaunchKernelGGL(k_star_find, dim3(blocks_for(n)), dim3(kBlock), 0, s, n, rp, ci, out);
}

void launch_star_verify(hipStream_t s, int n, const int *rp, const int *ci, const double *v, int hub, int *out) {
    hipLaunchKernelGGL(k_star_verify, dim3(blocks_for(n)), dim3(kBlock), 0, s, n, rp, ci, v, hub, out);
}

int star_blocks(int n) { return blocks_for(n); }

void launch_star_best(hipStream_t s, int n, const double *v, const double *w, int hub, int *hub_out, double *pc,
                      int *pi) {
    hipLaunchKernelGGL(k_star_best, dim3(star_blocks(n)), dim3(kBlock), 0, s, n, v, w, hub, hub_out, pc, pi);
}

void launch_star_sweep(hipStream_t s, const StarSweep &S) {
    hipLaunchKernelGGL(k_star_sweep, dim3(star_blocks(S.nf)), dim3(kBlock), 0, s, S);
}

void launch_star_dinv(hipStream_t s, const ChainLevel *tab, int nlev, int nmax, double *part) {
    const int nb = star_blocks(nmax);
    hipLaunchKernelGGL(k_star_dinv, dim3(nb, nlev), dim3(kBlock), 0, s, tab, part);
    hipLaunchKernelGGL(k_star_dhub, dim3(nlev), dim3(kBlock), 0, s, tab, part, nb);
}

int chain_sums(int L, int sweeps) { return ChainDims{0, L, sweeps}.M(); }

// scratch doubles of launch_chain_build
size_t chain_scratch(int n, int L, int sweeps) {
    const ChainDims D{n, L, sweeps};
    const size_t nb = blocks_for(n), M = D.M(), cols = D.cols();
    return 5 * (size_t)(L + 1) * n + (size_t)n + 4 * (size_t)(L + 1) + (size_t)D.Z() * n + n + cols * nb * M +
           cols * M + (cols + 1) * (M + 1) + 64;
}

void launch_chain_build(hipStream_t s, const ChainLevel *tab, int n, int L, int sweeps, double *scratch, double *A,
                        double *V, double *delta) {
    const ChainDims D{n, L, sweeps};
    const int nb = blocks_for(n), M = D.M();
    double *at = scratch;
    auto take = [&](size_t c) {
        double *p = at;
        at += c;
        return p;
    };
    ChainParams P;
    const size_t ln = (size_t)(L + 1) * n;
    P.d = take(ln);
    P.jh = take(ln);
    P.hj = take(ln);
    P.p = take(ln);
    P.c = take(ln);
    P.mrg = reinterpret_cast<int *>(take(n));
    P.hs = take(4 * (size_t)(L + 1));
    double *Vd = take((size_t)D.Z() * n), *vw = take(n);
    double *Bp = take((size_t)D.cols() * nb * M), *B = take((size_t)D.cols() * M);
    double *Zm = take((size_t)(D.cols() + 1) * (M + 1));
    hipLaunchKernelGGL(k_chain_params, dim3(blocks_for(n > L ? n : L + 1)), dim3(kBlock), 0, s, D, tab, P);
    const size_t lds = sizeof(double) * (size_t)M * (kBlock / 64);
    hipLaunchKernelGGL(k_chain_sim<true>, dim3(nb, L + 1), dim3(kBlock), lds, s, D, P, 0, A, delta, Vd, vw, Bp);
    if (D.cols() > L)
        hipLaunchKernelGGL(k_chain_sim<false>, dim3(nb, D.cols() - L), dim3(kBlock), lds, s, D, P, L + 1, A, delta, Vd,
                           vw, Bp);
    if (D.cols() > 0) hipLaunchKernelGGL(k_chain_bsum, dim3(D.cols()), dim3(kBlock), 0, s, M, nb, Bp, B);
    hipLaunchKernelGGL(k_chain_z, dim3(M + 1), dim3(64), 0, s, D, P.hs, B, Zm);
    hipLaunchKernelGGL(k_chain_v, dim3(nb, (M + 1 + kVB - 1) / kVB), dim3(kBlock), 0, s, D, P.mrg, Vd, vw, Zm, V);
}

void launch_chain_dense(hipStream_t s, const ChainOp &C, double *T) {
    hipLaunchKernelGGL(k_chain_dense, dim3(blocks_for((long long)C.n * C.n)), dim3(kBlock), 0, s, C.n, C.M, C.hub, C.A,
                       C.V, C.delta, T);
}

template <typename VB, typename VX>
static void chain_t(hipStream_t s, const ChainOp &C, const VB *b, VX *x, const double *done) {
    const int nch = (C.n + kChainChunk - 1) / kChainChunk;
    if (C.M > 0)
        hipLaunchKernelGGL((k_chain_sums<VB>), dim3(nch * C.M), dim3(kBlock), 0, s, C.n, C.M, nch, C.A, b,
                           C.E, done);
    const bool fin = C.M > 0 && nch > kChainFew;
    double *Es = C.E + (size_t)C.M * nch;
    if (fin) hipLaunchKernelGGL(k_chain_fin, dim3(C.M), dim3(64), 0, s, nch, C.E, Es, done);
    hipLaunchKernelGGL((k_chain_apply<VB, VX>), dim3((C.n + 63) / 64), dim3(kBlock), 0, s, C.n, C.M, fin ? 1 : nch,
                       C.hub, C.V, C.delta, fin ? Es : C.E, b, x, done);
}

void launch_chain(hipStream_t s, const ChainOp &C, const void *b, void *x, int b_f64, int x_f64, const double *done) {
    if (b_f64 && x_f64) chain_t<double, double>(s, C, (const double *)b, (double *)x, done);
    else chain_t<float, float>(s, C, (const float *)b, (float *)x, done);
}

}  // namespace bcm
