// The leading eigenpairs of a symmetric D x D matrix in double precision, for the PCA front-end (p of D directions).
//
//   1. Householder tridiagonalisation, one launch per column (k_eig_step): D launches, at D = 1000 each bound by its latencies
//      (the launch, one round of loads, two sums over a workgroup) and not by the rows it reads and writes, 2 x 8 D^2 bytes
//      at most (16 MB; 67 MB at D = 2048).
//   2. The p largest eigenvalues of the tridiagonal matrix T by multisection on Sturm counts (k_eig_bisect).
//   3. Their vectors by inverse iteration on T from pseudo-random starts (k_eig_invit), made orthogonal where
//      eigenvalues lie close together (k_eig_ortho).
//   4. The reflections applied to the p vectors, last one first (k_eig_back), sign and rounding.
//
// Against one-sided Jacobi on all D rows (cat_pca.hip, which remains for more than kEigMaxP directions and for callers
// that ask for a number of sweeps) it does 4/3 D^3 flops instead of about 12 * 6 D^3, and D launches instead of 3 D.
// Measured at D = 1000, p = 50 (a whole cat_pca_fit on 65536 rows, 1.5 ms of it the covariance): 56.3 ms with the sweeps,
// 8.1 ms here; of that 4.6 ms the tridiagonalisation (3.5 us a launch over the last 256 columns, 6.2 us over the first),
// 0.55 ms the eigenvalues, 0.8 ms their vectors, 0.63 ms the reflections.
#include "cat_eig.h"

namespace cat {

constexpr int kEigT = 256;                 // threads of a tridiagonalisation step
constexpr int kEigWaves = kEigT / kWave;
constexpr double kEps = 2.220446049250313e-16;

// ---- one column of the tridiagonalisation --------------------------------------------------------------------------
// State before launch k: rows and columns i, j >= k of W hold the matrix after the reflections 0 .. k - 2; the reflection
// k - 1 (v = row k - 1 of V, unit entry at position k, and tau[k - 1]) has been chosen and p_in = W v computed, but not
// applied: A' = A - v w^T - w v^T with w = tau p - (tau^2 / 2)(p . v) v.  Every workgroup computes column k of A' from
// row k of A (the matrix is symmetric), with it d[k], e[k] and reflection k; then it updates its own rows, stores them
// and leaves p_out = A' v_k for them.  All of a workgroup's loads are issued together at the start; thread t holds the
// columns k0 + t + 256 m of every vector and of up to NI rows in registers (k0: k rounded down to 64 bytes).  Only
// workgroup 0 writes V, d, e, tau.  Grid: min(256, n - k0) workgroups, row k0 + blockIdx + 256 r; n - k0 <= 256 NI.
template <int NI>
__global__ __launch_bounds__(kEigT) void k_eig_step(double* __restrict__ W, double* __restrict__ V, int64_t ld, int32_t n, int32_t k,
                                                    const double* __restrict__ p_in, double* __restrict__ p_out,
                                                    double* __restrict__ d, double* __restrict__ e, double* __restrict__ tau) {
    __shared__ double s_red[2][kEigWaves];
    __shared__ double s_rows[NI][kEigWaves];
    __shared__ double s_x0;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int k0 = k & ~7;
    const bool first = k == 0;
    const double* vprev = V + (int64_t)(first ? 0 : k - 1) * ld;  // (first: any readable row, its values are dropped)
    const double* prow = first ? W : p_in;
    const double tp = first ? 0.0 : tau[k - 1];
    const double pk = first ? 0.0 : p_in[k];
    int jc[NI];
    bool in[NI];  // column inside the trailing matrix (j >= k)
    double v[NI], p[NI], col[NI], a[NI][NI], vi[NI], pi[NI];
#pragma unroll
    for (int m = 0; m < NI; m++) {
        const int j = k0 + tid + kEigT * m;
        in[m] = j >= k && j < n;
        jc[m] = j < n ? j : n - 1;  // past the end: a valid column, dropped below
        v[m] = vprev[jc[m]];
        p[m] = prow[jc[m]];
        col[m] = W[(int64_t)k * ld + jc[m]];
    }
#pragma unroll
    for (int r = 0; r < NI; r++) {
        const int i = k0 + (int)blockIdx.x + kEigT * r;
        const int ic = (i > k && i < n) ? i : k;  // rows that are not ours to update: row k again, dropped below
#pragma unroll
        for (int m = 0; m < NI; m++) a[r][m] = W[(int64_t)ic * ld + jc[m]];
        vi[r] = vprev[ic];
        pi[r] = prow[ic];
    }
    double pv = 0.0;
#pragma unroll
    for (int m = 0; m < NI; m++) {
        if (first || !in[m]) v[m] = p[m] = 0.0;
        pv = fma(p[m], v[m], pv);
    }
    pv = wave_total(pv);
    if (lane == 0) s_red[0][wave] = pv;
    __syncthreads();
    pv = (s_red[0][0] + s_red[0][1]) + (s_red[0][2] + s_red[0][3]);
    const double c = 0.5 * tp * tp * pv;
    const double wk = tp * pk - c;  // v[k] = 1
    double w[NI], x[NI], ss = 0.0;
#pragma unroll
    for (int m = 0; m < NI; m++) {
        const int j = k0 + tid + kEigT * m;
        w[m] = tp * p[m] - c * v[m];
        x[m] = in[m] ? (first ? col[m] : col[m] - (v[m] * wk + w[m])) : 0.0;
        if (j == k && blockIdx.x == 0) d[k] = x[m];
        if (j == k + 1) s_x0 = x[m];
        if (j > k + 1) ss = fma(x[m], x[m], ss);
    }
    ss = wave_total(ss);
    if (lane == 0) s_red[1][wave] = ss;
    __syncthreads();
    if (k + 1 >= n) return;  // the last diagonal entry is written
    ss = (s_red[1][0] + s_red[1][1]) + (s_red[1][2] + s_red[1][3]);
    const double x0 = s_x0;
    double beta = x0, tk = 0.0, scale = 0.0;
    if (ss > 0.0) {
        const double nrm = sqrt(fma(x0, x0, ss));
        beta = x0 >= 0.0 ? -nrm : nrm;
        tk = (beta - x0) / beta;
        scale = 1.0 / (x0 - beta);
    }
    double vn[NI];
#pragma unroll
    for (int m = 0; m < NI; m++) {
        const int j = k0 + tid + kEigT * m;
        vn[m] = j == k + 1 ? 1.0 : (j > k + 1 && in[m] ? x[m] * scale : 0.0);
        if (blockIdx.x == 0 && j > k && j < n) V[(int64_t)k * ld + j] = vn[m];
    }
    if (blockIdx.x == 0 && tid == 0) {
        e[k] = beta;
        tau[k] = tk;
    }
    double acc[NI];
#pragma unroll
    for (int r = 0; r < NI; r++) {
        const int i = k0 + (int)blockIdx.x + kEigT * r;
        const bool mine = i > k && i < n;  // uniform
        const double vr = first ? 0.0 : vi[r], wr = first ? 0.0 : tp * pi[r] - c * vi[r];
        acc[r] = 0.0;
#pragma unroll
        for (int m = 0; m < NI; m++) {
            const double y = a[r][m] - (vr * w[m] + wr * v[m]);
            acc[r] = fma(y, vn[m], acc[r]);
            if (mine && in[m] && !first) W[(int64_t)i * ld + jc[m]] = y;
        }
    }
#pragma unroll
    for (int r = 0; r < NI; r++) {
        acc[r] = wave_total(acc[r]);
        if (lane == 0) s_rows[r][wave] = acc[r];
    }
    __syncthreads();
    if (tid < NI) {
        const int i = k0 + (int)blockIdx.x + kEigT * tid;
        if (i > k && i < n) p_out[i] = (s_rows[tid][0] + s_rows[tid][1]) + (s_rows[tid][2] + s_rows[tid][3]);
    }
}

// ---- eigenvalues of the tridiagonal matrix ---------------------------------------------------------------------------
__device__ __forceinline__ double fast_rcp(double q) {  // within a few ulp for normal q
    double r = __builtin_amdgcn_rcp(q);
    r = fma(fma(-q, r, 1.0), r, r);
    return fma(fma(-q, r, 1.0), r, r);
}
// Workgroup j finds the j-th largest eigenvalue: 256 shifts at a time inside the interval that holds it, the number of
// eigenvalues below each shift from the signs of the pivots of T - x I, 8 bits of the interval a round.  Bound by the
// serial chain of a count (n pivots, a reciprocal each).  out: lambda[j]; norm2[0] = a bound of |T| (workgroup 0).
constexpr int kBisT = 256;
__global__ __launch_bounds__(kBisT) void k_eig_bisect(const double* __restrict__ d, const double* __restrict__ e, int32_t n,
                                                      double* __restrict__ lambda, double* __restrict__ tnorm) {
    extern __shared__ double s_t[];  // n diagonal entries, then n squared off-diagonal ones (entry i couples i - 1 and i)
    __shared__ double s_lo[kBisT / kWave], s_hi[kBisT / kWave];
    __shared__ int s_first[2];
    double* s_d = s_t;
    double* s_e2 = s_t + n;
    double lo = 1.7e308, hi = -1.7e308;
    for (int i = threadIdx.x; i < n; i += kBisT) {
        const double el = i > 0 ? e[i - 1] : 0.0, er = i + 1 < n ? e[i] : 0.0, di = d[i];
        s_d[i] = di;
        s_e2[i] = el * el;
        lo = fmin(lo, di - fabs(el) - fabs(er));
        hi = fmax(hi, di + fabs(el) + fabs(er));
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        lo = fmin(lo, __shfl_xor(lo, o, kWave));
        hi = fmax(hi, __shfl_xor(hi, o, kWave));
    }
    if ((threadIdx.x & (kWave - 1)) == 0) {
        s_lo[threadIdx.x / kWave] = lo;
        s_hi[threadIdx.x / kWave] = hi;
    }
    if (threadIdx.x < 2) s_first[threadIdx.x] = kBisT;
    __syncthreads();
    lo = fmin(fmin(s_lo[0], s_lo[1]), fmin(s_lo[2], s_lo[3]));
    hi = fmax(fmax(s_hi[0], s_hi[1]), fmax(s_hi[2], s_hi[3]));
    const double norm = fmax(fabs(lo), fabs(hi));
    if (blockIdx.x == 0 && threadIdx.x == 0) tnorm[0] = norm;
    lo -= 4.0 * kEps * norm;
    hi += 4.0 * kEps * norm;
    const double tiny = fmax(kEps * kEps * norm, 1e-290);  // a pivot below this counts as a small negative one
    const int want = n - (int)blockIdx.x;  // the eigenvalue is the smallest x with at least `want` eigenvalues below or at it
    for (int round = 0; round < 8; round++) {  // 64 bits: past the last one that a double holds
        const double step = (hi - lo) * (1.0 / (kBisT + 1));
        const double x = lo + step * (double)(threadIdx.x + 1);
        int below = 0;
        double q = 1.0;
        for (int i = 0; i < n; i += 8) {  // the entries of eight pivots ahead of the chain that uses them
            double dd[8], ee[8];
#pragma unroll
            for (int u = 0; u < 8; u++) {
                const int ic = i + u < n ? i + u : n - 1;
                dd[u] = s_d[ic] - x;
                ee[u] = s_e2[ic];
            }
#pragma unroll
            for (int u = 0; u < 8; u++) {
                if (i + u < n) {  // uniform
                    q = fma(-ee[u], fast_rcp(q), dd[u]);
                    if (fabs(q) < tiny) q = -tiny;
                    below += q < 0.0 ? 1 : 0;
                }
            }
        }
        if (below >= want) atomicMin(&s_first[round & 1], (int)threadIdx.x);
        __syncthreads();
        const int f = s_first[round & 1];
        if (threadIdx.x == 0) s_first[(round & 1) ^ 1] = kBisT;
        const double nlo = f > 0 ? lo + step * (double)f : lo;
        const double nhi = f < kBisT ? lo + step * (double)(f + 1) : hi;
        lo = nlo;
        hi = nhi;
        __syncthreads();
    }
    if (threadIdx.x == 0) lambda[blockIdx.x] = 0.5 * (lo + hi);
}

// ---- eigenvectors of the tridiagonal matrix --------------------------------------------------------------------------
// Workgroup (one wave) j: T - lambda_j I = P L U with partial pivoting, then two solves from a pseudo-random start (a
// start of its own for every vector, so that the vectors of a multiple eigenvalue are independent).  The recurrences are
// serial; every lane runs them on the same values, their operands are requested ahead of the chain, lane 0 stores.
// Z: row j receives the unit vector.
constexpr int kInvArrays = 5;
static inline size_t invit_lds_bytes(int32_t n) { return (size_t)n * (kInvArrays * 8 + 4); }
__global__ __launch_bounds__(kWave) void k_eig_invit(const double* __restrict__ d, const double* __restrict__ e, int32_t n,
                                                     const double* __restrict__ lambda, const double* __restrict__ tnorm,
                                                     double* __restrict__ Z, int64_t ld) {
    extern __shared__ double s_t[];
    double* u0 = s_t;       // 1 / diagonal of U (before that: the diagonal of T)
    double* u1 = u0 + n;    // first super-diagonal of U (before that: of T)
    double* u2 = u1 + n;    // second super-diagonal of U
    double* l = u2 + n;     // multipliers
    double* x = l + n;      // the vector
    int* sw = (int*)(x + n);  // rows i and i + 1 were interchanged
    const int lane = threadIdx.x, j = blockIdx.x;
    const double lam = lambda[j], norm = tnorm[0];
    const double pert = norm > 0.0 ? kEps * norm : 1.0;  // least pivot
    for (int i = lane; i < n; i += kWave) {
        u0[i] = d[i];
        u1[i] = i + 1 < n ? e[i] : 0.0;
        x[i] = (double)(int64_t)splitmix64_at(0x5851F42D4C957F2Dull + (uint64_t)j, (uint64_t)i) * (1.0 / 9223372036854775808.0);
    }
    __syncthreads();
    {
        double a = u0[0] - lam, b = u1[0], ei = b;  // the current row, and the sub-diagonal entry below it
        double dn = u0[n > 1 ? 1 : 0], en = u1[n > 1 ? 1 : 0];
        for (int i = 0; i + 1 < n; i++) {
            const int i2 = i + 2 < n ? i + 2 : n - 1;
            const double dnn = u0[i2], enn = u1[i2];
            const double an = dn - lam;
            const bool swap = fabs(ei) > fabs(a);
            double p0 = swap ? ei : a;
            if (fabs(p0) < pert) p0 = p0 < 0.0 ? -pert : pert;
            const double r0 = 1.0 / p0;
            const double m = (swap ? a : ei) * r0;
            const double nb = swap ? -m * en : en;
            if (lane == 0) {
                u0[i] = r0;
                u1[i] = swap ? an : b;
                u2[i] = swap ? en : 0.0;
                l[i] = m;
                sw[i] = swap;
            }
            a = swap ? b - m * an : an - m * b;
            b = nb;
            ei = en;
            dn = dnn;
            en = enn;
        }
        if (fabs(a) < pert) a = a < 0.0 ? -pert : pert;
        if (lane == 0) {
            u0[n - 1] = 1.0 / a;
            u1[n - 1] = u2[n - 1] = 0.0;
        }
    }
    __syncthreads();
    for (int it = 0; it < 2; it++) {
        double cur = x[0];
        constexpr int U = 4;  // steps whose operands are requested together
        for (int i = 0; i + 1 < n; i += U) {
            double xs[U], ls[U], out[U];
            int ss[U];
#pragma unroll
            for (int u = 0; u < U; u++) {
                const int ic = i + u + 1 < n ? i + u : n - 2;
                xs[u] = x[ic + 1];
                ls[u] = l[ic];
                ss[u] = sw[ic];
            }
#pragma unroll
            for (int u = 0; u < U; u++) {
                if (i + u + 1 < n) {  // uniform
                    out[u] = ss[u] ? xs[u] : cur;
                    cur = ss[u] ? cur - ls[u] * xs[u] : xs[u] - ls[u] * cur;
                }
            }
#pragma unroll
            for (int u = 0; u < U; u++)
                if (lane == 0 && i + u + 1 < n) x[i + u] = out[u];
        }
        if (lane == 0) x[n - 1] = cur;
        __syncthreads();
        double x1 = 0.0, x2 = 0.0;  // x[i + 1], x[i + 2]
        for (int i = n - 1; i >= 0; i -= U) {
            double xs[U], a0[U], a1[U], a2[U], out[U];
#pragma unroll
            for (int u = 0; u < U; u++) {
                const int ic = i - u >= 0 ? i - u : 0;
                xs[u] = x[ic];
                a0[u] = u0[ic];
                a1[u] = u1[ic];
                a2[u] = u2[ic];
            }
#pragma unroll
            for (int u = 0; u < U; u++) {
                if (i - u >= 0) {  // uniform
                    const double v = (xs[u] - fma(a2[u], x2, a1[u] * x1)) * a0[u];
                    out[u] = v;
                    x2 = x1;
                    x1 = v;
                }
            }
#pragma unroll
            for (int u = 0; u < U; u++)
                if (lane == 0 && i - u >= 0) x[i - u] = out[u];
        }
        __syncthreads();
        // scale by the largest entry first: the solve multiplies by up to 1 / pert
        double big = 0.0;
        for (int i = lane; i < n; i += kWave) big = fmax(big, fabs(x[i]));
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) big = fmax(big, __shfl_xor(big, o, kWave));
        const double sc = big > 0.0 ? 1.0 / big : 0.0;
        double ss = 0.0;
        for (int i = lane; i < n; i += kWave) {
            const double v = x[i] * sc;
            ss = fma(v, v, ss);
        }
        ss = wave_total(ss);
        const double nf = ss > 0.0 ? sc / sqrt(ss) : 0.0;
        for (int i = lane; i < n; i += kWave) x[i] *= nf;
        __syncthreads();
    }
    for (int i = lane; i < n; i += kWave) Z[(int64_t)j * ld + i] = x[i];
}

// One workgroup: vector by vector, the components along the vectors before it whose eigenvalues lie within 1e-4 |T| are
// taken out (Gram-Schmidt against all of them at once, twice).  Inverse iteration leaves such components at the size of
// eps |T| / gap: below 1e-11 where the gap is larger than that, everything where the eigenvalue is multiple.
constexpr int kOrtT = 1024;
__global__ __launch_bounds__(kOrtT) void k_eig_ortho(double* __restrict__ Z, int64_t ld, int32_t n, int32_t p,
                                                     const double* __restrict__ lambda, const double* __restrict__ tnorm) {
    __shared__ double s_x[kEigMaxD];
    __shared__ double s_c[kEigMaxP];
    __shared__ double s_red[kOrtT / kWave];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const double tol = 1e-4 * tnorm[0];
    int g = 0;  // first vector of the run of close eigenvalues that reaches j
    for (int j = 1; j < p; j++) {
        const double lj = lambda[j];
        while (g < j && lambda[g] - lj > tol) g++;  // uniform
        if (g == j) continue;
        double* zj = Z + (int64_t)j * ld;
        for (int i = tid; i < n; i += kOrtT) s_x[i] = zj[i];
        for (int pass = 0; pass < 2; pass++) {
            __syncthreads();
            for (int v = g + wave; v < j; v += kOrtT / kWave) {
                const double* zv = Z + (int64_t)v * ld;
                double s = 0.0;
                for (int i = lane; i < n; i += kWave) s = fma(zv[i], s_x[i], s);
                s = wave_total(s);
                if (lane == 0) s_c[v] = s;
            }
            __syncthreads();
            double ss = 0.0;
            for (int i = tid; i < n; i += kOrtT) {
                double y = s_x[i];
                for (int v = g; v < j; v++) y = fma(-s_c[v], Z[(int64_t)v * ld + i], y);
                s_x[i] = y;
                ss = fma(y, y, ss);
            }
            ss = wave_total(ss);
            if (lane == 0) s_red[wave] = ss;
            __syncthreads();
            ss = 0.0;
#pragma unroll
            for (int h = 0; h < kOrtT / kWave; h++) ss += s_red[h];
            const double nf = ss > 0.0 ? 1.0 / sqrt(ss) : 0.0;
            for (int i = tid; i < n; i += kOrtT) s_x[i] *= nf;
        }
        for (int i = tid; i < n; i += kOrtT) zj[i] = s_x[i];  // (each thread the entries it has just scaled)
        __syncthreads();  // visible to the whole workgroup (stores of a workgroup to global memory are, after a barrier)
    }
}

// ---- back to the basis of the matrix, sign, output ---------------------------------------------------------------------
// One wave per vector: the reflections n - 3 .. 0 in turn, the next one's entries in flight while one is applied.
template <int NI>  // entries per lane: n <= 64 NI
__global__ __launch_bounds__(kWave) void k_eig_back(const double* __restrict__ Z, const double* __restrict__ V, int64_t ld, int32_t n,
                                                    const double* __restrict__ tau, const double* __restrict__ lambda,
                                                    float* __restrict__ comps, double* __restrict__ evals) {
    const int lane = threadIdx.x, j = blockIdx.x;
    double y[NI], v[NI];
#pragma unroll
    for (int m = 0; m < NI; m++) {
        const int i = lane + kWave * m;
        y[m] = i < n ? Z[(int64_t)j * ld + i] : 0.0;
    }
    auto load = [&](int k, double (&r)[NI]) {
#pragma unroll
        for (int m = 0; m < NI; m++) {
            const int i = lane + kWave * m;
            r[m] = V[(int64_t)k * ld + (i < n ? i : n - 1)];  // positions up to k and past the end: dropped where used
        }
    };
    int k = n - 3;
    double tk = k >= 0 ? tau[k] : 0.0;
    if (k >= 0) load(k, v);
    while (k >= 0) {
        double nx[NI];
        const int kn = k > 0 ? k - 1 : 0;
        load(kn, nx);
        const double tn = tau[kn];
        double s = 0.0;
#pragma unroll
        for (int m = 0; m < NI; m++) {
            const int i = lane + kWave * m;
            v[m] = (i > k && i < n) ? v[m] : 0.0;
            s = fma(v[m], y[m], s);
        }
        s = tk * wave_total(s);
#pragma unroll
        for (int m = 0; m < NI; m++) y[m] = fma(-s, v[m], y[m]);
#pragma unroll
        for (int m = 0; m < NI; m++) v[m] = nx[m];
        tk = tn;
        k--;
    }
    double am = -1.0;  // the first entry of largest magnitude decides the sign
    int ai = n;
    double av = 1.0;
#pragma unroll
    for (int m = 0; m < NI; m++) {
        const int i = lane + kWave * m;
        const double f = fabs(y[m]);
        if (i < n && f > am) {
            am = f;
            ai = i;
            av = y[m];
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const double om = __shfl_xor(am, o, kWave), ov = __shfl_xor(av, o, kWave);
        const int oi = __shfl_xor(ai, o, kWave);
        if (om > am || (om == am && oi < ai)) {
            am = om;
            ai = oi;
            av = ov;
        }
    }
    const double sgn = av < 0.0 ? -1.0 : 1.0;
#pragma unroll
    for (int m = 0; m < NI; m++) {
        const int i = lane + kWave * m;
        if (i < n) comps[(int64_t)j * n + i] = (float)(sgn * y[m]);
    }
    if (lane == 0 && evals) evals[j] = lambda[j];
}

cat_status launch_eig_leading(double* W, double* V, int64_t ld, int32_t D, int32_t p, double* scratch, float* comps,
                              double* evals, hipStream_t st) {
    if (D < 1 || D > kEigMaxD || p < 1 || p > D || p > kEigMaxP || ld < D)
        return set_error(CAT_ERR_UNSUPPORTED, "leading eigenpairs: D=%d p=%d", (int)D, (int)p);
    double* pb[2] = {scratch, scratch + D};
    double* d = scratch + 2 * (size_t)D;
    double* e = d + D;
    double* tau = e + D;
    double* lambda = tau + D;
    double* tnorm = pb[0];  // the products are no longer needed once the last column is done
    for (int32_t k = 0; k < D; k++) {
        const int32_t rest = D - (k & ~7);
        const dim3 grid((unsigned)(rest < 256 ? rest : 256)), block(kEigT);
#define CAT_EIG_STEP(NI) hipLaunchKernelGGL(k_eig_step<NI>, grid, block, 0, st, W, V, ld, D, k, pb[(k & 1) ^ 1], pb[k & 1], d, e, tau)
        if (rest <= 256) CAT_EIG_STEP(1);
        else if (rest <= 512) CAT_EIG_STEP(2);
        else if (rest <= 768) CAT_EIG_STEP(3);
        else if (rest <= 1024) CAT_EIG_STEP(4);
        else if (rest <= 1536) CAT_EIG_STEP(6);
        else CAT_EIG_STEP(8);
#undef CAT_EIG_STEP
        CAT_LAUNCH_CHECK("k_eig_step");
    }
    hipLaunchKernelGGL(k_eig_bisect, dim3((unsigned)p), dim3(kBisT), (size_t)D * 16, st, d, e, D, lambda, tnorm);
    CAT_LAUNCH_CHECK("k_eig_bisect");
    const size_t lds = invit_lds_bytes(D);  // 90 KB at D = 2048
    if (lds > 64 * 1024)
        CAT_HIP_TRY(hipFuncSetAttribute((const void*)k_eig_invit, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL(k_eig_invit, dim3((unsigned)p), dim3(kWave), lds, st, d, e, D, lambda, tnorm, W, ld);
    CAT_LAUNCH_CHECK("k_eig_invit");
    hipLaunchKernelGGL(k_eig_ortho, dim3(1), dim3(kOrtT), 0, st, W, ld, D, p, lambda, tnorm);
    CAT_LAUNCH_CHECK("k_eig_ortho");
#define CAT_EIG_BACK(NI) hipLaunchKernelGGL(k_eig_back<NI>, dim3((unsigned)p), dim3(kWave), 0, st, W, V, ld, D, tau, lambda, comps, evals)
    if (D <= 256) CAT_EIG_BACK(4);
    else if (D <= 512) CAT_EIG_BACK(8);
    else if (D <= 1024) CAT_EIG_BACK(16);
    else CAT_EIG_BACK(32);
#undef CAT_EIG_BACK
    CAT_LAUNCH_CHECK("k_eig_back");
    return CAT_OK;
}

}  // namespace cat
