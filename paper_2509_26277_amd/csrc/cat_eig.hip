// The leading eigenpairs of a symmetric D x D matrix in double precision, for the PCA front-end (p of D directions).
//
//   1. Householder tridiagonalisation: below 64 one workgroup with the matrix in registers (k_eig_small), for 64 <= D <= 1024 one
//      launch whose workgroups pass the products of a column on through memory (k_eig_grid), otherwise one launch per column
//      (k_eig_step).  Each is a chain of D steps bound by latencies.
//   2. The p largest eigenvalues of the tridiagonal matrix T by multisection on Sturm counts (k_eig_bisect).
//   3. Their vectors from the two-sided factorisation of T - lambda I, or by inverse iteration from pseudo-random starts where
//      eigenvalues all but coincide (k_eig_invit), made orthogonal where they lie close together (k_eig_ortho).
//   4. The reflections applied to the p vectors, last one first (k_eig_back), sign and rounding.
//
// Against one-sided Jacobi on all D rows (cat_pca.hip, which remains for more than kEigMaxP directions and for callers
// that ask for a number of sweeps) it does 4/3 D^3 flops instead of about 12 * 6 D^3.
// Measured at D = 1000, p = 50 (a whole cat_pca_fit on 65536 rows): 56.3 ms with the sweeps,
// 4.3 ms here, 1.3 of it the covariance and 2.5 the tridiagonalisation (one launch per column: 4.6), 0.16 ms the eigenvalues,
// 0.05 ms their vectors, 0.29 ms the reflections.
#include "cat_eig.h"

#include <atomic>
#include <type_traits>

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

// ---- all columns in one launch (64 <= n <= 1024) ------------------------------------------------------------------------
// A chain of n - 1 dependent steps: what bounds it is what one step takes from the last product of one workgroup to the first
// of the next.  As a launch per column that is 4.6 us at n = 1000 (the launch, the loads, three sums); here G workgroups keep
// their rows of the matrix (i = blockIdx + G r) in registers from the first column to the last and pass each other two doubles
// a row and step through memory: 2.5 us (n = 500: 1.9, 250: 1.6; 1.4 of the 2.5 the instructions of a step, which every
// workgroup issues for its own copy of the vectors).  1000 x 1000: 4.55 -> 2.48 ms, 256 x 256: 0.88 -> 0.41.
//
// Step k, with the reflection k - 1 (v, tau) and p = A v known for the thread's columns j = tid + T m:
//   sum 1: p . v over the workgroup; w = tau p - (tau^2 / 2)(p . v) v; x = row k of A - v w^T - w v^T
//   own rows: A -= v w^T + w v^T; acc_i = sum over j > k + 1 of A[i][j] x[j];  the owner of row k + 1 hands it on at once
//   sum 2: the acc_i and |x|^2; the acc_i are handed on; beta, tau, v = scale x + e_{k+1} meanwhile, from |x|^2
//   wait for all acc_i and row k + 1; p_i = A[k+1][i] + scale acc_i (A is symmetric)
// Two barriers a step; the square root and the quotients run while the products travel.
//
// Handing on: a double goes as two 8-byte words, each half of it in the upper and the number of the step in the lower 32
// bits, so a word says by itself whether it is there: relaxed device-scope atomics, no fences, no counters.  The products go to
// eight copies, each read by an eighth of the workgroups (one copy for all of them: 3.2 us a step; handing the row on a step
// earlier: 3.5).  Two slots are used in turn.  A workgroup writes a slot again at step k + 2, after it has read the
// products of step k + 1 of all workgroups that have rows left, and those were made after their workgroups had read the slot at
// the end of step k; a workgroup leaves after the step before its last row becomes a pivot row, and does not read any more
// then.  The owner of the last row stays to the end and writes V, d, e, tau.
//
// The workgroups wait for each other, so all of them must be resident: at most 128 of at most 8 waves and 128 registers, two to
// a CU, so that four calls at once still fit on 256 CUs (stream_holds_grid).  Should other work keep some of them out for longer
// than `patience` looks at the words (0.2 us each, 0.4 for two columns a thread), the waiting ones raise *fail and leave, and
// k_eig_whole, which the matrix in memory was left unchanged for, does the columns in one workgroup.  Every wait ends.  The
// patience is 20 .. 40 ms, 10^4 steps and more: longer than this library's longest launches, and not much beside what giving up
// costs (a whole cat_pca_fit of 2000 rows, ms, the grid / given up at once: D = 256: 0.6 / 3.2; 512: 1.3 / 19; 768: 2.3 / 69;
// 1000: 3.1 / 190; 1024: 3.1 / 200).  Looks and not time: a wave that was itself taken off the chip meanwhile has not waited for
// the others (and with time added up in this loop D = 256 took 3 % longer).
constexpr int kGridMin = 64, kGridMax = 1024;
// rows of V, from the last one up, whose entries before the diagonal carry the words, and how many entries of each
__host__ __device__ static inline int32_t grid_ring_rows(int32_t copies) { return 2 * (4 + 4 * copies); }
__host__ __device__ static inline int32_t grid_ring_width(int32_t n, int32_t copies) { return n - grid_ring_rows(copies) - 4; }
static inline int32_t grid_copies(int32_t n) { return n < 160 ? 1 : 8; }  // (below, two rows of V would not hold n words)

typedef unsigned long long u64;
__device__ __forceinline__ void pass_on(u64* at, int next, double v, uint32_t step) {
    const u64 b = (u64)__double_as_longlong(v);
    __hip_atomic_store(at, (b << 32) | step, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(at - next, (b & 0xFFFFFFFF00000000ull) | step, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void pass_half(u64* at, double v, int half, uint32_t step) {
    const u64 b = (u64)__double_as_longlong(v);
    __hip_atomic_store(at, (half ? b & 0xFFFFFFFF00000000ull : b << 32) | step, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u64 peek(const u64* at) { return __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ double passed(u64 a, u64 b) { return __longlong_as_double((long long)((b & 0xFFFFFFFF00000000ull) | (a >> 32))); }

// the value that the lane permutation brings (the whole double)
template <int CTRL>
__device__ __forceinline__ double dpp_get(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xFFFFFFFFll), CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
// sums of R values (2, 4 or 8) over the 16 lanes of a row: halves of the row take halves of the values while there are several.
// Lane l of the row ends with value l >> log2(16 / R).
template <int R>
__device__ __forceinline__ double row_sums(const double (&a)[R], int lane) {
    double h[R];
#pragma unroll
    for (int u = 0; u < R; u++) h[u] = a[u];
    const bool b3 = lane & 8, b2 = lane & 4, b1 = lane & 2;
#pragma unroll
    for (int u = 0; u < R / 2; u++) h[u] = (b3 ? h[u + R / 2] : h[u]) + dpp_get<0x140>(b3 ? h[u] : h[u + R / 2]);
    if (R >= 4) {
#pragma unroll
        for (int u = 0; u < R / 4; u++) h[u] = (b2 ? h[u + R / 4] : h[u]) + dpp_get<0x141>(b2 ? h[u] : h[u + R / 4]);
    } else {
        h[0] = dpp_add<0x141>(h[0]);
    }
    if (R >= 8) h[0] = (b1 ? h[1] : h[0]) + dpp_get<0x4E>(b1 ? h[0] : h[1]);
    else h[0] = dpp_add<0x4E>(h[0]);
    return dpp_add<0xB1>(h[0]);
}

template <int T, int C, int R>  // threads, columns per thread, rows per workgroup
__global__ __launch_bounds__(T, T / 128) void k_eig_grid(const double* __restrict__ W, double* V, int64_t ld, int32_t n,
                                                        double* __restrict__ d, double* __restrict__ e, double* __restrict__ tau,
                                                        int32_t copies, int32_t patience, uint32_t* fail) {
    constexpr int NW = T / kWave, kParts = T / 16;
    constexpr int kEvery = R == 8 ? 1 : R == 4 ? 2 : 3;  // log2(16 / R)
    __shared__ double s_v[T * C], s_p[T * C];
    __shared__ double s_part[R][kParts];
    __shared__ double s_red[NW], s_ss[NW];
    __shared__ double s_x0;
    __shared__ int s_fail;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int g = blockIdx.x, G = gridDim.x;
    const int last = g + (n - 1 - g) / G * G;  // the last row of this workgroup
    const bool writer = last == n - 1;
    // Arrays of n words, two rows of V each: halves of the pivot rows (two slots), then of the products (two slots, copies)
    const int next = 2 * (int)ld, width = grid_ring_width(n, copies);
    auto word = [&](int i) { return (u64*)V + (i < width ? (n - 1) * (int)ld + i : (n - 2) * (int)ld + i - width); };
    u64* at[C];
#pragma unroll
    for (int m = 0; m < C; m++) at[m] = word(tid + T * m < n ? tid + T * m : 0);
    // 16 threads add up a row's product: each then hands on one half to one copy
    u64* const mine = word(g + G * (tid >> 4) < n ? g + G * (tid >> 4) : 0) - (4 + (tid & 15)) * next;
    const int copy = 4 + 2 * (g & (copies - 1));
    double a[R][C], v[C], p[C], col[C];
#pragma unroll
    for (int m = 0; m < C; m++) {
        const int j = tid + T * m;
        col[m] = j < n ? W[j] : 0.0;
        v[m] = p[m] = 0.0;
#pragma unroll
        for (int r = 0; r < R; r++) {
            const int i = g + G * r;
            a[r][m] = i < n && j < n ? W[(int64_t)i * ld + j] : 0.0;
        }
    }
    if (tid == 0) s_fail = 0;
    auto total = [&](const double (&part)[NW]) {
        double t[NW];
#pragma unroll
        for (int h = 0; h < NW; h++) t[h] = part[h];
#pragma unroll
        for (int o = NW / 2; o > 0; o /= 2)
#pragma unroll
            for (int h = 0; h < o; h++) t[h] += t[h + o];
        return t[0];
    };
    double tp = 0.0;
    for (int k = 0;; k++) {
        const uint32_t step = (uint32_t)k + 1u;
        u64 in[C][4];
        bool miss[C];
        auto ask = [&](int m) {
            const u64* pa = at[m] - (copy + 2 * copies * (k & 1)) * next;
            const u64* pr = at[m] - 2 * (k & 1) * next;
            in[m][0] = peek(pa);
            in[m][1] = peek(pa - next);
            in[m][2] = peek(pr);
            in[m][3] = peek(pr - next);
        };
#pragma unroll
        for (int m = 0; m < C; m++) {
            const int j = tid + T * m;
            miss[m] = j > k && j < n && last > k + 1;
            in[m][0] = in[m][1] = in[m][2] = in[m][3] = 0;
        }
        double pv = 0.0;
#pragma unroll
        for (int m = 0; m < C; m++) {
            const int j = tid + T * m;
            s_v[j] = v[m];
            s_p[j] = p[m];
            pv = fma(p[m], v[m], pv);
        }
        pv = wave_total(pv);
        if (lane == 0) s_red[wave] = pv;
        __syncthreads();
        if (s_fail) return;
        pv = total(s_red);
        const double c = 0.5 * tp * tp * pv;
        const double wk = tp * s_p[k] - c;  // v[k] = 1 (column 0: nothing to apply, all zero)
        double w[C], x[C], ss = 0.0, acc[R];
#pragma unroll
        for (int m = 0; m < C; m++) {
            const int j = tid + T * m;
            w[m] = tp * p[m] - c * v[m];
            x[m] = j >= k && j < n ? col[m] - (v[m] * wk + w[m]) : 0.0;
            if (j == k && writer) d[k] = x[m];
            if (j == k + 1) s_x0 = x[m];
            if (j <= k + 1) x[m] = 0.0;
            ss = fma(x[m], x[m], ss);
        }
        // the rows and columns that are left: all of a register's, or of the upper half of them (rows and columns before k change
        // nothing: there v and w are zero)
        auto rows = [&](auto from) {
            constexpr int R0 = decltype(from)::value ? R / 2 : 0, C0 = decltype(from)::value ? C / 2 : 0;
            double vr[R], pr[R];
#pragma unroll
            for (int r = R0; r < R; r++) {
                const int i = g + G * r < n ? g + G * r : 0;
                vr[r] = s_v[i];
                pr[r] = s_p[i];
            }
#pragma unroll
            for (int r = 0; r < R0; r++) acc[r] = 0.0;
#pragma unroll
            for (int r = R0; r < R; r++) {
                const double wr = c * vr[r] - tp * pr[r];
                acc[r] = 0.0;
#pragma unroll
                for (int m = C0; m < C; m++) {
                    a[r][m] = fma(-vr[r], w[m], fma(wr, v[m], a[r][m]));
                    acc[r] = fma(a[r][m], x[m], acc[r]);
                }
            }
        };
        if (k >= T * (C / 2) && k >= G * (R / 2)) rows(std::true_type());
        else rows(std::false_type());
        if ((k + 1 - g) % G == 0) {
#pragma unroll
            for (int r = 0; r < R; r++) {
                if (g + G * r != k + 1) continue;  // uniform
#pragma unroll
                for (int m = 0; m < C; m++) {
                    const int j = tid + T * m;
                    if (j > k && j < n) pass_on(at[m] - 2 * (k & 1) * next, next, a[r][m], step);
                }
            }
        }
        {
            const double h = row_sums<R>(acc, lane);
            if ((lane & ((1 << kEvery) - 1)) == 0) s_part[(lane & 15) >> kEvery][wave * 4 + (lane >> 4)] = h;
        }
        ss = wave_total(ss);
        if (lane == 0) s_ss[wave] = ss;
        __syncthreads();
        if (wave < (16 * R + kWave - 1) / kWave) {  // 16 threads add up a row
            double h = 0.0;
            if (tid < 16 * R) {
#pragma unroll
                for (int q = 0; q < kParts; q += 16) h += s_part[tid >> 4][q + (tid & 15)];
            }
            h = dpp_add<0x140>(dpp_add<0x141>(dpp_add<0x4E>(dpp_add<0xB1>(h))));
            const int i = g + G * (tid >> 4);
            if ((tid & 15) < 2 * copies && tid < 16 * R && i > k && i < n) pass_half(mine - 2 * copies * (k & 1) * next, h, tid & 1, step);
        }
        ss = total(s_ss);
        const double x0 = s_x0;
        double beta = x0, tk = 0.0, scale = 0.0;
        if (ss > 0.0) {
            const double nrm = sqrt(fma(x0, x0, ss));
            beta = x0 >= 0.0 ? -nrm : nrm;
            tk = (beta - x0) / beta;
            scale = 1.0 / (x0 - beta);
        }
#pragma unroll
        for (int m = 0; m < C; m++) {
            const int j = tid + T * m;
            v[m] = j == k + 1 ? 1.0 : x[m] * scale;
        }
        // an answer that comes too early costs another round through memory: 64 x 8 cycles from here, the products are there
        __builtin_amdgcn_s_sleep(8);
#pragma unroll
        for (int m = 0; m < C; m++)
            if (miss[m]) ask(m);
#pragma unroll
        for (int m = 0; m < C; m++) {
            const int j = tid + T * m;
            if (writer && j > k && j < n) V[(int64_t)k * ld + j] = v[m];
        }
        if (writer && tid == 0) {
            e[k] = beta;
            tau[k] = tk;
        }
        if (last <= k + 1) {
            if (writer) {  // k = n - 2: the last reflection is none
#pragma unroll
                for (int r = 0; r < R; r++) {
#pragma unroll
                    for (int m = 0; m < C; m++)
                        if (g + G * r == n - 1 && tid + T * m == n - 1) d[n - 1] = a[r][m];
                }
            }
            return;
        }
        for (uint32_t spins = 0;; spins++) {
            bool any = false;
#pragma unroll
            for (int m = 0; m < C; m++) {
                miss[m] = miss[m] && ((uint32_t)in[m][0] != step || (uint32_t)in[m][1] != step || (uint32_t)in[m][2] != step ||
                                      (uint32_t)in[m][3] != step);
                any = any || miss[m];
            }
            if (patience >= 0 && !__any(any)) break;
            if (patience < 0 || (spins & 63u) == 63u) {
                if ((int32_t)spins > patience || __hip_atomic_load(fail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u) {
                    if (lane == 0) {
                        __hip_atomic_store(fail, (uint32_t)CAT_PCA_ALONE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        s_fail = 1;
                    }
                    break;
                }
            }
#pragma unroll
            for (int m = 0; m < C; m++)
                if (miss[m]) ask(m);
        }
        tp = tk;
#pragma unroll
        for (int m = 0; m < C; m++) {
            const int j = tid + T * m;
            const bool live = j > k && j < n;
            col[m] = live ? passed(in[m][2], in[m][3]) : 0.0;
            p[m] = live ? fma(scale, passed(in[m][0], in[m][1]), col[m]) : 0.0;
        }
    }
}

// The same columns by one workgroup on the matrix in memory, if *fail says that k_eig_grid gave up; otherwise it notes there that
// the grid has done them (for the tests; nothing reads it).
constexpr int kWholeT = 1024;
__global__ __launch_bounds__(kWholeT) void k_eig_whole(double* W, double* __restrict__ V, int64_t ld, int32_t n, double* __restrict__ d,
                                                       double* __restrict__ e, double* __restrict__ tau, uint32_t* fail) {
    const bool done = *fail == 0u;
    __syncthreads();  // all have read it
    if (done) {
        if (threadIdx.x == 0) *fail = CAT_PCA_GRID;
        return;
    }
    constexpr int NW = kWholeT / kWave;
    __shared__ double s_v[kGridMax], s_w[kGridMax], s_red[2][NW];
    __shared__ double s_x0;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    for (int k = 0; k < n; k++) {
        const bool live = tid > k && tid < n;
        const double x = tid >= k && tid < n ? W[(int64_t)k * ld + tid] : 0.0;
        if (tid == k) d[k] = x;
        if (k + 1 >= n) return;
        if (tid == k + 1) s_x0 = x;
        double ss = wave_total(tid > k + 1 ? x * x : 0.0);
        if (lane == 0) s_red[0][wave] = ss;
        __syncthreads();
        ss = 0.0;
#pragma unroll
        for (int h = 0; h < NW; h++) ss += s_red[0][h];
        const double x0 = s_x0;
        double beta = x0, tk = 0.0, scale = 0.0;
        if (ss > 0.0) {
            const double nrm = sqrt(fma(x0, x0, ss));
            beta = x0 >= 0.0 ? -nrm : nrm;
            tk = (beta - x0) / beta;
            scale = 1.0 / (x0 - beta);
        }
        const double v = tid == k + 1 ? 1.0 : live ? x * scale : 0.0;
        if (live) V[(int64_t)k * ld + tid] = v;
        if (tid == 0) {
            e[k] = beta;
            tau[k] = tk;
        }
        s_v[tid] = v;
        __syncthreads();
        for (int i = k + 1 + wave; i < n; i += NW) {
            double s = 0.0;
            for (int j = k + 1 + lane; j < n; j += kWave) s = fma(W[(int64_t)i * ld + j], s_v[j], s);
            s = wave_total(s);
            if (lane == 0) s_w[i] = s;
        }
        __syncthreads();
        const double p = live ? s_w[tid] : 0.0;
        double pv = wave_total(p * v);
        if (lane == 0) s_red[1][wave] = pv;
        __syncthreads();
        pv = 0.0;
#pragma unroll
        for (int h = 0; h < NW; h++) pv += s_red[1][h];
        s_w[tid] = tk * p - 0.5 * tk * tk * pv * v;
        __syncthreads();
        for (int i = k + 1 + wave; i < n; i += NW) {
            const double vi = s_v[i], wi = s_w[i];
            for (int j = k + 1 + lane; j < n; j += kWave) W[(int64_t)i * ld + j] -= vi * s_w[j] + wi * s_v[j];
        }
        __syncthreads();
    }
}

// All columns by one workgroup that holds the matrix in registers, below the sizes the grid is for: lane i of wave q has columns
// 16 q .. 16 q + 15 of row i.  The matrix is symmetric, so column k is row k, which its lane lays in LDS; every wave makes the
// reflection for itself, the waves' shares of the products A v meet in LDS.  Two barriers a column: a chain of latencies, LDS and
// the divisions of the reflection: 72 us at n = 60 (a launch per column 226; A x requested before the norm is known, 76).
constexpr int kSmallT = 256, kSmallC = kGridMin / (kSmallT / kWave);
__global__ __launch_bounds__(kSmallT) void k_eig_small(const double* __restrict__ W, double* __restrict__ V, int64_t ld, int32_t n,
                                                       double* __restrict__ d, double* __restrict__ e, double* __restrict__ tau) {
    constexpr int NW = kSmallT / kWave, C = kSmallC;
    __shared__ __align__(16) double s_x[kGridMin], s_p[NW][kGridMin], s_v[NW][kGridMin], s_w[NW][kGridMin];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    double a[C];
#pragma unroll
    for (int j = 0; j < C; j++) a[j] = lane < n && C * wave + j < n ? W[(int64_t)lane * ld + C * wave + j] : 0.0;
    for (int k = 0; k < n; k++) {
        if (lane == k) {
#pragma unroll
            for (int j = 0; j < C; j++) s_x[C * wave + j] = a[j];
        }
        __syncthreads();
        const double x = s_x[lane];
        if (tid == k) d[k] = x;
        if (k + 1 >= n) return;
        const double x0 = s_x[k + 1];
        const double ss = wave_total(lane > k + 1 ? x * x : 0.0);
        double beta = x0, tk = 0.0, scale = 0.0;
        if (ss > 0.0) {
            const double nrm = sqrt(fma(x0, x0, ss));
            beta = x0 >= 0.0 ? -nrm : nrm;
            tk = (beta - x0) / beta;
            scale = 1.0 / (x0 - beta);
        }
        const double v = lane == k + 1 ? 1.0 : lane > k + 1 ? x * scale : 0.0;
        if (wave == 0 && lane > k && lane < n) V[(int64_t)k * ld + lane] = v;
        if (tid == 0) {
            e[k] = beta;
            tau[k] = tk;
        }
        s_v[wave][lane] = v;
        __builtin_amdgcn_wave_barrier();  // (a wave's own copy; LDS serves it in order)
        double vj[C], s0 = 0.0, s1 = 0.0;
#pragma unroll
        for (int j = 0; j < C; j++) vj[j] = s_v[wave][C * wave + j];
#pragma unroll
        for (int j = 0; j < C; j += 2) {
            s0 = fma(a[j], vj[j], s0);
            s1 = fma(a[j + 1], vj[j + 1], s1);
        }
        s_p[wave][lane] = s0 + s1;
        __syncthreads();
        double p = 0.0;
#pragma unroll
        for (int h = 0; h < NW; h++) p += s_p[h][lane];
        p = lane > k ? p : 0.0;
        const double pv = wave_total(p * v);
        const double w = tk * p - 0.5 * tk * tk * pv * v;
        s_w[wave][lane] = w;
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < C; j++) a[j] -= v * s_w[wave][C * wave + j] + w * vj[j];
    }
}

// ---- eigenvalues of the tridiagonal matrix ---------------------------------------------------------------------------
// Workgroup j finds the j-th largest eigenvalue: 256 shifts at a time inside the interval that holds it, the number of
// eigenvalues below each shift from the sign changes of the leading minors of T - x I, 8 bits of the interval a round.
// Bound by the serial chain of a count (n terms).  The minors follow P' = (d - x) P - e^2 P'' and need no division: the chain is
// one fused multiply-add a term (the pivots, quotients of minors, cost a reciprocal each: D = 1000, p = 50: 547 us, 159 so).
// T is scaled by a power of two to a norm of 1 .. 2, so that minors grow by less than 2^4 a term, and the pair at hand is
// brought back to 1 .. 2 after every eight terms.  Where it has all but vanished by then (a shift that is an eigenvalue of a
// leading block which nothing couples to the rest), the eight terms are taken again with each minor kept away from zero.
// out: lambda[j]; tnorm[0] = a bound of |T| (workgroup 0).
constexpr int kBisT = 256;
constexpr int kBisU = 8;  // terms between two rescalings
// terms of a chain as its loop reads them: whole groups, and one requested ahead of the last
__host__ __device__ static inline int32_t minor_terms(int32_t n) { return (n + kBisU - 1) / kBisU * kBisU + kBisU; }
__global__ __launch_bounds__(kBisT) void k_eig_bisect(const double* __restrict__ d, const double* __restrict__ e, int32_t n,
                                                      double* __restrict__ lambda, double* __restrict__ tnorm) {
    extern __shared__ double2 s_t[];  // diagonal entry, squared off-diagonal one (entry i couples i - 1 and i); whole groups + 1
    __shared__ double s_lo[kBisT / kWave], s_hi[kBisT / kWave];
    __shared__ int s_first[2];
    double lo = 1.7e308, hi = -1.7e308;
    for (int i = threadIdx.x; i < n; i += kBisT) {
        const double el = i > 0 ? e[i - 1] : 0.0, er = i + 1 < n ? e[i] : 0.0, di = d[i];
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
    const int up = norm > 1e-307 && norm < 1e300 ? -ilogb(norm) : 0;  // (a norm of zero, or none at all: as it is)
    for (int i = threadIdx.x; i < minor_terms(n); i += kBisT) {
        const double di = i < n ? ldexp(d[i], up) : 8.0;  // past the end: no change of sign
        const double el = i > 0 && i < n ? ldexp(e[i - 1], up) : 0.0;
        s_t[i] = make_double2(di, el * el);
    }
    const double margin = 4.0 * kEps * ldexp(norm, up);
    lo = ldexp(lo, up) - margin;
    hi = ldexp(hi, up) + margin;
    const double tiny = kEps * kEps;
    const int want = n - (int)blockIdx.x;  // the eigenvalue is the smallest x with at least `want` eigenvalues below or at it
    __syncthreads();
    for (int round = 0; round < 7; round++) {  // 56 bits of 4 |T| at most: past the last one that a double holds of |T|
        const double step = (hi - lo) * (1.0 / (kBisT + 1));
        const double x = lo + step * (double)(threadIdx.x + 1);
        int below = 0;
        double a = 0.0, b = 1.0;  // the last two minors
        double2 t[kBisU];
#pragma unroll
        for (int u = 0; u < kBisU; u++) t[u] = s_t[u];
        for (int i = 0; i < n; i += kBisU) {
            double2 nx[kBisU];
#pragma unroll
            for (int u = 0; u < kBisU; u++) nx[u] = s_t[i + kBisU + u];
            const double a0 = a, b0 = b;
            uint32_t signs = (uint32_t)__double2hiint(b) >> 31;  // one bit per minor, the latest lowest
#pragma unroll
            for (int u = 0; u < kBisU; u++) {
                const double c = fma(t[u].x - x, b, -(t[u].y * a));
                signs = __builtin_amdgcn_alignbit(signs, (uint32_t)__double2hiint(c), 31);
                a = b;
                b = c;
            }
            double m = fmax(fabs(a), fabs(b));
            if (__builtin_expect(__ballot(!(m > 1e-200)) != 0ull, 0)) {  // uniform
                a = a0;
                b = b0;
                signs = (uint32_t)__double2hiint(b) >> 31;
#pragma unroll 1
                for (int u = 0; u < kBisU; u++) {
                    const double2 tu = s_t[i + u];
                    double c = fma(tu.x - x, b, -(tu.y * a));
                    const double ref = b != 0.0 ? b : a;
                    if (!(fabs(c) >= tiny * fabs(ref))) c = -tiny * ref;
                    signs = __builtin_amdgcn_alignbit(signs, (uint32_t)__double2hiint(c), 31);
                    a = b;
                    b = c;
                }
                m = fmax(fabs(a), fabs(b));
            }
            below += __popc((signs ^ (signs >> 1)) & ((1u << kBisU) - 1u));
            const int ex = -__builtin_amdgcn_frexp_exp(m);
            a = __builtin_amdgcn_ldexp(a, ex);
            b = __builtin_amdgcn_ldexp(b, ex);
#pragma unroll
            for (int u = 0; u < kBisU; u++) t[u] = nx[u];
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
    if (threadIdx.x == 0) lambda[blockIdx.x] = ldexp(0.5 * (lo + hi), -up);
}

// ---- eigenvectors of the tridiagonal matrix --------------------------------------------------------------------------
// Workgroup (one wave) j.  An eigenvalue away from its neighbours: the pivots of T - lambda_j I eliminated from the top (D+) and
// from the bottom (D-), the row k where they meet with the smallest remainder g_k = D+_k + D-_k - (d_k - lambda_j), and the
// vector (T - lambda_j I) z = g_k e_k, z_k = 1, which is a product of multipliers on either side of k (Parlett and Dhillon,
// Linear Algebra Appl. 267, 1997).  Its residual is g_k / |z|, of the order of eps |T|; that is checked.
// Bound by the chain of the pivots: the two directions run in the even and the odd lanes, on minors as in k_eig_bisect (the
// pivots are their quotients, taken side by side afterwards), the products are a scan.  Two solves with the factors of
// a pivoted elimination, serial chains all, took 505 us for 50 vectors of 1000; 51 so.
// An eigenvalue with a neighbour within 1e-10 |T| (or a residual that is too large) takes those two solves, from a start of
// its own: the vectors of a multiple eigenvalue have to be independent.
constexpr double kInvGap = 1e-10;
__device__ void eig_invit_lu(double* s_lu, const double* __restrict__ d, const double* __restrict__ e, int32_t n, double lam,
                             double norm, int j, double* __restrict__ Z, int64_t ld);
// bytes: two directions of (diagonal entry, squared coupling), of minors and the minor before each group; two multipliers
__host__ __device__ static inline int32_t twist_at(int32_t i) { return i + (i >> 4); }  // (lanes walk 16 entries apart and more)
static inline size_t twist_lds_bytes(int32_t n) {
    return (size_t)minor_terms(n) * 32 + (size_t)minor_terms(n) * 16 + (size_t)minor_terms(n) / kBisU * 16 + (size_t)(twist_at(n) + 1) * 16;
}
__global__ __launch_bounds__(kWave) void k_eig_invit(const double* __restrict__ d, const double* __restrict__ e, int32_t n, int32_t p,
                                                     const double* __restrict__ lambda, const double* __restrict__ tnorm,
                                                     double* __restrict__ Z, int64_t ld) {
    extern __shared__ double2 s_iv[];
    const int lane = threadIdx.x, j = blockIdx.x;
    const double lam = lambda[j], norm = tnorm[0];
    const double gap = fmin(j > 0 ? lambda[j - 1] - lam : norm, j + 1 < p ? lam - lambda[j + 1] : norm);
    bool done = false;  // uniform
    if (gap > kInvGap * norm && norm > 1e-280 && norm < 1e280) {
        const int terms = minor_terms(n);
        double2* T = s_iv;                          // [direction][term]
        double* P = (double*)(T + 2 * terms);       // [direction][term]: minors
        double* B = P + 2 * terms;                  // [direction][group]: the minor before the group, as scaled there
        double* L = B + 2 * (terms / kBisU);        // multipliers up to k
        double* R = L + twist_at(n) + 1;            //   and from k on
        const int up = -ilogb(norm);
        const double ls = ldexp(lam, up);
        for (int i = lane; i < terms; i += kWave) {
            const bool ok = i < n;
            const int r = ok ? n - 1 - i : 0;  // the row of term i from the bottom
            const double et = ok && i > 0 ? ldexp(e[i - 1], up) : 0.0, eb = ok && i > 0 ? ldexp(e[r], up) : 0.0;
            T[i] = make_double2(ok ? ldexp(d[i], up) - ls : 1.0, et * et);
            T[terms + i] = make_double2(ok ? ldexp(d[r], up) - ls : 1.0, eb * eb);
        }
        __syncthreads();
        {
            const int dir = lane & 1;
            const double2* Td = T + dir * terms;
            double* Pd = P + dir * terms;
            double* Bd = B + dir * (terms / kBisU);
            const double tiny = kEps * kEps;
            double a = 0.0, b = 1.0;
            double2 t[kBisU];
#pragma unroll
            for (int u = 0; u < kBisU; u++) t[u] = Td[u];
            for (int i = 0; i < n; i += kBisU) {
                double2 nx[kBisU];
#pragma unroll
                for (int u = 0; u < kBisU; u++) nx[u] = Td[i + kBisU + u];
                const double b0 = b;
                double out[kBisU];
#pragma unroll
                for (int u = 0; u < kBisU; u++) {
                    double c = fma(t[u].x, b, -(t[u].y * a));
                    const double least = -tiny * b;  // no pivot below tiny |T|
                    c = fabs(c) >= fabs(least) ? c : least;
                    out[u] = c;
                    a = b;
                    b = c;
                }
                if (lane < 2) {
                    Bd[i / kBisU] = b0;
#pragma unroll
                    for (int u = 0; u < kBisU; u++) Pd[i + u] = out[u];
                }
                const int ex = -__builtin_amdgcn_frexp_exp(fmax(fabs(a), fabs(b)));
                a = __builtin_amdgcn_ldexp(a, ex);
                b = __builtin_amdgcn_ldexp(b, ex);
#pragma unroll
                for (int u = 0; u < kBisU; u++) t[u] = nx[u];
            }
        }
        __syncthreads();
        double gbest = 1.7e308;
        int k = n;
        for (int i = lane; i < n; i += kWave) {
            const int r = n - 1 - i;
            const double c = P[i], b = i % kBisU ? P[i - 1] : B[i / kBisU];
            const double cb = P[terms + r], bb = r % kBisU ? P[terms + r - 1] : B[terms / kBisU + r / kBisU];
            const double g = fabs(c / b + cb / bb - T[i].x);
            if (g < gbest) {
                gbest = g;
                k = i;
            }
            L[twist_at(i)] = i + 1 < n ? -ldexp(e[i], up) * (b / c) : 0.0;
            R[twist_at(i)] = i > 0 ? -ldexp(e[i - 1], up) * (bb / cb) : 0.0;
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const double og = __shfl_xor(gbest, o, kWave);
            const int ok = __shfl_xor(k, o, kWave);
            if (og < gbest || (og == gbest && ok < k)) {
                gbest = og;
                k = ok;
            }
        }
        __syncthreads();
        // z_i = L_i .. L_(k-1) above k, R_(k+1) .. R_i below: every lane a run of entries, the runs joined by scans
        const int C = (n + kWave - 1) / kWave, c0 = lane * C, c1 = min(c0 + C, n);
        double pl = 1.0, pr = 1.0;
        for (int i = c0; i < c1; i++) {
            if (i < k) pl *= L[twist_at(i)];
            if (i > k) pr *= R[twist_at(i)];
        }
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const double vl = __shfl_down(pl, o, kWave), vr = __shfl_up(pr, o, kWave);
            if (lane + o < kWave) pl *= vl;
            if (lane >= o) pr *= vr;
        }
        pl = __shfl_down(pl, 1, kWave);
        pr = __shfl_up(pr, 1, kWave);
        if (lane == kWave - 1) pl = 1.0;
        if (lane == 0) pr = 1.0;
        double big = 0.0;
        for (int i = c1 - 1; i >= c0; i--) {
            if (i < k) L[twist_at(i)] = pl = pl * L[twist_at(i)];
            if (i == k) L[twist_at(i)] = 1.0;
        }
        for (int i = c0; i < c1; i++)
            if (i > k) L[twist_at(i)] = pr = pr * R[twist_at(i)];
        for (int i = c0; i < c1; i++) big = fmax(big, fabs(L[twist_at(i)]));
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) big = fmax(big, __shfl_xor(big, o, kWave));
        const double sc = big > 0.0 ? 1.0 / big : 0.0;
        __syncthreads();
        double ss = 0.0;
        for (int i = lane; i < n; i += kWave) {
            const double v = L[twist_at(i)] * sc;
            ss = fma(v, v, ss);
        }
        ss = wave_total(ss);
        // Residual g_k / |z| in units of the scaled norm (1 .. 2).  Up to 16 eps sqrt(n): ten times the largest seen (6e-15 at n =
        // 1000, on spectra in close pairs, graded, of noise, of constant bands); over a gap of 1e-6, from which on nothing
        // makes the vectors orthogonal (k_eig_ortho), it turns one by 1e-7 at most, about the rounding of the float32 result.
        done = ss >= 1.0 && ss <= 1e6 && gbest * sc <= 16.0 * kEps * sqrt((double)n) * sqrt(ss);
        if (done) {
            const double nf = sc / sqrt(ss);
            for (int i = lane; i < n; i += kWave) Z[(int64_t)j * ld + i] = L[twist_at(i)] * nf;
        }
        __syncthreads();
    }
    if (!done) eig_invit_lu((double*)s_iv, d, e, n, lam, norm, j, Z, ld);
}

// T - lambda_j I = P L U with partial pivoting, then two solves from a pseudo-random start.  The recurrences are
// serial; every lane runs them on the same values, their operands are requested ahead of the chain, lane 0 stores.
// Z: row j receives the unit vector.
constexpr int kInvArrays = 5;
static inline size_t invit_lds_bytes(int32_t n) { return (size_t)n * (kInvArrays * 8 + 4); }
__device__ void eig_invit_lu(double* s_lu, const double* __restrict__ d, const double* __restrict__ e, int32_t n, double lam,
                             double norm, int j, double* __restrict__ Z, int64_t ld) {
    double* u0 = s_lu;      // 1 / diagonal of U (before that: the diagonal of T)
    double* u1 = u0 + n;    // first super-diagonal of U (before that: of T)
    double* u2 = u1 + n;    // second super-diagonal of U
    double* l = u2 + n;     // multipliers
    double* x = l + n;      // the vector
    int* sw = (int*)(x + n);  // rows i and i + 1 were interchanged
    const int lane = threadIdx.x;
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

// One workgroup: vector by vector, the components along the vectors before it whose eigenvalues lie within 1e-6 |T| are
// taken out (Gram-Schmidt against all of them at once, twice).  Without it such components are of the size of
// eps |T| / gap: 2e-10 at most where the gap is larger than that (measured, n = 64 .. 1000; the result is rounded to float32, 6e-8),
// everything where the eigenvalue is multiple.
// (50 vectors of 1000, nearly all of them within 1e-4 |T| of the next: 289 us with that as the line, 9 with 1e-6.)
constexpr int kOrtT = 1024;
__global__ __launch_bounds__(kOrtT) void k_eig_ortho(double* __restrict__ Z, int64_t ld, int32_t n, int32_t p,
                                                     const double* __restrict__ lambda, const double* __restrict__ tnorm) {
    __shared__ double s_x[kEigMaxD];
    __shared__ double s_c[kEigMaxP];
    __shared__ double s_red[kOrtT / kWave];
    __shared__ double s_lam[kEigMaxP];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const double tol = 1e-6 * tnorm[0];
    for (int i = tid; i < p; i += kOrtT) s_lam[i] = lambda[i];
    __syncthreads();
    int g = 0;  // first vector of the run of close eigenvalues that reaches j
    for (int j = 1; j < p; j++) {
        const double lj = s_lam[j];
        while (g < j && s_lam[g] - lj > tol) g++;  // uniform
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
// One wave per vector: the reflections n - 3 .. 0 in turn.  Bound by the latency of a reflection's entries and of its sum over
// the wave: AHEAD reflections are on their way while one is applied (one: 1000 x 1000, 628 us; four: 280), and the quarters of
// a row that lie before a reflection's first entry are neither read nor used.
template <int NI, int M0, int AHEAD>  // entries per lane; the first that the reflections from .. to (descending) can reach
__device__ __forceinline__ void eig_back_run(const double* __restrict__ V, int64_t ld, int32_t n, const double* __restrict__ tau,
                                             int from, int to, int lane, double (&y)[NI]) {
    constexpr int M = NI - M0;
    if (from < to) return;
    double r[AHEAD][M], t[AHEAD];
    auto load = [&](int k, double (&x)[M], double& tk) {
        const int kc = k > to ? k : to;  // past the last: that one again, never used
        tk = tau[kc];
#pragma unroll
        for (int m = 0; m < M; m++) {
            const int i = lane + kWave * (M0 + m);
            x[m] = V[(int64_t)kc * ld + (i < n ? i : n - 1)];  // positions up to k and past the end: dropped where used
        }
    };
    auto apply = [&](int k, double (&v)[M], double tk) {
        double s0 = 0.0, s1 = 0.0;
#pragma unroll
        for (int m = 0; m < M; m++) {
            const int i = lane + kWave * (M0 + m);
            v[m] = (i > k && i < n) ? v[m] : 0.0;
            if (m & 1) s1 = fma(v[m], y[M0 + m], s1);
            else s0 = fma(v[m], y[M0 + m], s0);
        }
        const double s = tk * wave_total(s0 + s1);
#pragma unroll
        for (int m = 0; m < M; m++) y[M0 + m] = fma(-s, v[m], y[M0 + m]);
    };
#pragma unroll
    for (int u = 0; u < AHEAD; u++) load(from - u, r[u], t[u]);
    for (int k = from; k >= to; k -= AHEAD) {
#pragma unroll
        for (int u = 0; u < AHEAD; u++) {
            if (k - u >= to) apply(k - u, r[u], t[u]);  // uniform
            load(k - u - AHEAD, r[u], t[u]);
        }
    }
}
template <int NI>  // entries per lane: n <= 64 NI
__global__ __launch_bounds__(kWave) void k_eig_back(const double* __restrict__ Z, const double* __restrict__ V, int64_t ld, int32_t n,
                                                    const double* __restrict__ tau, const double* __restrict__ lambda,
                                                    float* __restrict__ comps, double* __restrict__ evals) {
    const int lane = threadIdx.x, j = blockIdx.x;
    constexpr int Q = NI / 4, AHEAD = NI > 16 ? 2 : 4;
    double y[NI];
#pragma unroll
    for (int m = 0; m < NI; m++) {
        const int i = lane + kWave * m;
        y[m] = i < n ? Z[(int64_t)j * ld + i] : 0.0;
    }
    // reflection k reaches entries from k + 1 on: from 64 Q s - 1 on the first Q s of a lane stay as they are
    auto last = [&](int s) { return kWave * Q * s - 1; };
    eig_back_run<NI, 3 * Q, AHEAD>(V, ld, n, tau, n - 3, last(3), lane, y);
    eig_back_run<NI, 2 * Q, AHEAD>(V, ld, n, tau, min(n - 3, last(3) - 1), last(2), lane, y);
    eig_back_run<NI, Q, AHEAD>(V, ld, n, tau, min(n - 3, last(2) - 1), last(1), lane, y);
    eig_back_run<NI, 0, AHEAD>(V, ld, n, tau, min(n - 3, last(1) - 1), 0, lane, y);
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

static std::atomic<int32_t> g_grid_patience{CAT_PCA_PATIENCE};  // cat_debug_pca_patience

// Whether the workgroups of k_eig_grid will all be resident on this stream, once others have left: 128 of them at two to a CU
// take 64 CUs, so CUs / 64 calls fit at once; from 128 CUs on.  A stream that may not use all CUs of its device has a launch per
// column: which of the XCDs its CUs belong to, to each of which the dispatcher gives an eighth of the workgroups, is not known.
// (A graph may be replayed on another stream than it was captured on; there the bounded wait has to do.)
static cat_status stream_holds_grid(hipStream_t st, bool* yes) {
    static std::atomic<int> ncu[16];
    int dev = 0;
    CAT_HIP_TRY(hipGetDevice(&dev));
    int v = dev < 16 ? ncu[dev].load() : 0;
    if (v == 0) {
        CAT_HIP_TRY(hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev));
        if (dev < 16) ncu[dev].store(v);
    }
    *yes = v >= 128;
    if (!*yes) return CAT_OK;
    uint32_t mask[32] = {};  // (the handles of the default streams are no objects of their own: they have the device's mask)
    const bool named = st != nullptr && st != hipStreamLegacy && st != hipStreamPerThread;
    if (hipExtStreamGetCUMask(named ? st : nullptr, 32, mask) != hipSuccess) {  // not known: a launch per column will do
        (void)hipGetLastError();
        *yes = false;
        return CAT_OK;
    }
    int own = 0;
    for (uint32_t word : mask) own += __builtin_popcount(word);
    *yes = own >= v;
    return CAT_OK;
}

// the word that says whether a wait was given up: past the words that are passed on, before the diagonal, so that no row of V
// reaches it
static inline int64_t grid_fail_entry(int64_t ld, int32_t n) {
    const int64_t low = n - grid_ring_rows(grid_copies(n));
    return low * ld + (low - 2);
}
size_t eig_route_at(int64_t ld, int64_t D) {
    return D >= kGridMin && D <= kGridMax ? (size_t)grid_fail_entry(ld, (int32_t)D) * 8 : 0;
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
    bool grid_fits = false;
    if (D >= kGridMin && D <= kGridMax)
        if (cat_status s = stream_holds_grid(st, &grid_fits); s != CAT_OK) return s;
    if (grid_fits) {
        const int32_t copies = grid_copies(D), low = D - grid_ring_rows(copies);
        if (cat_status s = launch_fill_zero(V + (int64_t)low * ld, (size_t)(D - low) * ld * 8, st); s != CAT_OK) return s;
        uint32_t* fail = (uint32_t*)(V + grid_fail_entry(ld, D));
        const int32_t patience = g_grid_patience.load(std::memory_order_relaxed);
#define CAT_EIG_GRID(T, C, R, G) hipLaunchKernelGGL((k_eig_grid<T, C, R>), dim3(G), dim3(T), 0, st, W, V, ld, D, d, e, tau, copies, patience, fail)
        if (D <= 128) CAT_EIG_GRID(256, 1, 2, 64);
        else if (D <= 256) CAT_EIG_GRID(256, 1, 2, 128);
        else if (D <= 512) CAT_EIG_GRID(512, 1, 4, 128);
        else CAT_EIG_GRID(512, 2, 8, 128);
#undef CAT_EIG_GRID
        CAT_LAUNCH_CHECK("k_eig_grid");
        hipLaunchKernelGGL(k_eig_whole, dim3(1), dim3(kWholeT), 0, st, W, V, ld, D, d, e, tau, fail);
        CAT_LAUNCH_CHECK("k_eig_whole");
    } else if (D < kGridMin) {
        hipLaunchKernelGGL(k_eig_small, dim3(1), dim3(kSmallT), 0, st, W, V, ld, D, d, e, tau);
        CAT_LAUNCH_CHECK("k_eig_small");
    } else {
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
    }
    hipLaunchKernelGGL(k_eig_bisect, dim3((unsigned)p), dim3(kBisT), (size_t)minor_terms(D) * 16, st, d, e, D, lambda, tnorm);
    CAT_LAUNCH_CHECK("k_eig_bisect");
    const size_t lds = invit_lds_bytes(D) > twist_lds_bytes(D) ? invit_lds_bytes(D) : twist_lds_bytes(D);  // 139 KB at D = 2048
    if (lds > 64 * 1024)
        CAT_HIP_TRY(hipFuncSetAttribute((const void*)k_eig_invit, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL(k_eig_invit, dim3((unsigned)p), dim3(kWave), lds, st, d, e, D, p, lambda, tnorm, W, ld);
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

extern "C" cat_status cat_debug_pca_patience(int64_t looks) {
    cat::g_grid_patience.store(looks < 0 ? -1 : looks < (1 << 30) ? (int32_t)looks : 1 << 30);
    return CAT_OK;
}
