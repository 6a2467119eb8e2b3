// Fused CAT Inferencing (Algorithm 2) with the centroid operand streamed from L2: every row is read from memory once,
// whatever the number of clusters (up to 256), and ranked with the two-part operand.
//
// k_infer (cat_infer_kernel.h) keeps the operand in registers for the whole launch; 64 clusters on rows of 4 KB make
// 512 KB of it, which no workgroup holds.  Here the rows stay on the chip and the operand passes by.  A workgroup of 8
// waves owns a tile of 16 RG rows in LDS (128 KB at most), as they are in memory.  Each wave
//   - contracts all rows of the tile against its share of the operand (8 / SC cluster shares of KW tiles of 16 clusters,
//     times SC channel shares): fragments come from L2, a batch of steps ahead of their use, each used for RG row groups;
//     fp32 rows are split into two bf16 parts as they are read from LDS.  The partial dot products go to LDS;
//   - after a barrier, ranks the centroids of its own 2 RG rows, measures rows inside the error bound of the split
//     arithmetic in double precision (row from LDS; the exact nearest centroid, lowest index on ties), and applies that
//     cluster's gamma / beta: rows from LDS, parameters and results in whole rows;
//   - stages its rows of the next tile, which it requested behind the last operand fragments: loads return in order, so
//     rows requested earlier hold up the operand (a few rows with every batch of fragments: 262144 x 2048 bf16, K = 64,
//     690 us instead of 570), and the ranking that follows needs no load.
// Two barriers per tile.  Bound by memory (one read, one write of the rows); per tile the operand costs K D 4 bytes of L2
// traffic and the parameters 8 bytes per entry.
//
// UA: rows that are not whole 16-byte groups (LDS rows start on 16 bytes all the same).  They and their parameters move in words, 64
// consecutive words per wave instruction, or in 16-byte vectors on word boundaries (wide_in_vectors).
#pragma once
#include "cat_infer_kernel.h"
#include "cat_wide.h"

namespace cat {

struct WideParams {
    const void* lq;
    void* out;
    int32_t* assign;  // nullable
    int64_t N, D, ntiles;
    int32_t K, psteps;      // clusters; 32-channel steps present in packA
    const uint16_t* packA;  // [step][ktile][part][lane][8] bf16, channels of a step in order (8 per lane group)
    const float* cnorm;     // 16 KT squared norms (padding clusters: huge)
    const float* cent;      // K x D fp32
    const float* gamma;
    const float* beta;
    float tau, tau2;
};

typedef iu32x4 __attribute__((aligned(4))) iu32x4_w;  // vectors on a word boundary
typedef if32x4 __attribute__((aligned(4))) if32x4_w;

// Unaligned rows in vectors: bf16 ones, in the instances that gain.  us per cat_apply by words / by vectors, from a graph, KT and VPR as
// there: KT = 8, VPR = 3: 112771 x 1114, K = 116: 346 / 246; 8, 4: 65554 x 1846, K = 80: 343 / 270; 8, 2: 90085 x 986, K = 85: 143 / 132 (a single tile a
// workgroup loses a little: 1950 x 594, K = 89: 24.5 / 25.6); 4, 4:
// 79833 x 1702, K = 34: 270 / 201; 2, 4: 73117 x 2044, K = 8: 213 / 182; 16, 2: 237423 x 550, K = 225: 530 / 454; 16, 3: 42587 x 1490, K = 186:
// 221 / 184.  Not 2, 3: 2282 x 1126, K = 8: 21.5 / 24.0, 44001 x 1038, K = 3: 80 / 85; 4, 3: 2825 x 1074, K = 52: 23.3 / 25.8, 37634 x
// 1042, K = 47: 78 / 81; 4, 2: 1247 x 526, K = 36: 21.3 / 23.3, 52013 x 586, K = 36: 72 / 74 (121776 x 930: 151 / 142); 8, 1: 2783 x 294, K = 77:
// 19.4 / 20.4, 144248 x 268, K = 95: 107 / 109.  And not fp32, whose parameters then lie on 4 instead of 8 bytes: 50021 x 1001, K = 50: 124 / 145;
// 100003 x 769, K = 40: 183 / 221.
constexpr bool wide_in_vectors(bool bf16, int kt, int vpr) { return bf16 && (vpr == 4 || kt == 16 || (kt == 8 && vpr >= 2)); }
constexpr int wide_row_stride(int vpr) { return vpr * 1024 + 16; }  // bytes; 16 rows apart in banks
constexpr int wide_dots_stride(int kt, int sc) { return infer_dots_stride(sc * kt * 16); }
constexpr size_t wide_lds_bytes(int kt, int sc, int rg, int vpr) {
    return (size_t)16 * rg * wide_row_stride(vpr) + (size_t)16 * rg * wide_dots_stride(kt, sc) * 4;
}

// KT: cluster tiles (K <= 16 KT).  VPR: 16-byte vectors per lane and row (rows of at most VPR KB).
template <bool BF16, int KT, int RG, int VPR, bool UA>
__global__ __launch_bounds__(kInferWaves * kWave) void k_wide(const WideParams p) {
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int KW = KT > 8 ? KT / 8 : 1, SK = KT / KW, SC = kInferWaves / SK;  // tiles per wave; cluster, channel shares
    constexpr int K16 = 16 * KT, ROWS = 16 * RG, RPW = 2 * RG;
    constexpr int XS = wide_row_stride(VPR), DS = wide_dots_stride(KT, SC);
    constexpr int EPL = BF16 ? 8 : 4;
    constexpr int STEPS = VPR * 1024 / (BF16 ? 64 : 128);  // steps of 32 channels a row has room for
    constexpr int SPW = (STEPS + SC - 1) / SC;             // of a wave
    constexpr int U = SPW < 4 ? SPW : 4;                   // steps per batch of operand fragments
    constexpr int NB = (SPW + U - 1) / U;
    constexpr int NSLOT = (K16 + kWave - 1) / kWave;
    constexpr int NL = RPW * VPR;                          // row vectors of a wave
    constexpr bool UV = UA && wide_in_vectors(BF16, KT, VPR), UW = UA && !UV;      // unaligned rows in vectors, in words
    typedef typename std::conditional<BF16, bf16_t, float>::type T;

    float* s_dots = (float*)(smem + (size_t)ROWS * XS);  // [row][channel share][cluster], rows DS apart
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int n = lane & 15, g = lane >> 4;
    const int ik = wave % SK, ic = wave / SK;

    for (int i = threadIdx.x; i < ROWS * XS / 16; i += kInferWaves * kWave) ((iu32x4*)smem)[i] = (iu32x4){0u, 0u, 0u, 0u};
    float cn[NSLOT], cmax;
    {
        float cm2 = 0.f;
#pragma unroll
        for (int j = 0; j < NSLOT; j++) {
            const int k = lane + kWave * j;
            cn[j] = k < K16 ? p.cnorm[k] : 0.f;
            if (k < p.K) cm2 = fmaxf(cm2, cn[j]);
        }
        cmax = sqrtf(wave_all(cm2, [](float a, float b) { return fmaxf(a, b); }));
    }
    // positions of this lane in a row: elements, or (UA) words; past the row a valid one, so that no load is conditional
    const int W = (int)(UA ? (BF16 ? p.D / 2 : p.D) : p.D);
    auto pos = [&](int v, int e) { return UV ? 4 * (v * kWave + lane) + e : UW ? 256 * v + 64 * e + lane : (v * kWave + lane) * EPL; };
    auto ok = [&](int v, int e) { return pos(v, e) < W; };
    // UV: the vector that a row ends in runs on into the next row, which it drops; in the last row (of the rows, or of the parameters) it
    // is loaded as the row's last four words and moved down where it is used
    auto whole = [&](int v) { return pos(v, 0) + 4 <= W; };
    auto at = [&](int v, bool last) { return whole(v) ? pos(v, 0) : ok(v, 0) ? (last ? W - 4 : pos(v, 0)) : 0; };
    auto split = [&](int v, bool last) { return last && (W & 3) != 0 && !whole(v) && ok(v, 0); };
    auto settle = [&](iu32x4& t, int v, bool last) {
        if (!split(v, last)) return;
        const int left = W & 3;  // words of the row in it
        t = left == 1 ? (iu32x4){t.w, 0u, 0u, 0u} : left == 2 ? (iu32x4){t.z, t.w, 0u, 0u} : (iu32x4){t.y, t.z, t.w, 0u};
    };
    auto settle_params = [&](if32x4& lo4, if32x4& hi4, int v, bool last) {  // (two channels a word)
        if (!split(v, last)) return;
        const int left = W & 3;
        const if32x4 a = lo4, b = hi4;
        lo4 = left == 1 ? (if32x4){b.z, b.w, 0.f, 0.f} : left == 2 ? b : (if32x4){a.z, a.w, b.x, b.y};
        hi4 = left == 3 ? (if32x4){b.z, b.w, 0.f, 0.f} : (if32x4){0.f, 0.f, 0.f, 0.f};
    };

    iu32x4 X[RPW][VPR];
    auto load_vec = [&](int64_t tile, int r, int v) {
        int64_t row = tile * ROWS + wave * RPW + r;
        row = row < p.N ? row : p.N - 1;  // rows past N (and tiles past the last) repeat the last row
        const T* x = (const T*)p.lq + row * p.D;
        if (UV) {
            X[r][v] = *(const iu32x4_w*)((const uint32_t*)x + at(v, row == p.N - 1));
        } else if (UW) {
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const int w = pos(v, e);
                X[r][v][e] = ((const uint32_t*)x)[w < W ? w : W - 1];
            }
        } else {
            const int c = pos(v, 0);
            X[r][v] = *(const iu32x4*)(x + (c < W ? c : 0));
        }
    };
    float xn2[RPW];  // |x|^2 of the wave's rows of the tile in LDS
    auto stage = [&](int64_t tile) {
#pragma unroll
        for (int r = 0; r < RPW; r++) {
            const bool last = tile * ROWS + wave * RPW + r >= p.N - 1;
            unsigned char* xr = smem + (size_t)(wave * RPW + r) * XS;
            float s = 0.f;
#pragma unroll
            for (int v = 0; v < VPR; v++) {
                if (UV) settle(X[r][v], v, last);
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    if (!ok(v, UA ? e : 0)) continue;
                    const uint32_t w = X[r][v][e];
                    if (BF16) {
                        s = fmaf(ilo_half(w), ilo_half(w), fmaf(ihi_half(w), ihi_half(w), s));
                    } else {
                        s = fmaf(__uint_as_float(w), __uint_as_float(w), s);
                    }
                    if (UW || (UV && !whole(v))) *(uint32_t*)(xr + 4 * pos(v, e)) = w;
                }
                if (UV ? whole(v) : !UA && ok(v, 0)) *(iu32x4*)(xr + 16 * (v * kWave + lane)) = X[r][v];
            }
            xn2[r] = wave_sum_all(s);
        }
    };
    // the fp32 parameters under vector v of a parameter row
    auto params = [&](const float* row, int v, bool last, if32x4& lo4, if32x4& hi4) {
        if (!UA) {
            const int c = pos(v, 0);
            const float* q = row + (c < W ? c : 0);
            lo4 = *(const if32x4*)q;
            if (BF16) hi4 = *(const if32x4*)(q + 4);
        } else if (UV) {  // (to be settled where it is used)
            const float* q = row + 2 * at(v, last);
            lo4 = *(const if32x4_w*)q;
            hi4 = *(const if32x4_w*)(q + 4);
        } else {
#pragma unroll
            for (int e = 0; e < 4; e++) {
                int w = pos(v, e);
                w = w < W ? w : W - 1;
                if (BF16) {  // two channels per word; D is even, so the pairs are 8-byte aligned
                    const if32x2 t = *(const if32x2*)(row + 2 * w);
                    if (e < 2) {
                        lo4[2 * e] = t.x;
                        lo4[2 * e + 1] = t.y;
                    } else {
                        hi4[2 * e - 4] = t.x;
                        hi4[2 * e - 3] = t.y;
                    }
                } else {
                    lo4[e] = row[w];
                }
            }
        }
    };
    // vector v of row `trow` of the tile, as loaded
    auto lds_vec = [&](int trow, int v) {
        const unsigned char* xr = smem + (size_t)trow * XS;
        iu32x4 w;
        if (UW) {
#pragma unroll
            for (int e = 0; e < 4; e++) w[e] = *(const uint32_t*)(xr + 4 * pos(v, e));
        } else {
            w = *(const iu32x4*)(xr + 16 * (v * kWave + lane));  // (past the row: zeros)
        }
        return w;
    };
    auto load_a = [&](int b, ibf16x8 (&a)[U][KW][2]) {
#pragma unroll
        for (int u = 0; u < U; u++) {
            int st = ic * SPW + b * U + u;
            st = st < p.psteps ? st : p.psteps - 1;  // past the row's channels: any fragment, against zeros
            const uint16_t* q = p.packA + ((size_t)st * KT + ik * KW) * (2 * 512) + lane * 8;
#pragma unroll
            for (int kw = 0; kw < KW; kw++)
#pragma unroll
                for (int part = 0; part < 2; part++) a[u][kw][part] = __builtin_bit_cast(ibf16x8, *(const iu32x4*)(q + (2 * kw + part) * 512));
        }
    };

    int64_t tile = blockIdx.x;
    if (tile >= p.ntiles) return;  // uniform
#pragma unroll
    for (int r = 0; r < RPW; r++)
#pragma unroll
        for (int v = 0; v < VPR; v++) load_vec(tile, r, v);
    __syncthreads();  // the zeroed rows
    stage(tile);
    __syncthreads();
    for (; tile < p.ntiles; tile += gridDim.x) {
        const int64_t next = tile + gridDim.x;
        // ---- contraction; the rows of the next tile are requested along the way ----
        {
            if32x4 acc[KW][RG][2];
#pragma unroll
            for (int kw = 0; kw < KW; kw++)
#pragma unroll
                for (int rg = 0; rg < RG; rg++) acc[kw][rg][0] = acc[kw][rg][1] = (if32x4){0.f, 0.f, 0.f, 0.f};
            ibf16x8 A[2][U][KW][2];
            load_a(0, A[0]);
            const unsigned char* xb = smem + (size_t)n * XS + (size_t)(ic * SPW) * (BF16 ? 64 : 128) + g * (BF16 ? 16 : 32);
#pragma unroll
            for (int b = 0; b < NB; b++) {
                __builtin_amdgcn_sched_barrier(0);
                if (b + 1 < NB) load_a(b + 1, A[(b + 1) & 1]);
                if (b == NB - 1) {
#pragma unroll
                    for (int l = 0; l < NL; l++) load_vec(next, l / VPR, l % VPR);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < U; u++) {
                    const int sl = b * U + u;
                    if (sl >= SPW) break;
                    ibf16x8 bh[RG], bl[RG];
#pragma unroll
                    for (int rg = 0; rg < RG; rg++) {
                        const unsigned char* xa = xb + (size_t)(16 * rg) * XS + sl * (BF16 ? 64 : 128);
                        if (BF16) {
                            bh[rg] = __builtin_bit_cast(ibf16x8, *(const iu32x4*)xa);
                        } else {
                            const if32x4 x0 = *(const if32x4*)xa, x1 = *(const if32x4*)(xa + 16);
                            iu32x4 h = {ipack_bf16(x0.x, x0.y), ipack_bf16(x0.z, x0.w), ipack_bf16(x1.x, x1.y), ipack_bf16(x1.z, x1.w)};
                            iu32x4 l = {ipack_bf16(x0.x - ilo_half(h.x), x0.y - ihi_half(h.x)), ipack_bf16(x0.z - ilo_half(h.y), x0.w - ihi_half(h.y)),
                                        ipack_bf16(x1.x - ilo_half(h.z), x1.y - ihi_half(h.z)), ipack_bf16(x1.z - ilo_half(h.w), x1.w - ihi_half(h.w))};
                            bh[rg] = __builtin_bit_cast(ibf16x8, h);
                            bl[rg] = __builtin_bit_cast(ibf16x8, l);
                        }
                    }
                    const ibf16x8(&a)[KW][2] = A[b & 1][u];
#pragma unroll
                    for (int kw = 0; kw < KW; kw++)
#pragma unroll
                        for (int rg = 0; rg < RG; rg++) acc[kw][rg][sl & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[kw][0], bh[rg], acc[kw][rg][sl & 1], 0, 0, 0);
#pragma unroll
                    for (int kw = 0; kw < KW; kw++)
#pragma unroll
                        for (int rg = 0; rg < RG; rg++) acc[kw][rg][sl & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[kw][1], bh[rg], acc[kw][rg][sl & 1], 0, 0, 0);
                    if (!BF16) {
#pragma unroll
                        for (int kw = 0; kw < KW; kw++)
#pragma unroll
                            for (int rg = 0; rg < RG; rg++) acc[kw][rg][sl & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[kw][0], bl[rg], acc[kw][rg][sl & 1], 0, 0, 0);
                    }
                }
            }
            // lane (n, g) holds, for row n of a group, the clusters 4 g .. 4 g + 3 of each of its cluster tiles
#pragma unroll
            for (int kw = 0; kw < KW; kw++)
#pragma unroll
                for (int rg = 0; rg < RG; rg++)
                    *(if32x4*)(s_dots + (size_t)(16 * rg + n) * DS + ic * K16 + 16 * (ik * KW + kw) + 4 * g) = acc[kw][rg][0] + acc[kw][rg][1];
        }
        __syncthreads();
        // ---- rank the centroids of this wave's rows ----
        int idx[RPW];
        float thr[RPW];
        int flagged = 0;  // uniform: rows whose two best scores lie within the error bound of each other
        auto score = [&](int trow, int j) {
            const int k = lane + kWave * j;
            if (K16 % kWave != 0 && k >= K16) return 0x7fffffff;
            const float* q = s_dots + (size_t)trow * DS + k;
            float dot = q[0];
#pragma unroll
            for (int c = 1; c < SC; c++) dot += q[c * K16];
            return score_key(fmaf(-2.f, dot, cn[j]));
        };
#pragma unroll
        for (int r = 0; r < RPW; r++) {
            const int trow = wave * RPW + r;
            int sc[NSLOT], m1 = 0x7fffffff;
#pragma unroll
            for (int j = 0; j < NSLOT; j++) {
                sc[j] = score(trow, j);
                m1 = min(m1, sc[j]);
            }
            const int kb1 = wave_min_all(m1);
            int i1 = 0, m2 = 0x7fffffff;
            bool found = false;
#pragma unroll
            for (int j = 0; j < NSLOT; j++) {
                const unsigned long long hit = __ballot(sc[j] == kb1);
                const int wl = (!found && hit) ? (int)__builtin_ctzll(hit) : -1;  // uniform
                if (wl >= 0) {
                    i1 = wl + kWave * j;
                    found = true;
                }
                m2 = min(m2, lane == wl ? 0x7fffffff : sc[j]);
            }
            const float b1 = key_score(kb1), b2 = key_score(wave_min_all(m2));
            const float bound = p.tau * (1.000001f * __builtin_amdgcn_sqrtf(xn2[r])) * cmax + p.tau2 * cmax * cmax;
            thr[r] = b1 + bound;
            if (tile * ROWS + trow < p.N && !(b2 - b1 > bound)) flagged |= 1 << r;
            idx[r] = i1;
        }
        flagged = __builtin_amdgcn_readfirstlane(flagged);
        while (flagged) {  // one row after the other, its candidates two at a time
            const int r = __builtin_ctz(flagged);
            flagged &= flagged - 1;
            const int trow = wave * RPW + r;
            float th = thr[0];
#pragma unroll
            for (int q = 1; q < RPW; q++) th = q == r ? thr[q] : th;
            const int tk = score_key(th);
            unsigned long long m[NSLOT];
#pragma unroll
            for (int j = 0; j < NSLOT; j++) m[j] = __ballot(score(trow, j) <= tk && lane + kWave * j < p.K);
            auto pop = [&]() {  // the next candidate, -1 if there is none; in rising order
                int k = -1;
#pragma unroll
                for (int j = NSLOT - 1; j >= 0; j--)
                    if (m[j]) k = (int)__builtin_ctzll(m[j]) + kWave * j;
#pragma unroll
                for (int j = 0; j < NSLOT; j++)
                    if (k >= 0 && k / kWave == j) m[j] &= m[j] - 1;
                return __builtin_amdgcn_readfirstlane(k);
            };
            double dbest = __builtin_inf();
            int kbest = -1;
            for (int k0 = pop(); k0 >= 0; k0 = pop()) {
                const int k1 = pop();
                const float* c0 = p.cent + (int64_t)k0 * p.D;
                const int ke = k1 >= 0 ? k1 : k0;
                const float* c1 = p.cent + (int64_t)ke * p.D;
                double d0 = 0.0, d1 = 0.0;
#pragma unroll
                for (int v = 0; v < VPR; v++) {
                    if32x4 a[2], b[2];
                    params(c0, v, k0 == p.K - 1, a[0], a[1]);
                    params(c1, v, ke == p.K - 1, b[0], b[1]);
                    if (UV) {
                        settle_params(a[0], a[1], v, k0 == p.K - 1);
                        settle_params(b[0], b[1], v, ke == p.K - 1);
                    }
                    const iu32x4 w = lds_vec(trow, v);
#pragma unroll
                    for (int e = 0; e < 4; e++) {
                        if (!ok(v, UA ? e : 0)) continue;
#pragma unroll
                        for (int h = 0; h < (BF16 ? 2 : 1); h++) {
                            const double x = (double)(BF16 ? (h ? ihi_half(w[e]) : ilo_half(w[e])) : __uint_as_float(w[e]));
                            const double t0 = x - (double)(BF16 ? a[e >> 1][2 * (e & 1) + h] : a[0][e]);
                            const double t1 = x - (double)(BF16 ? b[e >> 1][2 * (e & 1) + h] : b[0][e]);
                            d0 = fma(t0, t0, d0);
                            d1 = fma(t1, t1, d1);
                        }
                    }
                }
                d0 = wave_total(d0);
                d1 = wave_total(d1);
                if (d0 < dbest) {
                    dbest = d0;
                    kbest = k0;
                }
                if (k1 >= 0 && d1 < dbest) {
                    dbest = d1;
                    kbest = k1;
                }
            }
            if (kbest >= 0) {
#pragma unroll
                for (int q = 0; q < RPW; q++) idx[q] = q == r ? kbest : idx[q];
            }
        }
#pragma unroll
        for (int r = 0; r < RPW; r++) {
            const int64_t row = tile * ROWS + wave * RPW + r;
            idx[r] = __builtin_amdgcn_readfirstlane(idx[r] < p.K ? idx[r] : p.K - 1);  // (non-finite rows: any cluster number)
            if (p.assign && lane == 0 && row < p.N) p.assign[row] = idx[r];
        }
        // ---- affine map of this wave's rows, parameters a few vectors ahead ----
        constexpr int AHEAD = BF16 ? 3 : 4;
        if32x4 P[AHEAD + 1][4];
        auto fetch = [&](int q) {
            const int64_t a = idx[q / VPR];
            params(p.gamma + a * p.D, q % VPR, a == p.K - 1, P[q % (AHEAD + 1)][0], P[q % (AHEAD + 1)][1]);
            params(p.beta + a * p.D, q % VPR, a == p.K - 1, P[q % (AHEAD + 1)][2], P[q % (AHEAD + 1)][3]);
        };
#pragma unroll
        for (int q = 0; q < AHEAD; q++)
            if (q < NL) fetch(q);
#pragma unroll
        for (int q = 0; q < NL; q++) {
            const int r = q / VPR, v = q % VPR;
            __builtin_amdgcn_sched_barrier(0);
            if (q + AHEAD < NL) fetch(q + AHEAD);
            if32x4(&t)[4] = P[q % (AHEAD + 1)];
            if (UV) {
                settle_params(t[0], t[1], v, idx[r] == p.K - 1);
                settle_params(t[2], t[3], v, idx[r] == p.K - 1);
            }
            const int64_t row = tile * ROWS + wave * RPW + r;
            const iu32x4 w = lds_vec(wave * RPW + r, v);
            iu32x4 y;
            if (BF16) {
                y.x = ipack_bf16(fmaf(t[0].x, ilo_half(w.x), t[2].x), fmaf(t[0].y, ihi_half(w.x), t[2].y));
                y.y = ipack_bf16(fmaf(t[0].z, ilo_half(w.y), t[2].z), fmaf(t[0].w, ihi_half(w.y), t[2].w));
                y.z = ipack_bf16(fmaf(t[1].x, ilo_half(w.z), t[3].x), fmaf(t[1].y, ihi_half(w.z), t[3].y));
                y.w = ipack_bf16(fmaf(t[1].z, ilo_half(w.w), t[3].z), fmaf(t[1].w, ihi_half(w.w), t[3].w));
            } else {
#pragma unroll
                for (int e = 0; e < 4; e++) y[e] = __float_as_uint(fmaf(t[0][e], __uint_as_float(w[e]), t[2][e]));
            }
            T* o = (T*)p.out + row * p.D;
            if (row < p.N) {
                if (UV && whole(v)) {
                    __builtin_nontemporal_store(y, (iu32x4_w*)((uint32_t*)o + pos(v, 0)));
                } else if (UA) {
#pragma unroll
                    for (int e = 0; e < 4; e++)
                        if (ok(v, e)) __builtin_nontemporal_store(y[e], (uint32_t*)o + pos(v, e));
                } else if (ok(v, 0)) {
                    __builtin_nontemporal_store(y, (iu32x4*)(o + pos(v, 0)));
                }
            }
        }
        // the rows of this tile are this wave's alone since the barrier: the next ones take their place
        stage(next);
        __syncthreads();
    }
}

}  // namespace cat
