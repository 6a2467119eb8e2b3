// Fused inference over rows of at most 512 bytes.
//
// k_infer moves and ranks a row per wave instruction: on a row of 240 bytes 15 of its 64 lanes have something to do, and the
// ranking of a row costs as much as on a long one.  Here a wave owns tiles of 16 consecutive rows, which in memory are one piece of
// 16 D elements, whole 16-byte groups whatever D is:
//   - it loads the piece as it lies, 64 consecutive 16-byte groups an instruction, the next tile's while it works on this one;
//   - lays the rows out in LDS 16 (2 n + 1) bytes apart (16 rows in 16 different banks), from where the matrix instructions take them
//     as in the tile kernel: clusters are the M dimension, so that a lane ranks 4 clusters per tile of 16 of ONE row, 16 rows at once;
//   - measures rows within the error bound of the split arithmetic in double precision (row from LDS);
//   - maps the piece from the registers it came in: every group knows its row from the start and takes that row's cluster; the
//     folded parameters lie in LDS where they fit (from L1 / L2 700001 x 61, K = 50 took 153 us instead of 80), the result leaves
//     as it came, in whole groups.
// Nothing crosses the waves after the operand, which every workgroup prepares for itself (one launch in all).  What bounds it: the
// row traffic from some 100 MB on; below, the launch and the latency of one tile after the other.
#include <atomic>

#include "cat_infer.h"
#include "cat_rank.h"
#include "cat_short.h"
#include "cat_tile_kernel.h"

namespace cat {

constexpr int kShortT = 512, kShortW = kShortT / kWave;

struct ShortParams {
    const void* lq;
    void* out;
    int32_t* assign;  // nullable
    int64_t N, ntiles;
    int32_t D, K, nsteps;
    const float* cent;
    const float* gamma;
    const float* beta;
    float alpha;
    float tau, tau2;
    uint32_t off_rows, row_stride, wave_stride;  // LDS: operand, norms, the waves' rows, (PL) the parameters
    uint32_t off_params;
};

// PL: the folded parameters lie in LDS, gamma and beta of a channel side by side.  KT: cluster tiles.  VV: 16-byte groups of a tile per lane (rows of up to 64 VV bytes).  UA: rows that are not whole 16-byte groups.
template <bool BF16, int KT, int VV, bool UA, bool PL>
__global__ __launch_bounds__(kShortT) void k_apply_short(const ShortParams p) {
    static_assert(PL || !UA, "unaligned rows take their parameters from LDS");
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int CPW = BF16 ? 2 : 1;  // channels of a word
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int n = lane & 15, q = lane >> 4;
    const int D = p.D, K = p.K, W = D / CPW, RS = (int)p.row_stride;
    float* s_cnorm = (float*)(smem + p.nsteps * KT * 2048);
    unsigned char* rows = smem + p.off_rows + wave * p.wave_stride;
    int* s_idx = (int*)(rows + 16 * RS);  // 16: the clusters of the tile's rows

    // ---- the tile's pieces ----
    const int64_t step = (int64_t)gridDim.x * kShortW;
    int64_t tile = (int64_t)blockIdx.x * kShortW + wave;
    const uint32_t* lq = (const uint32_t*)p.lq;
    int at[VV];  // row << 16 | word in the row, of the first word of the group; past the tile: row 16
#pragma unroll
    for (int j = 0; j < VV; j++) {
        const int w = 4 * (lane + kWave * j), r = w / W;
        at[j] = r < 16 ? (r << 16) | (w - r * W) : 16 << 16;
    }
    auto load = [&](int64_t t, u32x4 (&x)[VV]) {
        if (t >= p.ntiles) return;
        const uint32_t* src = lq + t * 16 * W;
        if ((t + 1) * 16 <= p.N) {
#pragma unroll
            for (int j = 0; j < VV; j++) x[j] = *(const u32x4*)(src + (at[j] >> 16 < 16 ? 4 * (lane + kWave * j) : 0));
        } else {  // the last, shorter tile: word by word, past its end the last one
            const int last = (int)(p.N - t * 16) * W - 1;
#pragma unroll
            for (int j = 0; j < VV; j++)
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    const int w = 4 * (lane + kWave * j) + e;
                    x[j][e] = src[w < last ? w : last];
                }
        }
    };
    u32x4 x[VV], xn[VV];
    load(tile, x);

    // ---- operand and norms ----
    for (int i = tid; i < (int)((p.off_rows + kShortW * p.wave_stride) / 16); i += kShortT) ((u32x4*)smem)[i] = (u32x4){0u, 0u, 0u, 0u};
    __syncthreads();
    if (tid < KT * 16 && tid >= K) s_cnorm[tid] = kPadNorm;
    const bool plain = p.alpha == 1.f;
    auto fold_g = [&](float g) { return plain ? g : 1.f + p.alpha * (g - 1.f); };
    auto fold_b = [&](float v) { return plain ? v : p.alpha * v; };
    float2* s_par = (float2*)(smem + p.off_params);
    if (PL) {
#pragma unroll 4
        for (int i = tid; i < K * D; i += kShortT) s_par[i] = float2{fold_g(p.gamma[i]), fold_b(p.beta[i])};
    }
    constexpr int CB = 4, CC = BF16 ? 4 : 2;  // clusters of a wave whose values are requested at once, 64 channels each
    for (int k0 = wave; k0 < K; k0 += CB * kShortW) {
        float c[CB][CC];
#pragma unroll
        for (int u = 0; u < CB; u++)
#pragma unroll
            for (int v = 0; v < CC; v++) {
                const int k = k0 + u * kShortW, ch = lane + v * kWave;
                c[u][v] = p.cent[(k < K ? k : k0) * D + (ch < D ? ch : 0)];
            }
#pragma unroll
        for (int u = 0; u < CB; u++) {
            const int k = k0 + u * kShortW;
            if (k >= K) break;
            double nn = 0.0;
#pragma unroll
            for (int v = 0; v < CC; v++) {
                const int ch = lane + v * kWave;
                if (ch >= D) continue;
                const float f = c[u][v];
                int g, e;
                operand_slot(ch & 31, false, g, e);
                uint16_t* a = (uint16_t*)(smem + ((ch >> 5) * KT + (k >> 4)) * 2048 + (g * 16 + (k & 15)) * 16) + e;
                const uint32_t hw = pack_bf16(f, 0.f) & 0xFFFFu;
                a[0] = (uint16_t)hw;
                a[512] = (uint16_t)(pack_bf16(f - lo_half(hw), 0.f) & 0xFFFFu);
                nn = fma((double)f, (double)f, nn);
            }
            nn = wave_total(nn);
            if (lane == 0) s_cnorm[k] = (float)nn;
        }
    }
    __syncthreads();
    float cmax = 0.f;
    for (int k = lane; k < K; k += kWave) cmax = fmaxf(cmax, s_cnorm[k]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) cmax = fmaxf(cmax, __shfl_xor(cmax, o, kWave));
    cmax = sqrtf(cmax);

    for (; tile < p.ntiles; tile += step) {
        load(tile + step, xn);
        // ---- rows to LDS ----
#pragma unroll
        for (int j = 0; j < VV; j++) {
            const int r = at[j] >> 16, w = at[j] & 0xFFFF;
            if (r < 16) {
                if (UA) {
#pragma unroll
                    for (int e = 0; e < 4; e++) {
                        const bool over = w + e >= W;
                        if (r + over < 16) *(uint32_t*)(rows + (r + over) * RS + 4 * (w + e - (over ? W : 0))) = x[j][e];
                    }
                } else {
                    *(u32x4*)(rows + r * RS + 4 * w) = x[j];
                }
            }
        }
        __builtin_amdgcn_wave_barrier();  // (the lanes read what others wrote; LDS serves a wave in order)
        // ---- contraction ----
        f32x4 acc[KT];
        float nrm = 0.f;
#pragma unroll
        for (int u = 0; u < KT; u++) acc[u] = (f32x4){0.f, 0.f, 0.f, 0.f};
        for (int s = 0; s < p.nsteps; s++) {  // (channels past the row: zeros, in LDS and in the operand)
            const unsigned char* xr = rows + n * RS + (BF16 ? 64 * s + 16 * q : 128 * s + 32 * q);
            bf16x8 bh, bl;
            if (BF16) {
                const u32x4 w = *(const u32x4*)xr;
#pragma unroll
                for (int j = 0; j < 4; j++) nrm = fmaf(lo_half(w[j]), lo_half(w[j]), fmaf(hi_half(w[j]), hi_half(w[j]), nrm));
                bh = bl = __builtin_bit_cast(bf16x8, w);
            } else {
                const f32x4 a = __builtin_bit_cast(f32x4, *(const u32x4*)xr), b = __builtin_bit_cast(f32x4, *(const u32x4*)(xr + 16));
                const float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
                u32x4 h, l;
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    nrm = fmaf(v[2 * j], v[2 * j], fmaf(v[2 * j + 1], v[2 * j + 1], nrm));
                    h[j] = pack_bf16(v[2 * j], v[2 * j + 1]);
                    l[j] = pack_bf16(v[2 * j] - lo_half(h[j]), v[2 * j + 1] - hi_half(h[j]));
                }
                bh = __builtin_bit_cast(bf16x8, h);
                bl = __builtin_bit_cast(bf16x8, l);
            }
            const unsigned char* ap = smem + s * KT * 2048 + lane * 16;
#pragma unroll
            for (int u = 0; u < KT; u++) {
                const bf16x8 ah = __builtin_bit_cast(bf16x8, *(const u32x4*)(ap + u * 2048));
                const bf16x8 al = __builtin_bit_cast(bf16x8, *(const u32x4*)(ap + u * 2048 + 1024));
                acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bh, acc[u], 0, 0, 0);
                acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bh, acc[u], 0, 0, 0);
                if (!BF16) acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bl, acc[u], 0, 0, 0);
            }
        }
        // ---- ranking: lane (n, q) has the clusters 16 u + 4 q .. + 3 of row n ----
        const float xn2 = sum_groups(nrm);
        float f1 = __builtin_inff(), f2 = __builtin_inff();
        int i1 = 0;
#pragma unroll
        for (int u = 0; u < KT; u++) {
            const f32x4 cn = *(const f32x4*)(s_cnorm + 16 * u + 4 * q);
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const float s = fmaf(-2.f, acc[u][i], cn[i]);
                f2 = s < f1 ? f1 : (s < f2 ? s : f2);
                i1 = s < f1 ? 16 * u + 4 * q + i : i1;
                f1 = s < f1 ? s : f1;
            }
        }
        best_two_groups(f1, i1, f2);
        i1 = i1 < K ? i1 : K - 1;  // (non-finite rows: any cluster number)
        const bool valid = tile * 16 + n < p.N;
        const float bound = p.tau * sqrtf(xn2) * cmax + p.tau2 * cmax * cmax;
        unsigned long long mask = __ballot(valid && !(f2 - f1 > bound) && q == 0);
        while (mask) {  // a row whose two best are within the error bound: exact distances to all clusters within it, rising
            const int r = __builtin_amdgcn_readfirstlane(__builtin_ctzll(mask));
            mask &= mask - 1;
            const float thr = readlane_f(f1, r) + readlane_f(bound, r);
            double dbest = __builtin_inf();
            int kbest = -1;
#pragma unroll
            for (int u = 0; u < KT; u++) {
                uint32_t cand = 0;  // of this tile of 16 clusters
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const unsigned long long m = __ballot(n == r && fmaf(-2.f, acc[u][i], s_cnorm[16 * u + 4 * q + i]) <= thr && 16 * u + 4 * q + i < K);
                    // lanes r, r + 16, r + 32, r + 48: clusters 16 u + 4 q + i
#pragma unroll
                    for (int g = 0; g < 4; g++) cand |= (uint32_t)(m >> (r + 16 * g) & 1ull) << (4 * g + i);
                }
                while (cand) {
                    const int ka = 16 * u + __builtin_amdgcn_readfirstlane(__builtin_ctz(cand));
                    cand &= cand - 1;
                    const int kb = cand ? 16 * u + __builtin_amdgcn_readfirstlane(__builtin_ctz(cand)) : ka;
                    if (cand) cand &= cand - 1;
                    double da = 0.0, db = 0.0;
                    for (int ch = lane; ch < D; ch += kWave) {
                        const uint32_t xw = ((const uint32_t*)(rows + r * RS))[ch / CPW];
                        const double v = (double)(!BF16 ? __uint_as_float(xw) : ch & 1 ? hi_half(xw) : lo_half(xw));
                        const double ua = v - (double)p.cent[ka * D + ch], ub = v - (double)p.cent[kb * D + ch];
                        da = fma(ua, ua, da);
                        db = fma(ub, ub, db);
                    }
                    da = wave_total(da);
                    db = wave_total(db);
                    if (da < dbest) {  // (an equal one later does not win)
                        dbest = da;
                        kbest = ka;
                    }
                    if (db < dbest) {
                        dbest = db;
                        kbest = kb;
                    }
                }
            }
            if (n == r && kbest >= 0) i1 = kbest;
        }
        if (q == 0) {
            s_idx[n] = i1;
            if (p.assign && valid) p.assign[tile * 16 + n] = i1;
        }
        __builtin_amdgcn_wave_barrier();
        // ---- the map, in the groups as they came ----
        const bool whole = (tile + 1) * 16 <= p.N;
        const int words = whole ? 16 * W : (int)(p.N - tile * 16) * W;
        uint32_t* dst = (uint32_t*)p.out + tile * 16 * W;
#pragma unroll
        for (int j = 0; j < VV; j++) {
            const int r = at[j] >> 16, w = at[j] & 0xFFFF;
            if (r < 16) {
                u32x4 y;
                const int ka = s_idx[r], kb = UA ? s_idx[r < 15 ? r + 1 : 15] : ka;
                if (PL) {
                    const float2* pa = s_par + (ka * W + w) * CPW;
                    const float2* pb = UA ? s_par + (kb * W + w - W) * CPW : pa;
#pragma unroll
                    for (int e = 0; e < 4; e++) {
                        const float2* o = (UA && w + e >= W ? pb : pa) + e * CPW;
                        if (BF16) {
                            const f32x4 t = *(const f32x4*)o;  // two channels: gamma, beta, gamma, beta
                            y[e] = pack_bf16(fmaf(t.x, lo_half(x[j][e]), t.y), fmaf(t.z, hi_half(x[j][e]), t.w));
                        } else {
                            const f32x2 t = *(const f32x2*)o;
                            y[e] = __float_as_uint(fmaf(t.x, __uint_as_float(x[j][e]), t.y));
                        }
                    }
                } else {
                    const int o = (ka * W + w) * CPW;
#pragma unroll
                    for (int h = 0; h < CPW; h++) {
                        const f32x4 g = *(const f32x4*)(p.gamma + o + 4 * h), c = *(const f32x4*)(p.beta + o + 4 * h);
                        if (BF16) {
#pragma unroll
                            for (int e = 0; e < 2; e++) {
                                const uint32_t v = x[j][2 * h + e];
                                y[2 * h + e] = pack_bf16(fmaf(fold_g(g[2 * e]), lo_half(v), fold_b(c[2 * e])),
                                                         fmaf(fold_g(g[2 * e + 1]), hi_half(v), fold_b(c[2 * e + 1])));
                            }
                        } else {
#pragma unroll
                            for (int e = 0; e < 4; e++) y[e] = __float_as_uint(fmaf(fold_g(g[e]), __uint_as_float(x[j][e]), fold_b(c[e])));
                        }
                    }
                }
                const int w0 = 4 * (lane + kWave * j);
                if (w0 + 4 <= words) {
                    __builtin_nontemporal_store(y, (u32x4*)(dst + w0));
                } else {
#pragma unroll
                    for (int e = 0; e < 4; e++)
                        if (w0 + e < words) dst[w0 + e] = y[e];
                }
            }
        }
#pragma unroll
        for (int j = 0; j < VV; j++) x[j] = xn[j];
    }
}

struct ShortCfg {
    bool ok = false;
    int KT = 0, VV = 0, nsteps = 0;
    bool params = false;  // in LDS
    uint32_t off_rows = 0, row_stride = 0, wave_stride = 0, off_params = 0;
    size_t lds = 0;
};
static ShortCfg short_config(int64_t N, int64_t D, int32_t K, cat_dtype dt) {
    ShortCfg c;
    const int b = dt == CAT_BF16 ? 2 : 4;
    if (N < 1 || N >= ((int64_t)1 << 40) || D * b < 16 || D * b > 512 || K > 128 || (dt == CAT_BF16 && D % 2)) return c;
    c.KT = 1;
    while (c.KT * 16 < K) c.KT *= 2;
    c.VV = D * b <= 128 ? 2 : D * b <= 256 ? 4 : 8;
    c.nsteps = (int)((D + 31) / 32);
    c.off_rows = (uint32_t)(c.nsteps * c.KT * 2048 + c.KT * 64);
    c.row_stride = (uint32_t)(c.nsteps * 32 * b + 16);  // an odd number of 16-byte groups: 16 rows in 16 different banks
    c.wave_stride = 16 * c.row_stride + 64;
    c.lds = c.off_rows + (size_t)kShortW * c.wave_stride;
    c.off_params = (uint32_t)c.lds;
    c.params = c.lds + (size_t)K * D * 8 <= kLdsLimit;
    if (c.params) c.lds += (size_t)K * D * 8;
    // (unaligned rows word by word from L2: 500001 x 101, K = 100: 310 us on the other kernels, 316 here)
    c.ok = c.lds <= kLdsLimit && (c.params || D % (16 / b) == 0);
    return c;
}

// us per cat_apply before / here: 700001 x 60, K = 16: 198 / 66, K = 120: 244 / 103; 700001 x 61, K = 50: 237 / 80; 500001 x 101, K = 50:
// 187 / 93; 500001 x 128, K = 50: 192 / 112; bf16: 700001 x 60, K = 16: 214 / 33; 758816 x 128, K = 5: 354 / 73; 400001 x 250, K = 30: 243 / 91.
// Wherever the row-tile kernel has no instance of two parts (bf16, K > 64), 1.3 times as fast or more; where it has one, always from 16384
// rows on (17830 x 114, K = 57: 14.4 / 13.9, the least gain of 894 calls).  Below, one launch less is set against an operand that every
// workgroup prepares for itself and a wave's one tile at the pace of its latencies: the difference in us, by least squares over 2300 random
// calls from a graph, must be 0.35 in favour.  Near ties are measured one after the other by the wave that has them, so that many clusters
// on few channels, and more than 64 at all, count against it.  Over 5000 calls, the same and others: 1.53 times as fast on average, 1.002
// times what the faster kernel takes; 37 longer than the row-tile kernel by more than 2 %, the worst 9.4 / 11.8 (3253 x 24, K = 90, overlapping
// clusters).  Either side of the line: 2041 x 118, K = 16: 8.2 / 10.6; bf16 6444 x 200, K = 54: 10.4 / 12.6; 4298 x 242 bf16, K = 2: 10.3 / 11.1;
// 3420 x 106 bf16, K = 3: 8.1 / 6.8; 12479 x 4, K = 22: 10.9 / 5.9; 15363 x 6, K = 35: 13.2 / 8.2; 9329 x 122 bf16, K = 4: 11.8 / 7.3.
bool short_apply_pays(int64_t N, int64_t D, int32_t K, cat_dtype dt) {
    const ShortCfg c = short_config(N, D, K, dt);
    if (!c.ok) return false;
    if (N >= 16384) return true;
    const double row = (double)D * (dt == CAT_BF16 ? 2.0 : 4.0);
    const bool ua = D % (dt == CAT_BF16 ? 8 : 4) != 0;
    const double longer = -3.3 + 0.18 * c.KT * c.nsteps + (ua ? 0.0103 : 0.0074) * row + 0.2 * (double)K / (double)D - 0.29e-3 * (double)N;
    return longer + (K > 64 ? 0.9 : 0.0) < -0.35 || !infer_two_parts(D, K, dt);
}

template <bool BF16, int KT, int VV, bool UA, bool PL>
static cat_status launch_short(const ShortParams& p, const ShortCfg& c, hipStream_t st) {
    auto kern = k_apply_short<BF16, KT, VV, UA, PL>;
    static thread_local int cached_lds = -1, cached_dev = -1, per_cu = 1, ncu = 256;
    int dev = 0;
    CAT_HIP_TRY(hipGetDevice(&dev));
    if (cached_lds != (int)c.lds || cached_dev != dev) {
        int nb = 0, v = 0;
        // (the most there is, not what this call needs: another thread may launch the same kernel for a larger K D meanwhile)
        CAT_HIP_TRY(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsLimit));
        CAT_HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, (const void*)kern, kShortT, c.lds));
        CAT_HIP_TRY(hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev));
        per_cu = nb < 1 ? 1 : nb;
        ncu = v > 0 ? v : 256;
        cached_lds = (int)c.lds;
        cached_dev = dev;
    }
    const int64_t want = (p.ntiles + kShortW - 1) / kShortW, cap = (int64_t)ncu * per_cu;
    const bool prof = profile_on();
    if (prof)
        if (cat_status s = profile_mark(true, st); s != CAT_OK) return s;
    hipLaunchKernelGGL(kern, dim3((unsigned)(want < cap ? want : cap)), dim3(kShortT), c.lds, st, p);
    CAT_LAUNCH_CHECK("k_apply_short");
    return prof ? profile_mark(false, st) : CAT_OK;
}
template <bool BF16, int KT, bool UA>
static cat_status launch_short_vv(const ShortParams& p, const ShortCfg& c, hipStream_t st) {
    if constexpr (!UA)
        if (!c.params)
            return c.VV == 2   ? launch_short<BF16, KT, 2, false, false>(p, c, st)
                   : c.VV == 4 ? launch_short<BF16, KT, 4, false, false>(p, c, st)
                               : launch_short<BF16, KT, 8, false, false>(p, c, st);
    return c.VV == 2   ? launch_short<BF16, KT, 2, UA, true>(p, c, st)
           : c.VV == 4 ? launch_short<BF16, KT, 4, UA, true>(p, c, st)
                       : launch_short<BF16, KT, 8, UA, true>(p, c, st);
}
template <bool BF16, bool UA>
static cat_status launch_short_kt(const ShortParams& p, const ShortCfg& c, hipStream_t st) {
    switch (c.KT) {
        case 1: return launch_short_vv<BF16, 1, UA>(p, c, st);
        case 2: return launch_short_vv<BF16, 2, UA>(p, c, st);
        case 4: return launch_short_vv<BF16, 4, UA>(p, c, st);
        default: return launch_short_vv<BF16, 8, UA>(p, c, st);
    }
}

cat_status short_apply(const void* lq, cat_dtype dt, int64_t N, int64_t D, int32_t K, const float* cent, const float* gamma,
                       const float* beta, float alpha, void* corrected, int32_t* assign, hipStream_t st) {
    const ShortCfg c = short_config(N, D, K, dt);
    if (!c.ok) return set_error(CAT_ERR_UNSUPPORTED, "inference over short rows does not fit D=%lld K=%d", (long long)D, (int)K);
    ShortParams p = {};
    p.lq = lq;
    p.out = corrected;
    p.assign = assign;
    p.N = N;
    p.ntiles = (N + 15) / 16;
    p.D = (int32_t)D;
    p.K = K;
    p.nsteps = c.nsteps;
    p.cent = cent;
    p.gamma = gamma;
    p.beta = beta;
    p.alpha = alpha;
    p.tau = split_tau(dt, (dt == CAT_BF16 ? 2 : 3) * c.nsteps + 8);
    p.tau2 = kSplitTau2;
    p.off_rows = c.off_rows;
    p.row_stride = c.row_stride;
    p.wave_stride = c.wave_stride;
    p.off_params = c.off_params;
    const bool ua = D % (dt == CAT_BF16 ? 8 : 4) != 0;
    if (dt == CAT_BF16) return ua ? launch_short_kt<true, true>(p, c, st) : launch_short_kt<true, false>(p, c, st);
    return ua ? launch_short_kt<false, true>(p, c, st) : launch_short_kt<false, false>(p, c, st);
}

}  // namespace cat
