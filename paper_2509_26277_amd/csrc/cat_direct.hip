// Fused inference for few rows: nearest centroid and affine map straight from the caller's arrays, in one launch.
//
// With a few hundred rows the call is bound by its chain of launches and memory round trips, not by bytes or flops: the
// matrix-core kernels need a launch that prepares their operand, tiles of 16 rows leave most of the chip idle, and a
// tile is a chain of operand, rows, ranking, parameters.  Here a workgroup takes R rows (R chosen so that the rows spread
// over the chip), its waves share the clusters, and a distance is summed in direct form in float32 on the vector units,
// every load of a round requested before the first is used.  The sums are of squares, so their error is relative and
// small; clusters within it of the nearest are measured again in double (lowest index on ties), which decides as the other
// kernels do.  The blending coefficient is folded into the parameters as they are read.
#include "cat_direct.h"

#include "cat_infer.h"
#include "cat_wide.h"

namespace cat {

namespace {

constexpr int kDirT = 512;                  // threads per workgroup
constexpr int kDirWaves = kDirT / kWave;
constexpr int kDirU = 8;                    // clusters a wave measures side by side
constexpr int kDirX = 8;                    // channels of a lane per round of an exact distance
constexpr int kDirMaxR = 4;

struct DirectParams {
    const void* lq;
    int64_t N, D;
    int32_t K;
    const float* cent;
    const float* gamma;
    const float* beta;
    float alpha;
    void* out;
    int32_t* assign;  // nullable
    float rel;        // relative error bound of a difference of two float32 sums
};

typedef __attribute__((ext_vector_type(2))) __bf16 dbf16x2;
typedef __attribute__((ext_vector_type(2))) float df32x2;
__device__ __forceinline__ uint32_t round_pair(float a, float b) {  // a -> low half, b -> high half, to nearest even
    const df32x2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, dbf16x2));
}

// V consecutive elements as floats: one load of 4 V (float) or 2 V (bfloat16) bytes
template <int V>
__device__ __forceinline__ void load_vec(const float* p, float (&x)[V]) {
    if constexpr (V == 4) {
        const float4 v = *(const float4*)p;
        x[0] = v.x, x[1] = v.y, x[2] = v.z, x[3] = v.w;
    } else {
        x[0] = *p;
    }
}
template <int V>
__device__ __forceinline__ void load_vec(const bf16_t* p, float (&x)[V]) {
    if constexpr (V == 4) {
        const uint2 v = *(const uint2*)p;
        x[0] = __uint_as_float(v.x << 16), x[1] = __uint_as_float(v.x & 0xFFFF0000u);
        x[2] = __uint_as_float(v.y << 16), x[3] = __uint_as_float(v.y & 0xFFFF0000u);
    } else {
        x[0] = bf16_to_f32(*p);
    }
}
template <int V>
__device__ __forceinline__ void store_vec(float* p, const float (&x)[V]) {
    if constexpr (V == 4)
        *(float4*)p = make_float4(x[0], x[1], x[2], x[3]);
    else
        *p = x[0];
}
template <int V>
__device__ __forceinline__ void store_vec(bf16_t* p, const float (&x)[V]) {
    if constexpr (V == 4)
        *(uint2*)p = make_uint2(round_pair(x[0], x[1]), round_pair(x[2], x[3]));
    else
        *p = (bf16_t)(round_pair(x[0], 0.f) & 0xFFFFu);
}

// The sum over each row of 16 lanes, in all of them (lane permutations fused into the additions).
template <int CTRL>
__device__ __forceinline__ float dpp_addf(float v) {
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float row16_total(float v) {
    v = dpp_addf<0xB1>(v);   // quad_perm [1, 0, 3, 2]
    v = dpp_addf<0x4E>(v);   // quad_perm [2, 3, 0, 1]
    v = dpp_addf<0x141>(v);  // row_half_mirror
    return dpp_addf<0x140>(v);  // row_mirror
}

}  // namespace

// V: elements per load (4 where rows and parameters are whole groups of 4, else 1).  R: rows per workgroup.
template <typename T, int V, int R>
__global__ __launch_bounds__(kDirT) void k_apply_direct(const DirectParams p) {
    extern __shared__ float4 s_dist[];  // R x K, each as the sums over the four rows of 16 lanes
    __shared__ int s_label[kDirMaxR];
    constexpr int STEP = kWave * V;                       // channels a wave covers with one load per lane
    constexpr int Q = V == 1 ? 8 : R > 2 ? 2 : 4;           // such steps per round of loads
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t row0 = (int64_t)blockIdx.x * R;
    const int D = (int)p.D;
    const T* xr[R];
#pragma unroll
    for (int r = 0; r < R; r++) xr[r] = (const T*)p.lq + (row0 + r < p.N ? row0 + r : p.N - 1) * p.D;

    for (int kb = wave; kb < p.K; kb += kDirWaves * kDirU) {
        const float* cr[kDirU];
        float acc[kDirU][R];
#pragma unroll
        for (int u = 0; u < kDirU; u++) {
            const int k = kb + kDirWaves * u;
            cr[u] = p.cent + (int64_t)(k < p.K ? k : kb) * p.D;  // (past the last: the first of the round again, dropped below)
#pragma unroll
            for (int r = 0; r < R; r++) acc[u][r] = 0.f;
        }
        for (int base = 0; base < D; base += STEP * Q) {
            float x[Q][R][V], c[Q][kDirU][V];
#pragma unroll
            for (int q = 0; q < Q; q++) {
                const int ch = base + q * STEP + lane * V, at = ch < D ? ch : 0;
#pragma unroll
                for (int r = 0; r < R; r++) load_vec<V>(xr[r] + at, x[q][r]);
#pragma unroll
                for (int u = 0; u < kDirU; u++) load_vec<V>(cr[u] + at, c[q][u]);
            }
#pragma unroll
            for (int q = 0; q < Q; q++) {
                if (base + (q + 1) * STEP <= D) {  // uniform
#pragma unroll
                    for (int u = 0; u < kDirU; u++)
#pragma unroll
                        for (int r = 0; r < R; r++)
#pragma unroll
                            for (int e = 0; e < V; e++) {
                                const float d = x[q][r][e] - c[q][u][e];
                                acc[u][r] = fmaf(d, d, acc[u][r]);
                            }
                } else if (base + q * STEP < D) {
                    const bool in = base + q * STEP + lane * V < D;
#pragma unroll
                    for (int u = 0; u < kDirU; u++)
#pragma unroll
                        for (int r = 0; r < R; r++)
#pragma unroll
                            for (int e = 0; e < V; e++) {
                                const float d = in ? x[q][r][e] - c[q][u][e] : 0.f;
                                acc[u][r] = fmaf(d, d, acc[u][r]);
                            }
                }
            }
        }
#pragma unroll
        for (int u = 0; u < kDirU; u++) {
            const int k = kb + kDirWaves * u;
            if (k >= p.K) break;  // uniform
#pragma unroll
            for (int r = 0; r < R; r++) {
                const float s = row16_total(acc[u][r]);
                if ((lane & 15) == 0) ((float*)s_dist)[4 * (r * p.K + k) + (lane >> 4)] = s;
            }
        }
    }
    __syncthreads();
    if (wave < R) {  // one wave per row: the nearest, or the clusters that may be
        auto dist = [&](int k) {
            const float4 v = s_dist[wave * p.K + (k < p.K ? k : p.K - 1)];
            return (v.x + v.y) + (v.z + v.w);
        };
        float best = __builtin_inff();
        for (int k = lane; k < p.K; k += kWave) best = fminf(best, dist(k));
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) best = fminf(best, __shfl_xor(best, o, kWave));
        const float thr = fmaf(best, p.rel, best) + 1e-36f;
        int label = -1;
        double dbest = __builtin_inf();
        const T* x = (const T*)p.lq + (row0 + wave < p.N ? row0 + wave : p.N - 1) * p.D;
        int cnt = 0, only = 0;
        for (int k0 = 0; k0 < p.K; k0 += kWave) {
            const unsigned long long m = __ballot(k0 + lane < p.K && !(dist(k0 + lane) > thr));
            cnt += __builtin_popcountll(m);
            if (m) only = k0 + __builtin_ctzll(m);
        }
        if (cnt == 1) {
            label = only;
        } else {
            for (int k0 = 0; k0 < p.K; k0 += kWave) {
                unsigned long long m = __ballot(k0 + lane < p.K && !(dist(k0 + lane) > thr));
                while (m) {
                    const int k = k0 + __builtin_amdgcn_readfirstlane(__builtin_ctzll(m));
                    m &= m - 1;
                    const float* c = p.cent + (int64_t)k * p.D;
                    double d2 = 0.0;
                    // Requested together and added up in the order of one at a time: with a trip through memory for every 64
                    // channels, rows near ties took longer than on the other kernels (us, those / one at a time / this: 1024 x 1000
                    // bf16, K = 16, overlapping clusters 11.3 / 12.8 / 10.7, equal ones 30.8 / 39.1 / 21.4; 256 x 1000, K = 50,
                    // overlapping: 20.8 / 10.0 / 7.9).
                    for (int base = lane; base < D; base += kWave * kDirX) {
                        float xe[kDirX], ce[kDirX];
#pragma unroll
                        for (int u = 0; u < kDirX; u++) {
                            const int at = base + kWave * u < D ? base + kWave * u : lane;
                            xe[u] = ld_elem(x + at);
                            ce[u] = c[at];
                        }
#pragma unroll
                        for (int u = 0; u < kDirX; u++) {
                            const double d = base + kWave * u < D ? (double)xe[u] - (double)ce[u] : 0.0;
                            d2 = fma(d, d, d2);
                        }
                    }
                    d2 = wave_total(d2);
                    if (label < 0 || d2 < dbest || (dbest != dbest && d2 == d2)) {  // in index order: the lowest on ties
                        dbest = d2;
                        label = k;
                    }
                }
            }
            label = label < 0 ? 0 : label;  // (no distance compares with the threshold: any cluster)
        }
        if (lane == 0) {
            s_label[wave] = label;
            if (p.assign && row0 + wave < p.N) p.assign[row0 + wave] = label;
        }
    }
    __syncthreads();
    const int nv = D / V;
    const int rows = p.N - row0 < R ? (int)(p.N - row0) : R;
    for (int i = threadIdx.x; i < rows * nv; i += kDirT) {
        const int r = R == 1 ? 0 : i / nv;
        const int ch = (i - r * nv) * V;
        const int64_t at = (int64_t)s_label[r] * p.D + ch;
        float x[V], g[V], b[V], y[V];
        load_vec<V>((const T*)p.lq + (row0 + r) * p.D + ch, x);
        load_vec<V>(p.gamma + at, g);
        load_vec<V>(p.beta + at, b);
#pragma unroll
        for (int e = 0; e < V; e++) {
            // (the same operations as the launch that folds the coefficient for the other kernels; 1 leaves them as they are)
            const float ge = p.alpha == 1.0f ? g[e] : 1.f + p.alpha * (g[e] - 1.f);
            const float be = p.alpha == 1.0f ? b[e] : p.alpha * b[e];
            y[e] = fmaf(ge, x[e], be);
        }
        store_vec<V>((T*)p.out + (row0 + r) * p.D + ch, y);
    }
}

// Where the line lies (us per call from a graph, the other kernels / here; fp32 unless said):
//   instances of the row-tile kernel with the two-part operand (their launches are short): 256 x 512, K = 128: 9.7 / 7.8, 512 rows
//   9.8 / 9.7, 1024 rows 10.0 / 11.0; 1024 x 512, K = 60: 10.3 / 7.6; 1024 x 1000, K = 16: 11.3 / 8.9; 1024 x 64, K = 100: 8.3 / 9.3;
//   its one-part instance and the streamed-operand kernel: 256 x 1000, K = 50: 13.9 / 5.9, 1024 rows 14.3 / 9.5; 1024 x 2048 bf16,
//   K = 64: 26.8 / 13.9; 1024 x 768, K = 256: 25.7 / 22.9; 1024 x 1200 bf16, K = 200: 38.9 / 30.0; 256 x 1001, K = 50: 22.0 / 6.6; but
//   520 x 301, K = 256: 19.1 / 19.6 and 520 x 102, K = 256: 18.0 / 18.4 (element loads), and with four rows to a workgroup, many
//   clusters and a step of 256 channels that is partly empty, against the streamed operand on rows of 1 .. 2 KB: 1024 x 300: K =
//   160: 18.4 / 16.1, K = 200: 18.5 / 19.9, K = 256: 18.0 / 20.9, 520 rows 18.0 / 19.9, 512 rows 18.1 / 17.2; 1024 x 512, K = 200: 19.4 /
//   18.3; bf16: 1024 x 640: K = 200: 24.2 / 25.0, K = 256: 24.0 / 25.8; 1024 x 768, K = 200: 25.4 / 23.7; 768 x 1000, K = 256: 26.0 / 27.4.  The
//   one-part instance for 65 .. 128 clusters varies with the data, since it measures again what lies within 1.6 %: 1024 x 384, K =
//   128: well separated rows 10.0 / 12.3, a feature map's 11.4 / 12.4, an even mixture's 11.6 / 12.4, a skewed one's 30.2 / 12.4;
//   the 2 us are given for the 18;
//   shapes neither has an instance for (rows of more than 4 KB above all): 4096 x 1500, K = 5: 49 / 34 (8192 rows: 59 / 65), 4096 x
//   1500, K = 100: 115 / 71, 4096 x 2048, K = 16: 77 / 44; not whole groups of 4, the LDS kernel: 1024 x 1101, K = 60: 396 / 14,
//   16384 x 1101, K = 5: 221 / 168 (32768 rows: 226 / 345), 16384 x 1501, K = 30: 400 / 206, 4096 x 2046 bf16, K = 130: 1950 / 138;
//   more than 128 clusters on fp32 rows of 769 .. 1024 channels, where the others rank in two launches or on the LDS kernel: 1024 x
//   900, K = 256: 102 / 30; 1024 x 1000, K = 129: 100 / 18; 512 x 1001, K = 256: 1352 / 25; longer rows of as many: 1024 x 2048: K =
//   129: 191 / 27, 256: 200 / 44; 1024 x 4096, K = 129: 364 / 51; 1024 x 3002, K = 256: 3931 / 83; the longest rows: 4096 x 4096, K =
//   5: 153 / 78; 4096 x 8192, K = 5: 296 / 144; 1024 x 8192, K = 50: 371 / 51; 16384 x 3002, K = 5: 614 / 372.  (3400 shapes of 1 ..
//   16384 rows, 4 .. 8192 channels and 1 .. 256 clusters: but for that instance none that comes here takes longer, to 4 %.)
bool direct_apply_pays(int64_t N, int64_t D, int32_t K, cat_dtype dt) {
    if (D > 8192 || K > 256) return false;
    const double work = (double)N * (double)D * (double)K;
    const bool rowtile = infer_supported(N, D, K, dt);
    if (rowtile && infer_two_parts(D, K, dt)) return N <= 256 || (N <= 1024 && K <= 64 && work <= 32e6);
    if (rowtile || wide_supported(N, D, K, dt)) {
        const int64_t kb = D * (dt == CAT_BF16 ? 2 : 4) / 1024;
        const bool partly = K > 180 && D % 256 != 0 && kb == 1;
        return N <= ((K > 128 && D % 4 != 0) || partly ? 512 : 1024) && work <= 256e6;
    }
    if (D <= 1024) return N <= 1024 && work <= 256e6;
    return D % 4 == 0 ? N <= 4096 && work <= 640e6 : N <= 16384 && work <= 1.1e9;
}

cat_status direct_apply(const void* lq, cat_dtype dt, int64_t N, int64_t D, int32_t K, const float* cent, const float* gamma,
                        const float* beta, float alpha, void* corrected, int32_t* assign, hipStream_t st) {
    if (D > 8192 || K > 1024 || N > ((int64_t)1 << 24))
        return set_error(CAT_ERR_UNSUPPORTED, "direct inference does not fit N=%lld D=%lld K=%d", (long long)N, (long long)D, (int)K);
    DirectParams p = {};
    p.lq = lq;
    p.N = N;
    p.D = D;
    p.K = K;
    p.cent = cent;
    p.gamma = gamma;
    p.beta = beta;
    p.alpha = alpha;
    p.out = corrected;
    p.assign = assign;
    // a sum of squares: (D / 64 + 1) terms in a lane and six levels of lanes, each term with three roundings; the sums of
    // two clusters, and as much again to be on the safe side
    p.rel = 4.f * ((float)((D + 63) / 64) + 4.f + 6.f + 3.f) * 5.96e-8f;
    const bool vec = D % 4 == 0;
    const int R = N <= 256 ? 1 : N <= 512 ? 2 : 4;  // (one workgroup per compute unit)
    const dim3 grid((unsigned)((N + R - 1) / R)), block(kDirT);
    const size_t lds = (size_t)R * (size_t)K * sizeof(float4);
    const bool prof = profile_on();
    if (prof) {
        const cat_status s = profile_mark(true, st);
        if (s != CAT_OK) return s;
    }
#define CAT_DIRECT_R(T, V, RR) hipLaunchKernelGGL((k_apply_direct<T, V, RR>), grid, block, lds, st, p)
#define CAT_DIRECT(T, V)                     \
    do {                                     \
        if (R == 1) CAT_DIRECT_R(T, V, 1);   \
        else if (R == 2) CAT_DIRECT_R(T, V, 2); \
        else CAT_DIRECT_R(T, V, 4);          \
    } while (0)
    if (dt == CAT_BF16) {
        if (vec) CAT_DIRECT(bf16_t, 4);
        else CAT_DIRECT(bf16_t, 1);
    } else {
        if (vec) CAT_DIRECT(float, 4);
        else CAT_DIRECT(float, 1);
    }
#undef CAT_DIRECT
#undef CAT_DIRECT_R
    CAT_LAUNCH_CHECK("k_apply_direct");
    if (prof) return profile_mark(false, st);
    return CAT_OK;
}

}  // namespace cat
