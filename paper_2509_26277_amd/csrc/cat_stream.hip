// Streaming (non-MFMA) kernels of the CAT hot path for gfx950: seeded init, the
// direct-form assignment / inference kernel that serves every shape, the
// segmented sums behind the centroid update and the affine statistics, and the
// small K x D finalisers.
#include "cat_common.h"

namespace cat {

// ---------------------------------------------------------------------------------
// small utilities
// ---------------------------------------------------------------------------------
__global__ void k_fill_zero(uint32_t* p, size_t nwords) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    size_t step = (size_t)gridDim.x * blockDim.x;
    for (; i < nwords; i += step) p[i] = 0u;
}
cat_status launch_fill_zero(void* p, size_t bytes, hipStream_t st) {
    if (bytes == 0) return CAT_OK;
    size_t nwords = bytes / 4;  // every workspace block is a multiple of 4 bytes
    int blocks = (int)((nwords + 255) / 256 < 2048 ? (nwords + 255) / 256 : 2048);
    hipLaunchKernelGGL(k_fill_zero, dim3(blocks), dim3(256), 0, st, (uint32_t*)p, nwords);
    CAT_LAUNCH_CHECK("k_fill_zero");
    return CAT_OK;
}

// Best-of-several bookkeeping, all on the device so that nothing waits for the host.  state[0]: 1 if the run
// just finished is the best so far (strictly lower objective, or the first run), state[1]: index of the best run.
__global__ void k_keep_best(const double* cur, double* best, int32_t* state, int32_t run, double* finals) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    const double v = *cur;
    if (finals) finals[run] = v;
    const bool take = run == 0 || v < *best;
    state[0] = take ? 1 : 0;
    if (take) {
        *best = v;
        state[1] = run;
    }
}
cat_status launch_keep_best(const double* cur, double* best, int32_t* state, int32_t run, double* finals, hipStream_t st) {
    hipLaunchKernelGGL(k_keep_best, dim3(1), dim3(64), 0, st, cur, best, state, run, finals);
    CAT_LAUNCH_CHECK("k_keep_best");
    return CAT_OK;
}
__global__ void k_copy_words_if(const int32_t* __restrict__ flag, const uint32_t* __restrict__ src, uint32_t* __restrict__ dst,
                                int64_t n) {
    if (*flag == 0) return;  // uniform
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += step) dst[i] = src[i];
}
cat_status launch_copy_words_if(const int32_t* flag, const void* src, void* dst, int64_t nwords, hipStream_t st) {
    if (nwords <= 0) return CAT_OK;
    const int64_t want = (nwords + 255) / 256;
    hipLaunchKernelGGL(k_copy_words_if, dim3((unsigned)(want < 4096 ? want : 4096)), dim3(256), 0, st, flag, (const uint32_t*)src,
                       (uint32_t*)dst, nwords);
    CAT_LAUNCH_CHECK("k_copy_words_if");
    return CAT_OK;
}

__global__ void k_copy_cols(const float* __restrict__ src, int64_t rows, int32_t src_ld, float* __restrict__ dst,
                            int32_t dst_ld, int32_t cols) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= rows * dst_ld) return;
    const int64_t r = i / dst_ld;
    const int32_t c = (int32_t)(i - r * dst_ld);
    dst[i] = c < cols ? src[r * src_ld + c] : 0.f;
}
cat_status launch_copy_cols(const float* src, int64_t rows, int32_t src_ld, float* dst, int32_t dst_ld, int32_t cols,
                            hipStream_t st) {
    const int64_t n = rows * dst_ld;
    hipLaunchKernelGGL(k_copy_cols, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, src, rows, src_ld, dst, dst_ld, cols);
    CAT_LAUNCH_CHECK("k_copy_cols");
    return CAT_OK;
}

// dst (rows x dst_ld) <- the first dst_ld columns of src (rows x src_ld), zeros where src has none (fp32 or 16-bit elements)
// In 4-byte words (bf16 rows have an even number of channels).  Rows of more than kPadFlat words: one wave per row; rows
// that are not whole 16-byte groups start anywhere on a word, so a wave instruction covers 256 consecutive bytes of the
// row instead of a lane 16 of them.  Bound by memory, a read and a write of the matrix: 50021 x 1001 to 1004 floats, 126 us
// with an element and a 64-bit division per thread, 68 us so.
constexpr int kPadWaves = 4;
__global__ __launch_bounds__(kPadWaves * kWave) void k_pad_words(const uint32_t* __restrict__ src, int64_t rows, int64_t src_w,
                                                                 int64_t dst_w, uint32_t* __restrict__ dst) {
    constexpr int U = 8;  // words in flight per lane
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t step = (int64_t)gridDim.x * kPadWaves;
    for (int64_t r = (int64_t)blockIdx.x * kPadWaves + threadIdx.x / kWave; r < rows; r += step) {
        const uint32_t* s = src + r * src_w;
        uint32_t* d = dst + r * dst_w;
        for (int64_t c0 = lane; c0 < dst_w; c0 += U * kWave) {
            uint32_t v[U];
#pragma unroll
            for (int u = 0; u < U; u++) {
                const int64_t c = c0 + u * kWave;
                v[u] = s[c < src_w ? c : src_w - 1];
            }
#pragma unroll
            for (int u = 0; u < U; u++) {
                const int64_t c = c0 + u * kWave;
                if (c < dst_w) d[c] = c < src_w ? v[u] : 0u;
            }
        }
    }
}
// Short rows leave most of a wave idle that way (879,482 x 28 bf16: 116 us, 46 us with an element per thread).  Here the
// output words are taken in order whatever row they are in, 512 consecutive ones per wave and round: 17 us there (a fit of 9 iterations 1266 -> 1190).  The row of a
// word comes from a multiplication (exact below 2^16 for divisors up to kPadFlat), the start of a round from the one before.
constexpr int kPadFlat = 192;
constexpr int kPadU = 8;
__global__ __launch_bounds__(kPadWaves * kWave) void k_pad_flat(const uint32_t* __restrict__ src, int64_t rows, uint32_t src_w,
                                                                uint32_t dst_w, uint32_t inv, uint32_t* __restrict__ dst) {
    constexpr uint32_t W = kPadU * kWave;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t n = rows * dst_w, step = (int64_t)gridDim.x * kPadWaves * W;
    int64_t i0 = ((int64_t)blockIdx.x * kPadWaves + threadIdx.x / kWave) * W;
    int64_t r0 = i0 / dst_w;
    uint32_t c0 = (uint32_t)(i0 - r0 * dst_w);
    const int64_t rstep = step / dst_w;
    const uint32_t cstep = (uint32_t)(step - rstep * dst_w);
    for (; i0 < n; i0 += step) {
        uint32_t v[kPadU];
#pragma unroll
        for (int u = 0; u < kPadU; u++) {
            const uint32_t c = c0 + lane + u * kWave, q = __umulhi(c, inv), cc = c - q * dst_w;
            const int64_t r = r0 + q < rows ? r0 + q : rows - 1;
            const uint32_t w = src[r * src_w + (cc < src_w ? cc : src_w - 1)];
            v[u] = cc < src_w ? w : 0u;
        }
#pragma unroll
        for (int u = 0; u < kPadU; u++) {
            const int64_t i = i0 + lane + u * kWave;
            if (i < n) dst[i] = v[u];
        }
        r0 += rstep;
        c0 += cstep;
        if (c0 >= dst_w) {
            c0 -= dst_w;
            r0++;
        }
    }
}
cat_status launch_pad_rows(const void* src, cat_dtype dt, int64_t rows, int64_t src_ld, int64_t dst_ld, void* dst, hipStream_t st) {
    if (rows * dst_ld == 0) return CAT_OK;
    const int64_t per = dt == CAT_F32 ? 1 : 2;
    if (src_ld % per || dst_ld % per) return set_error(CAT_ERR_INVALID_ARG, "row copy: rows of whole 4-byte words only");
    const int64_t src_w = src_ld / per, dst_w = dst_ld / per;
    if (dst_w > 1 && dst_w <= kPadFlat) {
        int64_t blocks = (rows * dst_w + kPadWaves * kPadU * kWave - 1) / (kPadWaves * kPadU * kWave);
        blocks = blocks > 2048 ? 2048 : blocks;
        hipLaunchKernelGGL(k_pad_flat, dim3((unsigned)blocks), dim3(kPadWaves * kWave), 0, st, (const uint32_t*)src, rows, (uint32_t)src_w,
                           (uint32_t)dst_w, 0xFFFFFFFFu / (uint32_t)dst_w + 1u, (uint32_t*)dst);
        CAT_LAUNCH_CHECK("k_pad_flat");
        return CAT_OK;
    }
    int64_t blocks = (rows + kPadWaves - 1) / kPadWaves;
    blocks = blocks > (1 << 16) ? (1 << 16) : blocks;
    hipLaunchKernelGGL(k_pad_words, dim3((unsigned)blocks), dim3(kPadWaves * kWave), 0, st, (const uint32_t*)src, rows, src_w, dst_w,
                       (uint32_t*)dst);
    CAT_LAUNCH_CHECK("k_pad_words");
    return CAT_OK;
}

// cat_stream_probe: a pure read (the values are folded into a word that is never stored) or a pure copy
__device__ uint32_t g_probe_sink;
typedef __attribute__((ext_vector_type(4))) uint32_t probe_u4;
template <bool COPY>
__global__ __launch_bounds__(256) void k_stream_probe(const probe_u4* __restrict__ src, probe_u4* __restrict__ dst, size_t nvec) {
    constexpr int U = 4;
    const size_t per_block = (nvec + gridDim.x - 1) / gridDim.x;
    const size_t b0 = (size_t)blockIdx.x * per_block;
    const size_t b1 = b0 + per_block < nvec ? b0 + per_block : nvec;
    uint32_t acc = 0;
    for (size_t i = b0 + threadIdx.x; i < b1; i += 256 * U) {
        probe_u4 v[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const size_t j = i + (size_t)u * 256;
            v[u] = src[j < b1 ? j : b1 - 1];
        }
#pragma unroll
        for (int u = 0; u < U; u++) {
            const size_t j = i + (size_t)u * 256;
            if (COPY) {
                if (j < b1) __builtin_nontemporal_store(v[u], dst + j);
            } else {
                acc ^= v[u].x ^ v[u].y ^ v[u].z ^ v[u].w;
            }
        }
    }
    if (!COPY && acc == 0x9E3779B9u && b1 == 1) g_probe_sink = acc;  // (never both: keeps the loads alive)
}
cat_status launch_stream_probe(const void* src, void* dst, size_t bytes, hipStream_t st) {
    const size_t nvec = bytes / 16;
    size_t blocks = (nvec + 1023) / 1024;  // spans of 16 KB do best (many short spans rather than few long ones)
    blocks = blocks > 65536 ? 65536 : (blocks < 1 ? 1 : blocks);
    if (dst)
        hipLaunchKernelGGL(k_stream_probe<true>, dim3((unsigned)blocks), dim3(256), 0, st, (const probe_u4*)src, (probe_u4*)dst, nvec);
    else
        hipLaunchKernelGGL(k_stream_probe<false>, dim3((unsigned)blocks), dim3(256), 0, st, (const probe_u4*)src, (probe_u4*)nullptr, nvec);
    CAT_LAUNCH_CHECK("k_stream_probe");
    return CAT_OK;
}

__global__ void k_fill_u64(unsigned long long* p, int64_t n, unsigned long long v) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}
cat_status launch_fill_u64(unsigned long long* p, int64_t n, unsigned long long v, hipStream_t st) {
    hipLaunchKernelGGL(k_fill_u64, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, n, v);
    CAT_LAUNCH_CHECK("k_fill_u64");
    return CAT_OK;
}

__global__ void k_copy_words(const uint32_t* src, uint32_t* dst, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += step) dst[i] = src[i];
}
cat_status launch_copy_words(const void* src, void* dst, int64_t nwords, hipStream_t st) {
    int64_t b = (nwords + 255) / 256;
    hipLaunchKernelGGL(k_copy_words, dim3((unsigned)(b < 1024 ? b : 1024)), dim3(256), 0, st, (const uint32_t*)src,
                       (uint32_t*)dst, nwords);
    CAT_LAUNCH_CHECK("k_copy_words");
    return CAT_OK;
}

// ---------------------------------------------------------------------------------
// seeded initial rows: one wave walks the SplitMix64 counter; its 64 lanes share
// the "already taken?" scan.  The walk has a hard draw cap, so the wave always exits.
// ---------------------------------------------------------------------------------
__device__ __forceinline__ void wave_lds_done() {  // a wave's LDS operations take place in order: only the compiler must keep to it
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}
// called by one wave alone: no barrier inside
__device__ __forceinline__ void draw_indices(int64_t N, int32_t K, uint64_t seed, int64_t* s_idx) {
    const int lane = threadIdx.x & (kWave - 1);
    const uint64_t cap = init_draw_cap(N);
    int32_t have = 0;
    uint64_t t = 0;
    // 64 draws at a time, one per lane: a draw is dropped if it is among those already kept or equals an earlier draw of
    // the batch, the others are kept in the order drawn (one draw at a time, with its 64-bit modulo and scan one after
    // the other, took 89 us at K = 200)
    while (have < K && t < cap) {
        const uint64_t mine = t + (uint64_t)lane;
        const int64_t cand = (int64_t)(splitmix64_at(seed, mine) % (uint64_t)N);
        bool dup = mine >= cap;
        for (int q = 0; q < have; q++) dup |= s_idx[q] == cand;
        for (int l = 0; l < kWave - 1; l++) {
            const int lo = __builtin_amdgcn_readlane((int)cand, l), hi = __builtin_amdgcn_readlane((int)(cand >> 32), l);
            dup |= l < lane && lo == (int)cand && hi == (int)(cand >> 32);
        }
        const unsigned long long keep = __ballot(!dup);
        const int at = have + __builtin_popcountll(keep & ((1ull << lane) - 1ull));
        if (!dup && at < K) s_idx[at] = cand;
        have += __builtin_popcountll(keep);
        have = have < K ? have : K;
        t += kWave;
        wave_lds_done();
    }
    // cap reached (not expected): complete with the smallest indices not yet taken
    for (int64_t c = 0; have < K && c < N; c++) {
        bool dup = false;
        for (int q = lane; q < have; q += kWave) dup |= (s_idx[q] == c);
        if (__ballot(dup) == 0ull) {
            if (lane == 0) s_idx[have] = c;
            have++;
        }
        wave_lds_done();
    }
}

template <typename T>
__global__ void k_gather_rows(const T* lq, int64_t D, const int64_t* idx, float* out) {
    const int k = blockIdx.x;
    const T* src = lq + idx[k] * D;
    for (int64_t j = threadIdx.x; j < D; j += blockDim.x) out[(int64_t)k * D + j] = ld_elem(src + j);
}
cat_status launch_gather_rows(const void* lq, cat_dtype dt, int64_t D, int32_t K, const int64_t* idx,
                              float* out, hipStream_t st) {
    if (dt == CAT_F32)
        hipLaunchKernelGGL(k_gather_rows<float>, dim3(K), dim3(256), 0, st, (const float*)lq, D, idx, out);
    else
        hipLaunchKernelGGL(k_gather_rows<bf16_t>, dim3(K), dim3(256), 0, st, (const bf16_t*)lq, D, idx, out);
    CAT_LAUNCH_CHECK("k_gather_rows");
    return CAT_OK;
}

// The seeded rows as the initial centroids.  One wave of every workgroup draws for itself, and the workgroup copies the rows that
// are its own: the draws take as long side by side as once, and a launch less is 3.5 us of a small fit.  No more workgroups than
// compute units: with one per row and every wave drawing, the scans shared the LDS of a CU from some 256 rows on (a fit of 0
// iterations, us; draws and copy as two launches / that / this: 1024 x 16, K = 1024: 2435 / 3340 / 2470; 8192 x 16, K = 1024:
// 948 / 1038 / 950; 60000 x 16, K = 512: 560 / 569 / 558; 8192 x 64, K = 128: 69 / 64 / 64).
constexpr int kSeedGroups = 256;
template <typename T>
__global__ __launch_bounds__(256) void k_seed_rows(const T* __restrict__ lq, int64_t N, int64_t D, int32_t K, uint64_t seed,
                                                   float* __restrict__ out) {
    __shared__ int64_t s_idx[CAT_MAX_K];
    if (__builtin_amdgcn_readfirstlane(threadIdx.x / kWave) == 0) draw_indices(N, K, seed, s_idx);
    __syncthreads();
    for (int k = blockIdx.x; k < K; k += gridDim.x) {
        const T* src = lq + s_idx[k] * D;
        for (int64_t j = threadIdx.x; j < D; j += blockDim.x) out[(int64_t)k * D + j] = ld_elem(src + j);
    }
}
cat_status launch_seed_rows(const void* lq, cat_dtype dt, int64_t N, int64_t D, int32_t K, uint64_t seed, float* out,
                            hipStream_t st) {
    const dim3 grid((unsigned)(K < kSeedGroups ? K : kSeedGroups)), block(256);
    if (dt == CAT_F32)
        hipLaunchKernelGGL(k_seed_rows<float>, grid, block, 0, st, (const float*)lq, N, D, K, seed, out);
    else
        hipLaunchKernelGGL(k_seed_rows<bf16_t>, grid, block, 0, st, (const bf16_t*)lq, N, D, K, seed, out);
    CAT_LAUNCH_CHECK("k_seed_rows");
    return CAT_OK;
}

// ---------------------------------------------------------------------------------
// assignment / inference, any shape: one wave per row, direct-form squared
// distances in double, strict "<" so the lowest index keeps a tie.
// ---------------------------------------------------------------------------------
constexpr int kAssignWaves = 4;

template <typename T, bool APPLY>
__global__ __launch_bounds__(kAssignWaves * kWave) void k_assign_stream(
    const T* __restrict__ lq, int64_t N, int64_t D, int32_t K, const float* __restrict__ cent,
    int32_t* __restrict__ assign, int32_t* counts, double* inertia, unsigned long long* rep,
    const float* __restrict__ gamma, const float* __restrict__ beta, T* __restrict__ out) {
    __shared__ int s_cnt[CAT_MAX_K];
    __shared__ unsigned long long s_rep[CAT_MAX_K];
    __shared__ double s_in[kAssignWaves];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const bool hist = (counts != nullptr) || (rep != nullptr);
    if (hist) {
        for (int k = threadIdx.x; k < K; k += blockDim.x) {
            s_cnt[k] = 0;
            s_rep[k] = ~0ull;
        }
        __syncthreads();
    }
    double in_acc = 0.0;
    const int64_t stride = (int64_t)gridDim.x * kAssignWaves;
    for (int64_t row = (int64_t)blockIdx.x * kAssignWaves + wave; row < N; row += stride) {
        const T* x = lq + row * D;
        double best = __builtin_inf();
        int arg = 0;
        for (int k = 0; k < K; k++) {
            const float* c = cent + (int64_t)k * D;
            double s = 0.0;
            for (int64_t j = lane; j < D; j += kWave) {
                double d = (double)ld_elem(x + j) - (double)c[j];
                s = fma(d, d, s);
            }
            s = wave_sum(s);
            if (s < best) {
                best = s;
                arg = k;
            }
        }
        if (lane == 0) {
            if (assign) assign[row] = arg;
            if (hist) {
                atomicAdd(&s_cnt[arg], 1);
                atomicMin(&s_rep[arg], (unsigned long long)row);
            }
            in_acc += best;
        }
        if (APPLY) {
            const float* g = gamma + (int64_t)arg * D;
            const float* b = beta + (int64_t)arg * D;
            T* o = out + row * D;
            for (int64_t j = lane; j < D; j += kWave) st_elem(o + j, fmaf(g[j], ld_elem(x + j), b[j]));
        }
    }
    if (hist || inertia) {
        if (lane == 0) s_in[wave] = in_acc;
        __syncthreads();
        if (hist)
            for (int k = threadIdx.x; k < K; k += blockDim.x) {
                if (counts && s_cnt[k]) atomicAdd(&counts[k], s_cnt[k]);
                if (rep && s_rep[k] != ~0ull) atomicMin(&rep[k], s_rep[k]);
            }
        if (inertia && threadIdx.x == 0) {
            double tot = 0.0;
            for (int w = 0; w < kAssignWaves; w++) tot += s_in[w];
            atomicAdd(inertia, tot);
        }
    }
}

cat_status launch_assign_stream(const void* lq, cat_dtype dt, int64_t N, int64_t D, int32_t K,
                                const float* cent, int32_t* assign, int32_t* counts, double* inertia,
                                unsigned long long* rep, const float* gamma, const float* beta,
                                void* corrected, hipStream_t st) {
    int64_t want = (N + kAssignWaves - 1) / kAssignWaves;
    unsigned blocks = (unsigned)(want < 4096 ? want : 4096);
    dim3 g(blocks), b(kAssignWaves * kWave);
    const bool apply = gamma != nullptr;
    if (dt == CAT_F32) {
        if (apply)
            hipLaunchKernelGGL((k_assign_stream<float, true>), g, b, 0, st, (const float*)lq, N, D, K, cent, assign,
                               counts, inertia, rep, gamma, beta, (float*)corrected);
        else
            hipLaunchKernelGGL((k_assign_stream<float, false>), g, b, 0, st, (const float*)lq, N, D, K, cent, assign,
                               counts, inertia, rep, gamma, beta, (float*)corrected);
    } else {
        if (apply)
            hipLaunchKernelGGL((k_assign_stream<bf16_t, true>), g, b, 0, st, (const bf16_t*)lq, N, D, K, cent, assign,
                               counts, inertia, rep, gamma, beta, (bf16_t*)corrected);
        else
            hipLaunchKernelGGL((k_assign_stream<bf16_t, false>), g, b, 0, st, (const bf16_t*)lq, N, D, K, cent,
                               assign, counts, inertia, rep, gamma, beta, (bf16_t*)corrected);
    }
    CAT_LAUNCH_CHECK("k_assign_stream");
    return CAT_OK;
}

// ---------------------------------------------------------------------------------
// counts and representative rows from a given partition
// ---------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_count_rep(const int32_t* __restrict__ assign, int64_t N, int32_t K,
                                                   int32_t* counts, unsigned long long* rep) {
    __shared__ int s_cnt[CAT_MAX_K];
    __shared__ unsigned long long s_rep[CAT_MAX_K];
    for (int k = threadIdx.x; k < K; k += blockDim.x) {
        s_cnt[k] = 0;
        s_rep[k] = ~0ull;
    }
    __syncthreads();
    int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += step) {
        int a = assign[i];
        if (a >= 0 && a < K) {
            if (counts) atomicAdd(&s_cnt[a], 1);
            // (rows come in rising order: after a cluster's first ones the minimum stands and a plain read tells)
            if (rep && (unsigned long long)i < s_rep[a]) atomicMin(&s_rep[a], (unsigned long long)i);
        }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < K; k += blockDim.x) {
        if (counts && s_cnt[k]) atomicAdd(&counts[k], s_cnt[k]);
        if (rep && s_rep[k] != ~0ull) atomicMin(&rep[k], s_rep[k]);
    }
}
cat_status launch_count_rep(const int32_t* assign, int64_t N, int32_t K, int32_t* counts,
                            unsigned long long* rep, hipStream_t st) {
    int64_t b = (N + 255) / 256;
    hipLaunchKernelGGL(k_count_rep, dim3((unsigned)(b < 1024 ? b : 1024)), dim3(256), 0, st, assign, N, K, counts,
                       rep);
    CAT_LAUNCH_CHECK("k_count_rep");
    return CAT_OK;
}

// The first row of every cluster alone: a block walks its contiguous share of the labels and stops once it has seen every
// cluster that has rows (a later row of the share cannot come before those).  On labels in no particular order that is
// after a few K rows; sorted labels make every block walk its whole share.  (k_count_rep, which looks at every label and
// merges every block's table: 22 us for 1,048,576 labels, K = 32.)
constexpr int kFirstThreads = 256, kFirstPer = 4;
__global__ __launch_bounds__(kFirstThreads) void k_first_rows(const int32_t* __restrict__ assign, int64_t N, int32_t K, int64_t share,
                                                              const int32_t* __restrict__ counts, unsigned long long* __restrict__ rep,
                                                              double* __restrict__ objective, int32_t nonneg) {
    if (blockIdx.x == 0)
        for (int t = threadIdx.x; t < nonneg; t += kFirstThreads)
            if (objective[t] < 0.0) objective[t] = 0.0;
    __shared__ uint32_t s_first[CAT_MAX_K];
    for (int k = threadIdx.x; k < K; k += kFirstThreads) s_first[k] = 0xFFFFFFFFu;
    __syncthreads();
    const int64_t b0 = (int64_t)blockIdx.x * share, b1 = b0 + share < N ? b0 + share : N;
    for (int64_t r0 = b0; r0 < b1; r0 += kFirstThreads * kFirstPer) {
        int a[kFirstPer];
#pragma unroll
        for (int u = 0; u < kFirstPer; u++) {
            const int64_t r = r0 + u * kFirstThreads + threadIdx.x;
            a[u] = r < b1 ? assign[r] : -1;
        }
#pragma unroll
        for (int u = 0; u < kFirstPer; u++) {
            const uint32_t at = (uint32_t)(r0 - b0) + u * kFirstThreads + threadIdx.x;
            if (a[u] >= 0 && a[u] < K && at < s_first[a[u]]) atomicMin(&s_first[a[u]], at);
        }
        __syncthreads();
        int all = 1;
        for (int k = threadIdx.x; k < K; k += kFirstThreads) all &= (s_first[k] != 0xFFFFFFFFu || counts[k] == 0) ? 1 : 0;
        if (__syncthreads_and(all)) break;  // uniform
    }
    for (int k = threadIdx.x; k < K; k += kFirstThreads)
        if (s_first[k] != 0xFFFFFFFFu) atomicMin(&rep[k], (unsigned long long)(b0 + s_first[k]));
}
cat_status launch_first_rows(const int32_t* assign, int64_t N, int32_t K, const int32_t* counts, unsigned long long* rep,
                             double* objective, int32_t nonneg, hipStream_t st) {
    if (N >= ((int64_t)1 << 31) || K > CAT_MAX_K) return set_error(CAT_ERR_UNSUPPORTED, "first rows: N or K too large");
    const int64_t step = kFirstThreads * kFirstPer;
    int64_t blocks = (N + step - 1) / step;
    blocks = blocks > 256 ? 256 : blocks;
    const int64_t share = ((N + blocks - 1) / blocks + step - 1) / step * step;
    hipLaunchKernelGGL(k_first_rows, dim3((unsigned)((N + share - 1) / share)), dim3(kFirstThreads), 0, st, assign, N, K, share, counts, rep,
                       objective, objective ? nonneg : 0);
    CAT_LAUNCH_CHECK("k_first_rows");
    return CAT_OK;
}

// ---------------------------------------------------------------------------------
// segmented sums.  grid = (row blocks, channel slices, cluster chunks).  A workgroup
// owns a [rows x slice] panel; each wave walks whole rows of the panel, so a row's
// cluster id is wave-uniform and the 64 lanes touch 64 different channels.  The
// panel accumulates in LDS doubles (on gfx950 the LDS f64 add runs ~20x faster than
// the f32 one) and is merged into the global doubles with one atomic per touched
// (cluster, channel) cell per workgroup.
// ---------------------------------------------------------------------------------
constexpr int kSegWaves = 8;

template <typename T, int NQ>
__global__ __launch_bounds__(kSegWaves * kWave) void k_segsum(
    const T* __restrict__ lq, const T* __restrict__ fp, const int32_t* __restrict__ assign, int64_t N, int64_t D,
    int32_t K, int32_t KC, int32_t SW, int32_t panel_rows, const float* __restrict__ pivx,
    const float* __restrict__ pivy, double* __restrict__ acc) {
    extern __shared__ double s_mem[];
    double* s_acc = s_mem;                                       // NQ x KC x SW
    float* s_px = (float*)(s_mem + (size_t)NQ * KC * SW);         // KC x SW (NQ == 4 only)
    float* s_py = s_px + (size_t)KC * SW;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t row0 = (int64_t)blockIdx.x * panel_rows;
    const int64_t ch0 = (int64_t)blockIdx.y * SW;
    const int k0 = blockIdx.z * KC;
    const int kc = (K - k0) < KC ? (K - k0) : KC;
    const int cells = KC * SW;

    for (int i = threadIdx.x; i < NQ * cells; i += blockDim.x) s_acc[i] = 0.0;
    if (NQ == 4) {
        for (int i = threadIdx.x; i < cells; i += blockDim.x) {
            int k = i / SW, c = i - k * SW;
            bool ok = (k < kc) && (ch0 + c < D);
            s_px[i] = ok ? pivx[(int64_t)(k0 + k) * D + ch0 + c] : 0.f;
            s_py[i] = ok ? pivy[(int64_t)(k0 + k) * D + ch0 + c] : 0.f;
        }
    }
    __syncthreads();

    const int64_t rend = (row0 + panel_rows < N) ? row0 + panel_rows : N;
    constexpr int RB = 4;  // rows in flight per wave: all their loads are issued before the first add
    for (int64_t rb = row0 + (int64_t)wave * RB; rb < rend; rb += (int64_t)kSegWaves * RB) {
        int a[RB];
#pragma unroll
        for (int u = 0; u < RB; u++) {
            int v = rb + u < rend ? __builtin_amdgcn_readfirstlane(assign[rb + u]) - k0 : -1;
            a[u] = (v >= 0 && v < kc) ? v : -1;  // other chunk, past the end, or an out-of-range label
        }
        for (int c = lane; c < SW && ch0 + c < D; c += kWave) {
            float xv[RB], yv[RB];
#pragma unroll
            for (int u = 0; u < RB; u++)
                if (a[u] >= 0) {
                    xv[u] = ld_elem(lq + (rb + u) * D + ch0 + c);
                    if (NQ == 4) yv[u] = ld_elem(fp + (rb + u) * D + ch0 + c);
                }
#pragma unroll
            for (int u = 0; u < RB; u++)
                if (a[u] >= 0) {
                    double* sa = s_acc + (size_t)a[u] * SW + c;
                    if (NQ == 1) {
                        atomicAdd(sa, (double)xv[u]);
                    } else {
                        // the shifts keep the raw second moments close to the centred ones
                        float xs = xv[u] - s_px[a[u] * SW + c];
                        float ys = yv[u] - s_py[a[u] * SW + c];
                        atomicAdd(sa, (double)xs);
                        atomicAdd(sa + cells, (double)ys);
                        atomicAdd(sa + 2 * cells, (double)xs * (double)xs);
                        atomicAdd(sa + 3 * cells, (double)xs * (double)ys);
                    }
                }
        }
    }
    __syncthreads();
    const int64_t KD = (int64_t)K * D;
    for (int i = threadIdx.x; i < NQ * cells; i += blockDim.x) {
        int q = i / cells;
        int r = i - q * cells;
        int k = r / SW, c = r - k * SW;
        double v = s_acc[i];
        if (k < kc && ch0 + c < D && v != 0.0) atomicAdd(acc + q * KD + (int64_t)(k0 + k) * D + ch0 + c, v);
    }
}

cat_status launch_segsum(int nq, const void* lq, const void* fp, cat_dtype dt, const int32_t* assign,
                         int64_t N, int64_t D, int32_t K, const float* pivx, const float* pivy,
                         double* acc, hipStream_t st) {
    // LDS bytes per (cluster, channel): the double accumulators, plus two float shifts for the statistics.
    // Narrow channel slices keep the merge traffic low: the global atomics of a launch total
    // (row panels) x K x D x NQ, and the number of row panels shrinks with the slice width.
    const int per_cell = (nq == 4) ? 40 : 8;
    const int budget = 64 * 1024;
    const int SW = 64;
    int KC = budget / (SW * per_cell);
    if (KC > K) KC = K;
    const int64_t slices = (D + SW - 1) / SW, kchunks = (K + KC - 1) / KC;
    // about 1024 workgroups in all
    int64_t panel_rows = (N * slices * kchunks + 1023) / 1024;
    panel_rows = (panel_rows + 31) & ~(int64_t)31;
    if (panel_rows < 256) panel_rows = 256;
    dim3 grid((unsigned)((N + panel_rows - 1) / panel_rows), (unsigned)slices, (unsigned)kchunks);
    dim3 block(kSegWaves * kWave);
    size_t lds = (size_t)KC * SW * per_cell;
#define CAT_SEG(T, NQ_)                                                                                          \
    do {                                                                                                         \
        CAT_HIP_TRY(hipFuncSetAttribute((const void*)k_segsum<T, NQ_>, hipFuncAttributeMaxDynamicSharedMemorySize, \
                                        budget)); /* (not lds: other threads may launch it with more meanwhile) */ \
        hipLaunchKernelGGL((k_segsum<T, NQ_>), grid, block, lds, st, (const T*)lq, (const T*)fp, assign, N, D, K, KC, \
                           SW, (int32_t)panel_rows, pivx, pivy, acc);                                                                 \
    } while (0)
    if (dt == CAT_F32) {
        if (nq == 1) CAT_SEG(float, 1); else CAT_SEG(float, 4);
    } else {
        if (nq == 1) CAT_SEG(bf16_t, 1); else CAT_SEG(bf16_t, 4);
    }
#undef CAT_SEG
    CAT_LAUNCH_CHECK("k_segsum");
    return CAT_OK;
}

// ---------------------------------------------------------------------------------
// segmented sums over rows ordered by cluster
// ---------------------------------------------------------------------------------
// offs[k] = number of rows in clusters below k (offs[K] = all labelled rows); cursor[k] = offs[k]
__global__ __launch_bounds__(1024) void k_sort_offsets(const int32_t* __restrict__ counts, int32_t K,
                                                       uint32_t* __restrict__ offs, uint32_t* __restrict__ cursor) {
    __shared__ uint32_t s[1024];
    const int t = threadIdx.x;
    const uint32_t mine = t < K ? (uint32_t)counts[t] : 0u;
    s[t] = mine;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
        uint32_t v = t >= o ? s[t - o] : 0u;
        __syncthreads();
        s[t] += v;
        __syncthreads();
    }
    if (t < K) {
        offs[t] = s[t] - mine;
        cursor[t] = s[t] - mine;
    }
    if (t == K - 1) offs[K] = s[t];
}

// perm[offs[k] ..] = the rows of cluster k (in no particular order)
constexpr int kSortRowsPerThread = 8;
__global__ __launch_bounds__(256) void k_sort_scatter(const int32_t* __restrict__ assign, int64_t N, int32_t K,
                                                      uint32_t* __restrict__ cursor, uint32_t* __restrict__ perm) {
    __shared__ uint32_t s_cnt[CAT_MAX_K];  // rows of this block per cluster, then their first position
    for (int k = threadIdx.x; k < K; k += blockDim.x) s_cnt[k] = 0;
    __syncthreads();
    const int64_t r0 = ((int64_t)blockIdx.x * blockDim.x) * kSortRowsPerThread + threadIdx.x;
    int a[kSortRowsPerThread];
    uint32_t rank[kSortRowsPerThread];
#pragma unroll
    for (int u = 0; u < kSortRowsPerThread; u++) {
        const int64_t r = r0 + (int64_t)u * blockDim.x;
        a[u] = r < N ? assign[r] : -1;
        if (a[u] < 0 || a[u] >= K) a[u] = -1;  // rows with a label outside [0, K) are left out, as in the counts
    }
#pragma unroll
    for (int u = 0; u < kSortRowsPerThread; u++)
        if (a[u] >= 0) rank[u] = atomicAdd(&s_cnt[a[u]], 1u);
    __syncthreads();
    for (int k = threadIdx.x; k < K; k += blockDim.x) {
        const uint32_t c = s_cnt[k];
        if (c) s_cnt[k] = atomicAdd(&cursor[k], c);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kSortRowsPerThread; u++)
        if (a[u] >= 0) perm[s_cnt[a[u]] + rank[u]] = (uint32_t)(r0 + (int64_t)u * blockDim.x);
}

// One wave per (run of R positions of the ordered rows) x (64 V channels).  The sums of the current
// cluster live in registers (doubles); when the run crosses into the next cluster, and at its end, they
// are added to acc with atomics.  V = 2 channels per lane (one 4-byte load of a bf16 row, one 8-byte load
// of an fp32 row; a wave still reads whole cache lines): measured against 16-byte loads per lane (V = 8 / 4)
// it is 1.3 - 1.5 x faster on bf16 rows and 1.1 x on fp32 rows, with a third of the registers and three
// times the waves in flight; V = 1 gains nothing more.
constexpr int kSortWaves = 4;
constexpr int kSortV = 2;
// ODD: fp32 rows of an odd length (rows start on 4 bytes, not 8): the lane's two channels are 64 apart, each a 4-byte load,
// and a wave instruction still reads 256 consecutive bytes.  (50021 x 1001, K = 200: the statistics 538 us on the
// LDS-panel kernel these rows took before, 91 so.)
// SQ (with NQ = 1): the sum of all x^2 as well, spread over kSumSqSlots entries of sumsq.
template <typename T, int NQ, bool ODD = false, bool SQ = false>
__global__ __launch_bounds__(kSortWaves * kWave) void k_segsum_sorted(
    const T* __restrict__ lq, const T* __restrict__ fp, const uint32_t* __restrict__ perm,
    const uint32_t* __restrict__ offs, int64_t D, int32_t K, int32_t R, int32_t nsl, int64_t nitems,
    const float* __restrict__ pivx, const float* __restrict__ pivy, double* __restrict__ acc, double* __restrict__ sumsq) {
    constexpr int V = kSortV;
    constexpr int RB = 4;  // rows per round; two rounds are in flight
    __shared__ uint32_t s_offs[CAT_MAX_K + 1];
    for (int k = threadIdx.x; k <= K; k += blockDim.x) s_offs[k] = offs[k];
    __syncthreads();
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t item = (int64_t)blockIdx.x * kSortWaves + wave;
    if (item >= nitems) return;
    const int slice = (int)(item % nsl);
    const uint32_t total = s_offs[K];
    const uint32_t p0 = (uint32_t)(item / nsl) * (uint32_t)R;
    const uint32_t p1 = (p0 + (uint32_t)R < total) ? p0 + (uint32_t)R : total;
    if (p0 >= p1) return;
    constexpr int CS = ODD ? kWave : 1;  // distance between the channels of a lane
    const int64_t c0 = (int64_t)slice * (kWave * V) + (int64_t)lane * (ODD ? 1 : V);
    bool on[V];  // (unless ODD, D is a multiple of V: a lane's group is inside or outside as a whole)
#pragma unroll
    for (int v = 0; v < V; v++) on[v] = c0 + v * CS < D;
    const int64_t KD = (int64_t)K * D;
    // Every load of the loop below is issued by every wave on every path (a lane outside the row reads channel 0, a
    // round past the end reads the last row again; neither is used).  The compiler counts the loads still in flight
    // at each use; a load it cannot prove was issued makes it wait for all of them, which would empty the pipeline
    // once per row.
    const int64_t cl = on[0] ? c0 : 0, cl1 = on[V - 1] ? c0 + (V - 1) * CS : 0;

    // cluster of position p0: the last k with offs[k] <= p0
    int k = 0;
    {
        int lo = 0, hi = K - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (s_offs[mid] <= p0) lo = mid; else hi = mid - 1;
        }
        k = lo;
    }
    uint32_t nextb = s_offs[k + 1];
    double sx[V], sy[V], sxx[V], sxy[V];
    float px[V], py[V];
#pragma unroll
    for (int v = 0; v < V; v++) {
        sx[v] = sy[v] = sxx[v] = sxy[v] = 0.0;
        px[v] = py[v] = 0.f;
    }
    double sq = 0.0;
    auto load_piv = [&]() {
        if (NQ == 4) {
#pragma unroll
            for (int v = 0; v < V; v++) {
                if (!on[v]) continue;
                px[v] = pivx[(int64_t)k * D + c0 + v * CS];
                py[v] = pivy[(int64_t)k * D + c0 + v * CS];
            }
        }
    };
    auto flush = [&]() {
        double* o = acc + (int64_t)k * D + c0;
#pragma unroll
        for (int v = 0; v < V; v++) {
            if (!on[v]) continue;
            atomicAdd(o + v * CS, sx[v]);
            if (NQ == 4) {
                atomicAdd(o + KD + v * CS, sy[v]);
                atomicAdd(o + 2 * KD + v * CS, sxx[v]);
                atomicAdd(o + 3 * KD + v * CS, sxy[v]);
            }
            sx[v] = sy[v] = sxx[v] = sxy[v] = 0.0;
        }
    };
    load_piv();

    // Rounds of RB rows, two register buffers: the loads of round r + 1 are requested before round r
    // is added up (each round is a gather of RB rows from anywhere in the matrix, a full memory
    // round trip).  The row numbers come 64 at a time (one per lane), one batch ahead.
    typedef __attribute__((ext_vector_type(V * sizeof(T) / 4))) uint32_t u4;  // the V channels of a lane
    const uint32_t n = p1 - p0;
    const int nr = (int)((n + RB - 1) / RB);
    uint32_t cur = perm[p0 + ((uint32_t)lane < n ? lane : n - 1)];
    uint32_t nxt = (n > (uint32_t)kWave) ? perm[p0 + (kWave + (uint32_t)lane < n ? kWave + lane : n - 1)] : 0u;
    auto advance = [&](int r) {  // entering round r: cur / nxt hold the batch of round r and the one after
        if (r > 0 && ((r * RB) & (kWave - 1)) == 0) {
            cur = nxt;
            const uint32_t nb0 = (uint32_t)(r * RB) + kWave;  // first position of the batch after this one
            nxt = nb0 < n ? perm[p0 + (nb0 + lane < n ? nb0 + lane : n - 1)] : 0u;
        }
    };
    auto issue = [&](int r, int rcur, u4 (&xv)[RB], u4 (&yv)[RB]) {  // rcur: the round being entered
        const uint32_t src = ((r * RB) >> 6) == ((rcur * RB) >> 6) ? cur : nxt;
#pragma unroll
        for (int u = 0; u < RB; u++) {
            uint32_t i = (uint32_t)(r * RB + u);
            if (i >= n) i = n - 1;  // past the end: the last row again, unused
            const int64_t row = (int64_t)__builtin_amdgcn_readlane(src, (int)(i & (kWave - 1)));
            if (ODD) {
                xv[u][0] = *(const uint32_t*)(lq + row * D + cl);
                xv[u][V * sizeof(T) / 4 - 1] = *(const uint32_t*)(lq + row * D + cl1);
                if (NQ == 4) {
                    yv[u][0] = *(const uint32_t*)(fp + row * D + cl);
                    yv[u][V * sizeof(T) / 4 - 1] = *(const uint32_t*)(fp + row * D + cl1);
                }
            } else {
                xv[u] = *(const u4*)(lq + row * D + cl);
                if (NQ == 4) yv[u] = *(const u4*)(fp + row * D + cl);
            }
        }
    };
    auto consume = [&](int r, const u4 (&xv)[RB], const u4 (&yv)[RB]) {
#pragma unroll
        for (int u = 0; u < RB; u++) {
            const uint32_t i = (uint32_t)(r * RB + u);
            if (i >= n) break;
            const uint32_t pos = p0 + i;
            if (pos >= nextb) {  // wave-uniform: the run enters another cluster
                flush();
                do {
                    k++;
                    nextb = s_offs[k + 1];
                } while (pos >= nextb);
                load_piv();
                // vmcnt(0): atomics count with the loads here and may complete out of order with them, so with any
                // of them possibly in flight every later wait in the loop would be for everything; drained once per
                // cluster boundary instead
                __builtin_amdgcn_s_waitcnt(0x0F70);
            }
            if (on[0]) {  // (a second channel past the row adds up numbers nobody keeps)
#pragma unroll
                for (int v = 0; v < V; v++) {
                    float x, y = 0.f;
                    if (sizeof(T) == 2) {
                        const uint32_t wx = xv[u][v >> 1];
                        x = (v & 1) ? __uint_as_float(wx & 0xFFFF0000u) : __uint_as_float(wx << 16);
                        if (NQ == 4) {
                            const uint32_t wy = yv[u][v >> 1];
                            y = (v & 1) ? __uint_as_float(wy & 0xFFFF0000u) : __uint_as_float(wy << 16);
                        }
                    } else {
                        x = __uint_as_float(xv[u][v & 3]);
                        if (NQ == 4) y = __uint_as_float(yv[u][v & 3]);
                    }
                    if (NQ == 1) {
                        sx[v] += (double)x;
                        if (SQ && on[v]) sq = fma((double)x, (double)x, sq);
                    } else {
                        // the shifts keep the raw second moments close to the centred ones
                        const float xs = x - px[v], ys = y - py[v];
                        sx[v] += (double)xs;
                        sy[v] += (double)ys;
                        sxx[v] = fma((double)xs, (double)xs, sxx[v]);
                        sxy[v] = fma((double)xs, (double)ys, sxy[v]);
                    }
                }
            }
        }
    };
    u4 xa[RB], ya[RB], xb[RB], yb[RB];
    issue(0, 0, xa, ya);
    for (int r = 0; r < nr; r += 2) {
        advance(r);
        issue(r + 1, r, xb, yb);
        consume(r, xa, ya);
        if (r + 1 >= nr) break;
        advance(r + 1);
        issue(r + 2, r + 1, xa, ya);
        consume(r + 1, xb, yb);
    }
    flush();
    if (SQ) {
        sq = wave_total(sq);
        if (lane == 0) atomicAdd(sumsq + (item % kSumSqSlots) * kSumSqStride, sq);
    }
}

bool segsum_sorted_supported(int nq, int64_t N, int64_t D, cat_dtype dt) {
    (void)nq;
    if (N >= ((int64_t)1 << 31) || (dt == CAT_BF16 && D % kSortV)) return false;
    // Where it pays (measured): always for bf16 rows (the LDS-panel kernel reads them two bytes per
    // lane); for fp32 rows from a few million elements on (65536 x 1000: 105 against 156 us for the
    // statistics, 47 against 64 us for the plain sums; 65536 x 256: 32 against 62 us).  Below that the two
    // launches of the ordering cost more than they save (16384 x 128: 38 against 34 us for the whole call).
    if (dt == CAT_BF16 || fast_paths_forced()) return true;
    return N * D >= ((int64_t)1 << 22);
}
size_t sort_workspace_words(int64_t N, int32_t K) { return (size_t)N + 2 * (size_t)K + 2; }

cat_status launch_segsum_sorted(int nq, const void* lq, const void* fp, cat_dtype dt, const int32_t* assign,
                                const int32_t* counts, int64_t N, int64_t D, int32_t K, const float* pivx,
                                const float* pivy, double* acc, uint32_t* sort_ws, hipStream_t st, double* sumsq) {
    uint32_t* offs = sort_ws;            // K + 1
    uint32_t* cursor = sort_ws + K + 1;  // K
    uint32_t* perm = sort_ws + 2 * (size_t)K + 2;
    hipLaunchKernelGGL(k_sort_offsets, dim3(1), dim3(1024), 0, st, counts, K, offs, cursor);
    CAT_LAUNCH_CHECK("k_sort_offsets");
    const int64_t per_block = 256 * kSortRowsPerThread;
    hipLaunchKernelGGL(k_sort_scatter, dim3((unsigned)((N + per_block - 1) / per_block)), dim3(256), 0, st, assign, N, K,
                       cursor, perm);
    CAT_LAUNCH_CHECK("k_sort_scatter");
    const int V = kSortV;
    const int nsl = (int)((D + kWave * V - 1) / (kWave * V));
    // One wave per run: as many runs as waves are resident at once (or a multiple of that), so
    // the launch has no ragged second round; a run is at least 64 rows (shorter runs only add
    // merge traffic) and at most about a thousand.
    static thread_local int slots_cache[3][2] = {{0, 0}, {0, 0}, {0, 0}}, slots_dev = -1;
    int dev = 0;
    CAT_HIP_TRY(hipGetDevice(&dev));
    if (dev != slots_dev) {
        for (auto& c : slots_cache) c[0] = c[1] = 0;
        slots_dev = dev;
    }
    const bool odd = D % V != 0;  // fp32 only (segsum_sorted_supported)
    if (odd && dt == CAT_BF16) return set_error(CAT_ERR_UNSUPPORTED, "ordered sums: bf16 rows of an odd length");
    int& slots = slots_cache[dt == CAT_BF16 ? 1 : odd ? 2 : 0][nq == 4];
    if (slots == 0) {
        const void* fn = dt == CAT_BF16 ? (nq == 1 ? (const void*)k_segsum_sorted<bf16_t, 1> : (const void*)k_segsum_sorted<bf16_t, 4>)
                         : odd          ? (nq == 1 ? (const void*)k_segsum_sorted<float, 1, true> : (const void*)k_segsum_sorted<float, 4, true>)
                                        : (nq == 1 ? (const void*)k_segsum_sorted<float, 1> : (const void*)k_segsum_sorted<float, 4>);
        int nb = 0, ncu = 0;
        CAT_HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fn, kSortWaves * kWave, 0));
        CAT_HIP_TRY(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
        slots = (nb < 1 ? 1 : nb) * (ncu < 1 ? 256 : ncu) * kSortWaves;
    }
    const int64_t work = N * nsl;
    const int64_t m = (work + (int64_t)slots * 1024 - 1) / ((int64_t)slots * 1024);
    int64_t runs = (int64_t)slots * m / nsl;
    if (runs < 1) runs = 1;
    int64_t R = (N + runs - 1) / runs;  // rows per run
    if (R < 64) R = 64;
    const int64_t nitems = ((N + R - 1) / R) * nsl;
    dim3 grid((unsigned)((nitems + kSortWaves - 1) / kSortWaves)), block(kSortWaves * kWave);
#define CAT_SEGS(T, ...)                                                                                          \
    hipLaunchKernelGGL((k_segsum_sorted<T, __VA_ARGS__>), grid, block, 0, st, (const T*)lq, (const T*)fp, perm, offs, D, K, \
                       (int32_t)R, nsl, nitems, pivx, pivy, acc, sumsq)
    if (sumsq && nq == 1) {
        if (odd) CAT_SEGS(float, 1, true, true);
        else if (dt == CAT_F32) CAT_SEGS(float, 1, false, true);
        else CAT_SEGS(bf16_t, 1, false, true);
    } else if (odd) {
        if (nq == 1) CAT_SEGS(float, 1, true); else CAT_SEGS(float, 4, true);
    } else if (dt == CAT_F32) {
        if (nq == 1) CAT_SEGS(float, 1); else CAT_SEGS(float, 4);
    } else {
        if (nq == 1) CAT_SEGS(bf16_t, 1); else CAT_SEGS(bf16_t, 4);
    }
#undef CAT_SEGS
    CAT_LAUNCH_CHECK("k_segsum_sorted");
    return CAT_OK;
}

// ---------------------------------------------------------------------------------
// K x D finalisers
// ---------------------------------------------------------------------------------
__global__ void k_finalize_centroids(const double* __restrict__ sums, const int32_t* __restrict__ counts,
                                     const float* prev, float* cent, int64_t D, int64_t KD) {  // cent may alias prev
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= KD) return;
    int n = counts[i / D];
    cent[i] = n > 0 ? (float)(sums[i] / (double)n) : prev[i];
}
cat_status launch_finalize_centroids(const double* sums, const int32_t* counts, const float* prev,
                                     float* cent, int64_t D, int32_t K, hipStream_t st) {
    int64_t KD = (int64_t)K * D;
    hipLaunchKernelGGL(k_finalize_centroids, dim3((unsigned)((KD + 255) / 256)), dim3(256), 0, st, sums, counts, prev,
                       cent, D, KD);
    CAT_LAUNCH_CHECK("k_finalize_centroids");
    return CAT_OK;
}

template <typename T>
__global__ void k_gather_pivots(const T* __restrict__ lq, const T* __restrict__ fp, int64_t D, int64_t KD,
                                const unsigned long long* __restrict__ rep, const float* __restrict__ hint,
                                float* __restrict__ pivx, float* __restrict__ pivy, double* __restrict__ acc) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= KD) return;
#pragma unroll
    for (int q = 0; q < 4; q++) acc[q * KD + i] = 0.0;  // the four sums of the statistics that follow
    int64_t k = i / D, j = i - k * D;
    unsigned long long r = rep[k];
    if (r == ~0ull) {
        pivx[i] = 0.f;
        pivy[i] = 0.f;
    } else {
        pivx[i] = hint ? hint[i] : ld_elem(lq + (int64_t)r * D + j);
        pivy[i] = ld_elem(fp + (int64_t)r * D + j);
    }
}
cat_status launch_gather_pivots(const void* lq, const void* fp, cat_dtype dt, int64_t D, int32_t K,
                                const unsigned long long* rep, const float* hint, float* pivx, float* pivy, double* acc,
                                hipStream_t st) {
    int64_t KD = (int64_t)K * D;
    dim3 g((unsigned)((KD + 255) / 256)), b(256);
    if (dt == CAT_F32)
        hipLaunchKernelGGL(k_gather_pivots<float>, g, b, 0, st, (const float*)lq, (const float*)fp, D, KD, rep, hint,
                           pivx, pivy, acc);
    else
        hipLaunchKernelGGL(k_gather_pivots<bf16_t>, g, b, 0, st, (const bf16_t*)lq, (const bf16_t*)fp, D, KD, rep,
                           hint, pivx, pivy, acc);
    CAT_LAUNCH_CHECK("k_gather_pivots");
    return CAT_OK;
}

// gamma = cov / max(var, floor), beta = mean_y - gamma * mean_x, from the shifted raw moments
__global__ void k_finalize_affine(const double* __restrict__ acc, const int32_t* __restrict__ counts,
                                  const float* __restrict__ pivx, const float* __restrict__ pivy,
                                  float* __restrict__ gamma, float* __restrict__ beta, int64_t D, int64_t KD,
                                  int32_t* __restrict__ counts_out) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= KD) return;
    int n = counts[i / D];
    if (counts_out && i % D == 0) counts_out[i / D] = n;
    if (n <= 0) {
        gamma[i] = 1.f;
        beta[i] = 0.f;
        return;
    }
    double inv = 1.0 / (double)n;
    double mx = acc[i] * inv, my = acc[KD + i] * inv;
    double var = acc[2 * KD + i] * inv - mx * mx;
    double cov = acc[3 * KD + i] * inv - mx * my;
    if (var < kVarFloor) var = kVarFloor;
    double g = cov / var;
    gamma[i] = (float)g;
    beta[i] = (float)(((double)pivy[i] + my) - g * ((double)pivx[i] + mx));
}
cat_status launch_finalize_affine(const double* acc, const int32_t* counts, const float* pivx,
                                  const float* pivy, float* gamma, float* beta, int64_t D, int32_t K,
                                  int32_t* counts_out, hipStream_t st) {
    int64_t KD = (int64_t)K * D;
    hipLaunchKernelGGL(k_finalize_affine, dim3((unsigned)((KD + 255) / 256)), dim3(256), 0, st, acc, counts, pivx,
                       pivy, gamma, beta, D, KD, counts_out);
    CAT_LAUNCH_CHECK("k_finalize_affine");
    return CAT_OK;
}

__global__ void k_fold_alpha(const float* __restrict__ gamma, const float* __restrict__ beta, float alpha,
                             float* __restrict__ g_eff, float* __restrict__ b_eff, int64_t KD) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= KD) return;
    g_eff[i] = 1.f + alpha * (gamma[i] - 1.f);
    b_eff[i] = alpha * beta[i];
}
cat_status launch_fold_alpha(const float* gamma, const float* beta, float alpha, float* g_eff, float* b_eff,
                             int64_t KD, hipStream_t st) {
    hipLaunchKernelGGL(k_fold_alpha, dim3((unsigned)((KD + 255) / 256)), dim3(256), 0, st, gamma, beta, alpha, g_eff,
                       b_eff, KD);
    CAT_LAUNCH_CHECK("k_fold_alpha");
    return CAT_OK;
}

}  // namespace cat
