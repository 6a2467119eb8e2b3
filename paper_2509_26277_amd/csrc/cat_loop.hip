// All passes of a Lloyd loop in one launch, for matrices whose passes are launches and round trips rather than traffic.
//
// As two launches a pass (k_tile, k_delta_prep) a pass over a few megabytes takes 12 .. 25 us, of which the rows are one or two:
// launches, and in each of them half a dozen dependent trips through memory (operand, rows, list, sums, counters).  Here every
// workgroup keeps its rows' tiles from the first pass to the last (the rows stay in its L2), holds the centroids in LDS (fp32 and
// the operand of k_tile), and once a pass the workgroups exchange through memory what changed:
//   rank the own rows; those that changed cluster are added to their new cluster's sums and taken from the old one's (fp64 atomics
//   in memory, many of them first combined in an LDS panel);  wait for these;  raise a flag that says which clusters they touched;
//   wait for everybody's flag;  read the sums of the touched clusters and rebuild those centroids (every workgroup for itself).
// The loop ends when no row changes any more.  What bounds it: three trips through memory in a row (additions, flags, sums, some
// 1 us each; 256 flags 2.4 us, 32 flags 0.9), the additions of all workgroups to the same addresses in the first passes, and the
// instructions of one tile.  us per cat_fit of a planted mixture, two launches a pass -> this, three seeds: 4096 x 64, K = 4, 20
// iterations: 363, 181, 275 -> 171, 74, 121; 33816 x 80, K = 37, 30: 747, 781, 764 -> 402, 397, 399; 3178 x 28, K = 123, 20: 518, 390, 346
// -> 200, 166, 143.
// From 64 MB on (BOUNDS) the passes that leave rows out by distance bounds run here too: tile_lloyd's passes 0 .. 2 read every row, the
// last of them lists the rows that changed and leaves the bounds; then every workgroup selects the due ones of its own rows, and
// the waves share the channels of a tile where a pass has few tiles.  A row within the error bound is measured at the end of the
// workgroup's tiles, by any wave.  us per cat_fit: 563519 x 40, K = 91, 30
// iterations, logits: 1986, 2098, 1999 -> 1323, 1388, 1318; 1048576 x 256, K = 32, 15, a feature map: 2453, 2102, 2639 -> 2303, 2038, 2536.
// Tried: as many copies of the sums as spread those additions (a copy more to read is a trip more: 27 % more time with two); a third and
// fourth chunk of rows in flight (registers spill, 7 .. 20 % slower); a delay before the first look at the flags (alone it makes a
// barrier of 256 workgroups 1.1 us instead of 2.4, here it is lost beside the waits for the last one to arrive).  The code has to
// stay small: at 64 KB (loops unrolled) it no longer fits the instruction cache and every phase took half as long again.
#include <atomic>

#include "cat_loop.h"
#include "cat_rank.h"
#include "cat_tile_kernel.h"

namespace cat {

constexpr int kLoopT = 512, kLoopW = kLoopT / kWave;
constexpr int kLoopMax = 256;      // workgroups
constexpr int kLoopDirect = 16;    // changed rows of a workgroup that may go to the sums without the panel (see loop_lloyd)
constexpr int kLoopList = 64;      // changed rows of a workgroup whose entries are kept in LDS too
constexpr uint32_t kLoopClosed = 0x80000000u;        // in the word that counts who has come: the loop is through
// a flag's lower word: the number of the pass, whether the rows are shared out anew after it (the first workgroup's), and in pass 0, from
// bit 16 on, the exponents of the workgroup's squared norms: the largest, and 255 less the smallest one
constexpr uint32_t kLoopTag = 0x7FFFu, kLoopRegroup = 0x8000u;
constexpr unsigned long long kLoopOver = ~0ull;      // in place of the number of a group: the loop is through

struct LoopParams {
    const void* lq;
    int64_t N;
    int32_t D, K, nsteps, iters, ntiles;
    float* cent;
    int32_t* assign;
    int32_t* counts;
    double* inertia;          // nullable
    unsigned long long* rep;
    int32_t* skipped;         // nullable
    int32_t* route;           // CAT_LOOP_RAN + members, for cat_debug_loop_route_offset
    double* sums;             // 3 x K x D; the first third zero on entry
    int32_t* dn;              // 3 x K; the first third zero on entry
    // zero on entry: [0] who has come, [1] number of the group << 32 | its members, [2] .. [5] for a change of groups: the pass to go on
    // with and `full` << 32, the drift so far, who has handed over, who has taken over; from [8] on by parity of the pass NM words a workgroup (the
    // clusters it changed, 32 to a word) and two words a workgroup (halves of its share of the objective)
    unsigned long long* words;
    unsigned long long* list; // N
    float tau, tau2;
    uint32_t off_cent, off_panel, off_small;
    int32_t W;                // channels of the panel, a multiple of 16
    int32_t share;            // waves that share the channels of a tile: 1, 2, 4 or 8 (BOUNDS: at most)
    int32_t direct;           // up to that many changed rows of a workgroup go to the sums without the panel
    int32_t looks, enough;    // the first workgroup waits that many looks for the others (and see `patience`), and for no more than `enough`
    int64_t patience;         // looks it waits on while few are there, times those
    int32_t step;             // a group has at most that many times the members of the one before
    // BOUNDS: the loop goes on after pass kLoopBounds of tile_lloyd, from that pass's sums but for the rows it listed
    double* expire;           // N: the drift at which a row has to be looked at again (see TileParams)
    int32_t* rows;            // N + 63: the members' lists of due rows
    const uint32_t* list_count;
    const int32_t* counts0;   // rows per cluster in that pass
    const double* sumsq;      // kSumSqSlots shares of the sum of |x|^2
};
constexpr int kLoopBounds = 2;
// Two launches a pass make the sums of passes 0 and 1 afresh from all rows.  Here pass 1 takes the rows that move from one sum and adds
// them to another, unless a row of large entries could leave a rounding of the sum that it was in: then, rows whose squared norms
// differ by more than 2^kLoopSpread, pass 1 is made afresh too.  us per cat_fit, always afresh / here: 3945 x 824, K = 2, 15
// iterations: 86 / 70; 15665 x 576, K = 2, 6: 107 / 90; 41877 x 136, K = 4, 25: 115 / 107; 14807 x 108 bf16, K = 4, 29: 74 / 67.
constexpr int kLoopSpread = 20;
struct LoopQueued {  // a row that is measured when the workgroup has run out of tiles
    uint32_t row;
    int prev;
    unsigned long long cand[2];
};
constexpr int kLoopQueue = 32;
static_assert(kLoopQueue * sizeof(LoopQueued) >= kLoopW * 16 * sizeof(int), "the loop without bounds keeps exponents there");
static_assert(kLoopMax <= 4 * kWave, "four words of exponents");

template <typename V>
__device__ __forceinline__ V far_load(const V* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename V>
__device__ __forceinline__ void far_store(V* p, V v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ double lane_double(double v, int l) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xFFFFFFFFll), l), hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
// halves of a double, each with the number of the pass: a word says by itself whether it is there
__device__ __forceinline__ void tagged_store(unsigned long long* at, int next, double v, uint32_t tag) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    far_store(at, (b << 32) | tag);
    far_store(at + next, (b & 0xFFFFFFFF00000000ull) | tag);
}
__device__ __forceinline__ double tagged_load(const unsigned long long* at, int next, uint32_t tag) {
    unsigned long long a, b;
    do {
        a = far_load(at);
        b = far_load(at + next);
    } while ((uint32_t)a != tag || (uint32_t)b != tag);
    return __longlong_as_double((long long)((b & 0xFFFFFFFF00000000ull) | (a >> 32)));
}
// the two largest of what the lanes hold (v1 >= v2 >= 0 each), in all lanes
template <int CTRL>
__device__ __forceinline__ double dpp_value(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xFFFFFFFFll), CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
// the larger ones of two pairs of bytes
__device__ __forceinline__ int larger_halves(int a, int b) {
    const int l = (a & 0xFF) > (b & 0xFF) ? a & 0xFF : b & 0xFF, h = (a >> 8) > (b >> 8) ? a >> 8 : b >> 8;
    return l | h << 8;
}
__device__ __forceinline__ int wave_larger(int v) {  // of all lanes
    v = larger_halves(v, __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, true));
    v = larger_halves(v, __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, true));
    v = larger_halves(v, __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, true));
    v = larger_halves(v, __builtin_amdgcn_update_dpp(0, v, 0x140, 0xF, 0xF, true));
    return larger_halves(larger_halves(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
                         larger_halves(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}
__device__ __forceinline__ void two_more(double& v1, double& v2, double o1, double o2) {
    v2 = fmax(fmin(v1, o1), fmax(v2, o2));
    v1 = fmax(v1, o1);
}
__device__ __forceinline__ void two_largest(double& v1, double& v2) {
    two_more(v1, v2, dpp_value<0xB1>(v1), dpp_value<0xB1>(v2));
    two_more(v1, v2, dpp_value<0x4E>(v1), dpp_value<0x4E>(v2));
    two_more(v1, v2, dpp_value<0x141>(v1), dpp_value<0x141>(v2));
    two_more(v1, v2, dpp_value<0x140>(v1), dpp_value<0x140>(v2));
    double r1 = lane_double(v1, 0), r2 = lane_double(v2, 0);
#pragma unroll
    for (int l = 16; l < kWave; l += 16) two_more(r1, r2, lane_double(v1, l), lane_double(v2, l));
    v1 = r1;
    v2 = r2;
}
__device__ __forceinline__ void own_memory_done() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0);
    asm volatile("" ::: "memory");
}

// Exact squared distances (fp64, direct form) of one row to two centroids in LDS, the whole wave on the row.
template <bool BF16>
__device__ __forceinline__ void near_dists(const unsigned char* xrow, int D, const float* c0, const float* c1, int lane, double& d0,
                                           double& d1) {
    constexpr int EPL = BF16 ? 8 : 4;
    double s0 = 0.0, s1 = 0.0;
    for (int j = lane * EPL; j < D; j += kWave * EPL) {
        const u32x4 w = *(const u32x4*)(xrow + (size_t)j * (BF16 ? 2 : 4));
#pragma unroll
        for (int e = 0; e < EPL; e += 4) {
            const f32x4 a = *(const f32x4*)(c0 + j + e), b = *(const f32x4*)(c1 + j + e);
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const double x = BF16 ? (double)((i & 1) ? hi_half(w[(e + i) >> 1]) : lo_half(w[(e + i) >> 1])) : (double)__uint_as_float(w[i]);
                const double u = x - (double)a[i], v = x - (double)b[i];
                s0 = fma(u, u, s0);
                s1 = fma(v, v, s1);
            }
        }
    }
    d0 = wave_total(s0);
    d1 = wave_total(s1);
}

template <int KT, bool BF16, bool BOUNDS>
__global__ __launch_bounds__(kLoopT) void k_lloyd_loop(const LoopParams p) {
    extern __shared__ __align__(16) unsigned char smem[];
    typedef typename std::conditional<BF16, bf16_t, float>::type T;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int n = lane & 15, q = lane >> 4;
    constexpr int NM = KT < 4 ? 1 : KT / 2;  // words of 32 clusters
    const int D = p.D, K = p.K, KD = K * D, W = p.W, Ds = D + 4, G = (int)gridDim.x;
    float* s_cent = (float*)(smem + p.off_cent);
    double* s_panel = (double*)(smem + p.off_panel);
    double* s_in = (double*)(smem + p.off_small);    // kLoopW
    float* s_cnorm = (float*)(s_in + kLoopW);         // KT * 16
    int* s_n = (int*)(s_cnorm + KT * 16);             // KT * 16
    int* s_dn = s_n + KT * 16;                        // KT * 16
    uint32_t* s_mask = (uint32_t*)(s_dn + KT * 16);   // 4: own changes; 2 x 4: everybody's, by parity of the pass
    // [0] rank, [1] members, [2] rows that changed, [3] queued rows, [4] due rows, [5] whether the group changes, [6] its number;
    // [8] .. [11] the exponents of the squared norms, of 64 workgroups each
    int* s_misc = (int*)(s_mask + 12);
    unsigned long long* s_list = (unsigned long long*)(s_misc + 12);  // kLoopList
    LoopQueued* s_queue = (LoopQueued*)(s_list + kLoopList);  // kLoopQueue
    float* s_score = (float*)(s_queue + kLoopQueue);  // kLoopW x KT * 16
    double* s_mv = (double*)(s_score + kLoopW * KT * 16);  // BOUNDS, KT * 16 each: squared movements; the first member: the clusters'
    double *s_obj = s_mv + KT * 16, *s_term = s_obj + KT * 16;  // terms of the objective as the centroids stand, and of the pass

    // ---- who takes part ----
    // The workgroups wait for each other, so those that wait must be resident: the members of the first group are the workgroups that
    // have come when the first one closes the door, which it does as soon as all of the grid are there or has waited long enough (see
    // run_loop: other kernels hold part of the chip).  The rows are shared out over the members there are, so every wait ends
    // whatever else runs, and nothing has to be known about the stream.  A workgroup that starts later waits for the next group: once an
    // eighth more are there, or all, the rows are shared out anew at the end of the pass.  One that starts when all is done leaves.
    if (tid == 0) {
        s_misc[0] = (int)__hip_atomic_fetch_add((uint32_t*)p.words, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_misc[2] = s_misc[3] = s_misc[4] = s_misc[5] = 0;
    }
    int* s_exp = (int*)s_queue;  // !BOUNDS, kLoopW x 16: the exponents of what a lane had in pass 0, largest | (255 - smallest) << 8
    if (tid < 12) s_mask[tid] = 0;
    if (tid < 4) s_misc[8 + tid] = 0;
    if (!BOUNDS && tid < kLoopW * 16) s_exp[tid] = 0;
    for (int i = tid; i < (int)(p.off_cent / 16); i += kLoopT) ((u32x4*)smem)[i] = (u32x4){0u, 0u, 0u, 0u};
    for (int i = tid; i < K * W; i += kLoopT) s_panel[i] = 0.0;
    if (tid < KT * 16) {
        s_n[tid] = BOUNDS && tid < K ? p.counts0[tid] : 0;
        s_dn[tid] = 0;
        s_cnorm[tid] = kPadNorm;
    }
    __syncthreads();
    const int rank = __builtin_amdgcn_readfirstlane(s_misc[0]);
    if ((uint32_t)rank & kLoopClosed) return;
    auto clear_counts = [&]() {
        if (tid < K) {
            far_store(p.counts + tid, 0);
            far_store(p.rep + tid, ~0ull);
        }
    };
    if (rank == 0 && !BOUNDS) {
        clear_counts();
        if (!BOUNDS && tid == 0 && p.inertia) far_store(p.inertia + p.iters, 0.0);
        own_memory_done();
    }

    // Norms and operand of the clusters that the wave owns (wave + kLoopW j, bit j of mine) from their fp32 values.  Of the operand's
    // 16-byte entries cluster m of a tile and lane group g take number 16 g + (m + 4 g + 2 (step & 1)) mod 16 instead of 16 g + m:
    // the channels of one cluster then lie in different banks, and what a wave reads stays 1 KB.
    const int nb = (D + kWave - 1) / kWave;
    auto emit = [&](unsigned long long mine) {
        for (; mine; mine &= mine - 1) {
            const int k = wave + kLoopW * __builtin_amdgcn_readfirstlane(__builtin_ctzll(mine));
            const float* c = s_cent + k * Ds;
            unsigned char* at = smem + (k >> 4) * 2048;
            double nn = 0.0;
#pragma unroll 2
            for (int ch = lane; ch < D; ch += kWave) {
                const float f = c[ch];
                int g, e;
                operand_slot(ch & 31, !BF16, g, e);
                const int step = ch >> 5;
                uint16_t* a = (uint16_t*)(at + step * KT * 2048 + (g * 16 + ((k + 4 * g + 2 * (step & 1)) & 15)) * 16) + e;
                const uint32_t hw = pack_bf16(f, 0.f) & 0xFFFFu;
                a[0] = (uint16_t)hw;
                a[512] = (uint16_t)(pack_bf16(f - lo_half(hw), 0.f) & 0xFFFFu);
                nn = fma((double)f, (double)f, nn);
            }
            nn = wave_total(nn);
            if (lane == 0) s_cnorm[k] = (float)nn;
        }
    };
    // The centroids of the clusters in the mask from the sums: a wave takes whole clusters, 64 channels at a time, AHEAD requests before anything waits.
    constexpr int AHEAD = 8;
    auto build = [&](const uint32_t* mask, const double* sums, const int32_t* dn, bool terms, bool last) {
        const int kd = wave + kLoopW * lane;  // lane j: the wave's cluster j
        const unsigned long long mine = __ballot(kd < K && (mask[(kd < K ? kd : 0) >> 5] >> (kd & 31) & 1u));
        if (BOUNDS && kd < K) s_mv[kd] = 0.0;
        if (mine == 0ull) return;
        int rows = kd < K ? far_load(dn + kd) : 0;
        double inv = 1.0, mv = 0.0, was = 0.0, now = 0.0;
        unsigned long long left = mine;
        int blk0 = 0;
        for (bool first = true; left; first = false) {
            double v[AHEAD];
            unsigned long long m = left;
            int blk = blk0;
#pragma unroll
            for (int u = 0; u < AHEAD; u++) {
                const int j = m ? __builtin_ctzll(m) : 0, ch = blk * kWave + lane;
                v[u] = far_load(sums + (wave + kLoopW * j) * D + (ch < D ? ch : 0));
                if (++blk == nb) {
                    blk = 0;
                    m &= m - 1;
                }
            }
            if (first) {
                if (kd < K) s_n[kd] = rows += s_n[kd];
                inv = 1.0 / (double)(rows > 0 ? rows : 1);
            }
            m = left;
            blk = blk0;
#pragma unroll
            for (int u = 0; u < AHEAD; u++) {
                const int j = m ? __builtin_ctzll(m) : 0, ch = blk * kWave + lane, k = wave + kLoopW * j;
                const int c = __builtin_amdgcn_readlane(rows, j);
                if (m && ch < D) {
                    const float old = BOUNDS ? s_cent[k * Ds + ch] : 0.f;
                    float f = old;
                    if (c > 0 && !(BOUNDS && last)) {  // v / c: the product with the reciprocal, corrected once (Markstein: the rounded quotient)
                        const double r = lane_double(inv, j), q0 = v[u] * r;
                        s_cent[k * Ds + ch] = f = (float)fma(fma(-q0, (double)c, v[u]), r, q0);
                    }
                    if (BOUNDS) {
                        const double d = (double)f - (double)old;
                        mv = fma(d, d, mv);
                        if (terms) {
                            was += (double)old * ((double)c * (double)old - 2.0 * v[u]);
                            now += (double)f * ((double)c * (double)f - 2.0 * v[u]);
                        }
                    }
                }
                if (++blk == nb) {
                    if (BOUNDS && m) {
                        mv = wave_total(mv);
                        if (lane == 0) s_mv[k] = mv;
                        if (terms) {
                            was = wave_total(was);
                            now = wave_total(now);
                            if (lane == 0) {
                                s_term[k] = was;
                                s_obj[k] = now;
                            }
                        }
                        mv = was = now = 0.0;
                    }
                    blk = 0;
                    m &= m - 1;
                }
            }
            left = m;
            blk0 = blk;
        }
        if (!(BOUNDS && last)) emit(mine);
    };
    // the centroids in memory, all of them (a workgroup that comes late may read some that are being written, and reads them again later)
    auto load_centroids = [&]() {
        int id = tid, row = D;
        asm volatile("" : "+v"(id), "+s"(row));  // (what follows from them is not to be kept in registers through the passes)
        int k = id / row, ch = id - k * row;
        const int qd = kLoopT / row, rd = kLoopT - qd * row;
#pragma unroll 4
        for (int i = id; i < KD; i += kLoopT) {
            s_cent[k * Ds + ch] = p.cent[i];
            ch += rd;
            k += qd;
            if (ch >= D) {
                ch -= D;
                k++;
            }
        }
        __syncthreads();
        emit(__ballot(wave + kLoopW * lane < K));
        __syncthreads();
    };
    // waits for a group after the one of that number which the workgroup belongs to; false: there will be none
    int M = 0;
    uint32_t group = 0;
    auto admitted = [&]() {
        if (tid == 0) {
            unsigned long long g;
            for (;;) {
                g = far_load(p.words + 1);
                if (g == kLoopOver || ((uint32_t)(g >> 32) > group && (uint32_t)rank < (uint32_t)g)) break;
                __builtin_amdgcn_s_sleep(1);
            }
            s_misc[1] = g == kLoopOver ? 0 : (int)(uint32_t)g;
            s_misc[6] = (int)(g >> 32);
        }
        __syncthreads();
        M = __builtin_amdgcn_readfirstlane(s_misc[1]);
        group = (uint32_t)__builtin_amdgcn_readfirstlane(s_misc[6]);
        return M > 0;
    };
    // The member's rows: consecutive tiles; BOUNDS: every M-th block of 64 (rows that are due lie together where the matrix is
    // sorted), of which a pass takes those that are due.  Its part of the list holds as many entries as it has rows.
    const uint32_t blocks64 = (uint32_t)((p.N + kWave - 1) / kWave);
    int t_lo = 0, t_hi = 0, z_lo = 0, z_hi = 0;  // tiles; the share of the sums to carry on
    uint32_t mine64 = 0;
    int32_t* due = nullptr;
    int64_t row_lo = 0;
    unsigned long long* own_list = nullptr;
    auto share_out = [&]() {
        t_lo = __builtin_amdgcn_readfirstlane((int)((int64_t)p.ntiles * rank / M));
        t_hi = __builtin_amdgcn_readfirstlane((int)((int64_t)p.ntiles * (rank + 1) / M));
        row_lo = (int64_t)t_lo * kRows;
        const uint32_t per = blocks64 / (uint32_t)M, extra = blocks64 % (uint32_t)M;
        mine64 = per + ((uint32_t)rank < extra ? 1u : 0u);
        if (BOUNDS) {
            row_lo = (int64_t)kWave * ((int64_t)rank * per + ((uint32_t)rank < extra ? (uint32_t)rank : extra));
            due = p.rows + row_lo;
            if ((p.N & (kWave - 1)) && (blocks64 - 1) % (uint32_t)M < (uint32_t)rank) row_lo -= kWave - (p.N & (kWave - 1));
        }
        own_list = p.list + row_lo;
        z_lo = (int)((int64_t)KD * rank / M);
        z_hi = (int)((int64_t)KD * (rank + 1) / M);
    };
    const unsigned long long* list = nullptr;
    const int nchunks = (p.nsteps + 3) / 4;
    int share = p.share, slots = kLoopW / share;
    int slot = wave / share, part = wave - slot * share;  // the wave's tile in a round, and its chunks of it
    int c_lo = nchunks * part / share, c_hi = nchunks * (part + 1) / share;
    int n_due = 0, lrow = 0;
    double gnow = 0.0, sq_total = 0.0;
    double *sums = p.sums, *sums_next = p.sums + KD, *sums_prev = p.sums + 2 * KD;
    const int k_start = (rank + wave) % K;
    double carry = 0.0;
    int32_t *dn = p.dn, *dn_next = p.dn + K, *dn_prev = p.dn + 2 * K;

    const int at_even = (q * 16 + ((n + 4 * q) & 15)) * 16, at_odd = (q * 16 + ((n + 4 * q + 2) & 15)) * 16;
    ChunkRegs<BF16> cur, next;
    f32x4 acc[KT];
    float nrm = 0.f, cmax = 0.f;
    double in_acc = 0.0;
    int full = 2;  // passes whose sums are made afresh
    int t = BOUNDS ? kLoopBounds : 0, tl = 0, cl = 0, tc = 0, cc = 0;
#pragma unroll
    for (int u = 0; u < KT; u++) acc[u] = (f32x4){0.f, 0.f, 0.f, 0.f};
    auto issue = [&](ChunkRegs<BF16>& r) {
        if (tl >= t_hi) return;
        int64_t row;
        if (BOUNDS) {
            if (cl == c_lo) {  // the number of the tile's row, and that of the tile after it
                r.row = lrow;
                const int e = (tl + slots) * kRows + n;
                lrow = due[e < n_due ? e : n_due - 1];
            } else {
                r.row = cur.row;
            }
            row = r.row;
        } else {
            const int64_t r0 = (int64_t)tl * kRows + n;
            row = r0 < p.N ? r0 : p.N - 1;
        }
        r.prev = p.assign[row];
        const T* x = (const T*)p.lq + row * D;
        const int ch = cl * kChunk + (BF16 ? 8 : 4) * q;
#pragma unroll
        for (int s = 0; s < 4; s++) {
            const int c = ch + 32 * s;
            if (BF16) {
                r.v[s] = *(const u32x4*)(x + (c < D ? c : 0));
            } else {
                r.v[2 * s] = *(const u32x4*)(x + (c < D ? c : 0));
                r.v[2 * s + 1] = *(const u32x4*)(x + (c + 16 < D ? c + 16 : 0));
            }
        }
        if (++cl == c_hi) {
            cl = c_lo;
            tl += slots;
        }
    };
    auto restart = [&]() {
        tl = tc = t_lo + slot;
        cl = cc = c_lo;
        if (BOUNDS && tl < t_hi) {
            const int e = tl * kRows + n;
            lrow = due[e < n_due ? e : n_due - 1];
        }
        issue(cur);
    };
    auto contract = [&](const ChunkRegs<BF16>& r) {
        const int s0 = 4 * cc;
        const unsigned char* base = smem + s0 * KT * 2048;
#pragma unroll
        for (int s = 0; s < 4; s++) {
            if (s > 0 && s0 + s >= p.nsteps) break;
            bf16x8 bh, bl;
            if (BF16) {
                const uint32_t m = (s0 + s) * 32 + 8 * q < D ? 0xFFFFFFFFu : 0u;
                u32x4 w = r.v[s];
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    w[j] &= m;
                    const float x0 = lo_half(w[j]), x1 = hi_half(w[j]);
                    nrm = fmaf(x0, x0, fmaf(x1, x1, nrm));
                }
                bh = bl = __builtin_bit_cast(bf16x8, w);
            } else {
                const int cf = (s0 + s) * 32 + 4 * q;
                const uint32_t m0 = cf < D ? 0xFFFFFFFFu : 0u, m1 = cf + 16 < D ? 0xFFFFFFFFu : 0u;
                float x[8];
                u32x4 h, l;
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    x[j] = __uint_as_float(r.v[2 * s][j] & m0);
                    x[4 + j] = __uint_as_float(r.v[2 * s + 1][j] & m1);
                }
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    nrm = fmaf(x[2 * j], x[2 * j], fmaf(x[2 * j + 1], x[2 * j + 1], nrm));
                    h[j] = pack_bf16(x[2 * j], x[2 * j + 1]);
                    l[j] = pack_bf16(x[2 * j] - lo_half(h[j]), x[2 * j + 1] - hi_half(h[j]));
                }
                bh = __builtin_bit_cast(bf16x8, h);
                bl = __builtin_bit_cast(bf16x8, l);
            }
#pragma unroll
            for (int u = 0; u < KT; u++) {
                const unsigned char* ap = base + (s * KT + u) * 2048 + (s & 1 ? at_odd : at_even);
                const bf16x8 ah = __builtin_bit_cast(bf16x8, *(const u32x4*)ap);
                const bf16x8 al = __builtin_bit_cast(bf16x8, *(const u32x4*)(ap + 1024));
                acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bh, acc[u], 0, 0, 0);
                acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bh, acc[u], 0, 0, 0);
                if (!BF16) acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bl, acc[u], 0, 0, 0);
            }
        }
    };
    // a row's cluster (the lanes with `on` hold one each): the label, and the lists of what changed (the first passes: of all rows)
    auto book = [&](bool on, int64_t row, int prev, int k) {
        const bool changed = on && prev != k, afresh = !BOUNDS && t < full && (t == 0 || K > 1), listed = changed || (on && afresh);
        const unsigned long long cm = __ballot(listed);
        if (!cm) return;
        int pos = 0;
        if (lane == 0) pos = atomicAdd(&s_misc[2], (int)__builtin_popcountll(cm));
        pos = __builtin_amdgcn_readfirstlane(pos) + (int)__builtin_popcountll(cm & ((1ull << lane) - 1ull));
        if (listed) {
            const unsigned long long ent = ((unsigned long long)row << 24) | ((unsigned long long)(afresh ? 0 : prev + 1) << 12) | (unsigned long long)k;
            own_list[pos] = ent;
            if (pos < kLoopList) s_list[pos] = ent;
        }
        if (changed) {
            p.assign[row] = k;
            atomicAdd(&s_dn[k], 1);
            atomicOr(&s_mask[k >> 5], 1u << (k & 31));
            if (prev >= 0) {
                atomicAdd(&s_dn[prev], -1);
                atomicOr(&s_mask[prev >> 5], 1u << (prev & 31));
            }
        }
    };
    // exact distances of a row to the clusters of `cand`, by the whole wave: the nearest, the lowest one on ties (0x7fffffff: no
    // distance compares)
    constexpr int NC = (KT + 3) / 4;
    auto measure = [&](int64_t row, unsigned long long (&cand)[NC], double& dbest) {
        dbest = __builtin_inf();
        int kbest = 0x7fffffff;
        const unsigned char* xrow = (const unsigned char*)p.lq + row * D * (int64_t)sizeof(T);
        auto take = [&]() {  // the lowest candidate left; 0x7fffffff: none
            int k = 0x7fffffff;
#pragma unroll
            for (int w = NC - 1; w >= 0; w--)
                if (cand[w]) k = 64 * w + __builtin_ctzll(cand[w]);
#pragma unroll
            for (int w = 0; w < NC; w++)
                if (k >> 6 == w) cand[w] &= cand[w] - 1;
            return __builtin_amdgcn_readfirstlane(k);
        };
        for (int ka = take(); ka != 0x7fffffff; ka = take()) {
            int kb = take();
            if (kb == 0x7fffffff) kb = ka;
            double da, db;
            near_dists<BF16>(xrow, D, s_cent + ka * Ds, s_cent + kb * Ds, lane, da, db);
            if (da < dbest) {  // (ascending: an equal one later does not win)
                dbest = da;
                kbest = ka;
            }
            if (db < dbest) {
                dbest = db;
                kbest = kb;
            }
        }
        return kbest;
    };
    auto finish = [&](int prev_in, int row_in) {
        const int64_t row0 = (int64_t)tc * kRows;
        const int64_t row = BOUNDS ? (int64_t)row_in : row0 + n;
        const bool valid = BOUNDS ? tc * kRows + n < n_due : row < p.N;
        const int prev = !BOUNDS && t == 0 ? -1 : prev_in;
        const float xn2 = sum_groups(nrm);
        float f1 = __builtin_inff(), f2 = __builtin_inff();
        int i1 = 0;
#pragma unroll
        for (int u = 0; u < KT; u++) {
            const f32x4 cn = *(const f32x4*)(s_cnorm + 16 * u + 4 * q);
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const int k = 16 * u + 4 * q + i;
                const float s = fmaf(-2.f, acc[u][i], cn[i]);
                f2 = s < f1 ? f1 : (s < f2 ? s : f2);
                i1 = s < f1 ? k : i1;
                f1 = s < f1 ? s : f1;
            }
        }
        best_two_groups(f1, i1, f2);
        i1 = i1 < K ? i1 : K - 1;  // (no real score compares: non-finite input)
        float dmin = fmaxf(xn2 + f1, 0.f);
        const float thr_in = p.tau * sqrtf(xn2) * cmax + p.tau2 * cmax * cmax;
        const bool near = valid && !(f2 - f1 > thr_in);
        bool queued = false;
        unsigned long long mask = __ballot(near && q == 0);
        while (mask) {  // rows whose two best are within the error bound: all within it are measured
            const int r = __builtin_amdgcn_readfirstlane(__builtin_ctzll(mask));
            mask &= mask - 1;
            const float thr = readlane_f(f1, r) + readlane_f(thr_in, r);
            float* sc = s_score + wave * (KT * 16);
#pragma unroll
            for (int u = 0; u < KT; u++)
                if (n == r) *(f32x4*)(sc + 16 * u + 4 * q) = acc[u];
            unsigned long long cand[NC];
#pragma unroll
            for (int w = 0; w < NC; w++) {
                const int k = 64 * w + lane;
                cand[w] = __ballot(k < K && fmaf(-2.f, sc[k < K ? k : 0], s_cnorm[k < K ? k : 0]) <= thr);
            }
            const int64_t xr = ((int64_t)__builtin_amdgcn_readlane((int)(row >> 32), r) << 32) | (int64_t)(uint32_t)__builtin_amdgcn_readlane((int)row, r);
            int pos = kLoopQueue;
            if (BOUNDS && lane == 0 && (cand[0] | cand[NC - 1]) != 0ull) pos = atomicAdd(&s_misc[3], 1);
            pos = __builtin_amdgcn_readfirstlane(pos);
            if (BOUNDS && pos < kLoopQueue) {  // by any wave, when all tiles are done
                const int pv = __builtin_amdgcn_readlane(prev, r);
                if (lane == 0) {
                    LoopQueued e;
                    e.row = (uint32_t)xr;
                    e.prev = pv;
                    e.cand[0] = cand[0];
                    e.cand[1] = NC > 1 ? cand[NC - 1] : 0ull;
                    s_queue[pos] = e;
                }
                if (n == r) queued = true;
                continue;
            }
            double dbest;
            const int kbest = measure(xr, cand, dbest);
            if (n == r && kbest != 0x7fffffff) {
                i1 = kbest;
                dmin = (float)dbest;
            }
        }
#pragma unroll
        for (int u = 0; u < KT; u++) acc[u] = (f32x4){0.f, 0.f, 0.f, 0.f};
        nrm = 0.f;
        const bool owner = q == 0 && valid && !queued;
        if (!BOUNDS && owner) {
            in_acc += (double)dmin;
            if (t == 0) {
                const int x = (int)(__float_as_uint(xn2) >> 23 & 0xFFu);
                int* at = s_exp + wave * 16 + n;
                *at = larger_halves(*at, x | (255 - x) << 8);
            }
        }
        if (BOUNDS && owner) {
            // as in finish_tile (cat_tile_kernel.h): the drift that leaves the nearest centroid the nearest
            double m = 0.0;
            if (!near) {
                const double e = (double)thr_in + (double)xn2 * (double)D * 1.5e-8;
                const double hi1 = (double)xn2 + (double)f1 + e, lo2 = (double)xn2 + (double)f2 - e;
                if (lo2 > hi1) m = (sqrt(lo2) - sqrt(hi1 > 0.0 ? hi1 : 0.0)) * (1.0 - 1e-9);
            }
            p.expire[row] = gnow + m;
        }
        book(owner, row, prev, i1);
    };

    constexpr uint32_t U = 4;  // blocks of a wave whose rows' bounds are requested at once
    double ex[U];
    auto bounds_of = [&](uint32_t i0) {
#pragma unroll
        for (uint32_t u = 0; u < U; u++) {
            const uint32_t i = i0 + kLoopW * u;
            const int64_t r = (int64_t)kWave * ((int64_t)rank + (int64_t)M * (i < mine64 ? i : mine64 - 1)) + lane;
            ex[u] = p.expire[r < p.N ? r : p.N - 1];
        }
    };

    bool settled = false, in = false, regroup = false;
    int e0 = 0, e1 = 0;  // BOUNDS: the member's share of the rows that the pass before the first listed
    for (;;) {  // groups; almost always one
        load_centroids();
        if (!in) {
            if (rank == 0 && tid == 0) {
                int come = 0;
                for (int64_t s = 0;; s++) {
                    come = (int)far_load((uint32_t*)p.words);
                    if (come >= p.enough || (s >= p.looks && s * come >= p.patience)) break;
                    __builtin_amdgcn_s_sleep(2);
                }
                far_store(p.words + 1, (1ull << 32) | (uint32_t)(come < p.enough ? come : p.enough));
            }
            if (!admitted()) return;
            in = true;
            if (group > 1) {
                __threadfence();
                continue;
            }
        }
        share_out();
        list = own_list;
        if (group > 1) {  // goes on where the last group has stopped
            const unsigned long long at = far_load(p.words + 2);
            t = __builtin_amdgcn_readfirstlane((int)at);
            full = __builtin_amdgcn_readfirstlane((int)(at >> 32));
            regroup = true;  // (BOUNDS: the bounds of its rows have not been requested yet)
            gnow = __longlong_as_double((long long)far_load(p.words + 3));
            const int turn = (t - (BOUNDS ? kLoopBounds : 0)) % 3, after = turn == 2 ? 0 : turn + 1, before = turn == 0 ? 2 : turn - 1;
            sums = p.sums + turn * KD;
            sums_next = p.sums + after * KD;
            sums_prev = p.sums + before * KD;
            dn = p.dn + turn * K;
            dn_next = p.dn + after * K;
            dn_prev = p.dn + before * K;
            if (tid < K) s_n[tid] = (int)far_load(p.rep + tid);
            own_memory_done();
            __syncthreads();
            if (tid == 0) {
                __hip_atomic_fetch_add(p.words + 5, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                while (far_load(p.words + 5) != (unsigned long long)M) __builtin_amdgcn_s_sleep(1);
            }
            __syncthreads();
            if (rank == 0 && tid < K) far_store(p.rep + tid, ~0ull);
            carry = z_lo + tid < z_hi && (BOUNDS || t >= full) ? far_load(sums_prev + z_lo + tid) : 0.0;
        } else if (BOUNDS) {
            const int64_t len = (int64_t)*p.list_count;
            e0 = (int)(len * rank / M);
            e1 = (int)(len * (rank + 1) / M);
            list = p.list + e0;
            if (tid < 4) s_mask[tid] = ~0u;
            if (rank == 0) sq_total = wave_total(p.sumsq[lane * kSumSqStride]);
            static_assert(kSumSqSlots == kWave, "one share a lane");
            if (tid == 0) s_misc[2] = e1 - e0;
            __syncthreads();
        }
        if (!BOUNDS) restart();
        for (;;) {
            // ---- assignment of the own rows ----
            if (BOUNDS && t > kLoopBounds) {  // the rows that are due
                for (uint32_t i0 = (uint32_t)wave; i0 < mine64; i0 += U * kLoopW) {
                    if (regroup || i0 != (uint32_t)wave) bounds_of(i0);
#pragma unroll
                    for (uint32_t u = 0; u < U; u++) {
                        const uint32_t i = i0 + kLoopW * u;
                        const int64_t r = (int64_t)kWave * ((int64_t)rank + (int64_t)M * i) + lane;
                        const bool is_due = i < mine64 && r < p.N && !(gnow <= ex[u]);
                        const unsigned long long m = __ballot(is_due);
                        if (!m) continue;
                        int pos = 0;
                        if (lane == 0) pos = atomicAdd(&s_misc[4], (int)__builtin_popcountll(m));
                        pos = __builtin_amdgcn_readfirstlane(pos) + (int)__builtin_popcountll(m & ((1ull << lane) - 1ull));
                        if (is_due) due[pos] = (int32_t)r;
                    }
                }
                __syncthreads();
                n_due = __builtin_amdgcn_readfirstlane(s_misc[4]);
                t_lo = 0;
                t_hi = (n_due + kRows - 1) / kRows;
                share = 1;
                while (2 * share <= p.share && t_hi * 2 * share <= kLoopW) share *= 2;
                slots = kLoopW / share;
                slot = wave / share;
                part = wave - slot * share;
                c_lo = nchunks * part / share;
                c_hi = nchunks * (part + 1) / share;
                list = own_list;
                restart();
            }
            regroup = false;
            {
                float c2 = 0.f;
                for (int k = lane; k < K; k += kWave) c2 = fmaxf(c2, s_cnorm[k]);
                c2 = fmaxf(c2, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(c2), 0xB1, 0xF, 0xF, true)));
                c2 = fmaxf(c2, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(c2), 0x4E, 0xF, 0xF, true)));
                c2 = fmaxf(c2, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(c2), 0x141, 0xF, 0xF, true)));
                c2 = fmaxf(c2, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(c2), 0x140, 0xF, 0xF, true)));
                cmax = sqrtf(fmaxf(fmaxf(readlane_f(c2, 0), readlane_f(c2, 16)), fmaxf(readlane_f(c2, 32), readlane_f(c2, 48))));
            }
            // Three buffers of sums take turns.  Pass t adds to buffer t what moves; its owner adds the sums up to pass t - 1, so that after
            // the flags of pass t buffer t holds the sums up to t.  Buffer t + 1 was read last after the flags of pass t - 2, which
            // everybody did before raising the flag of pass t - 1: it is free now, and clear before the flags of pass t.
            // The share of the sums so far moves on to this pass's (unless that adds up all rows), and the buffers of the pass that follows are cleared.
            for (int i = z_lo + tid; i < z_hi; i += kLoopT) {
                if (i != z_lo + tid) carry = t >= (BOUNDS ? kLoopBounds + 1 : full) ? far_load(sums_prev + i) : 0.0;
                if (carry != 0.0) atomicAdd(sums + i, carry);
                far_store(sums_next + i, 0.0);
            }
            if (rank == 0 && tid < K) far_store(dn_next + tid, 0);
            if (BOUNDS && rank == 0 && t == kLoopBounds + 1) clear_counts();  // (counts0 may be the same array: everybody has read it)
            in_acc = 0.0;
            int prev = -1, row = 0;
            for (int first = t_lo; first < (BOUNDS && t == kLoopBounds ? t_lo : t_hi); first += slots) {  // a round: every slot one tile
                if (tc < t_hi) {
                    prev = cur.prev;
                    row = cur.row;
                    while (cc < c_hi) {
                        issue(next);
                        contract(cur);
                        cc++;
                        cur = next;
                    }
                }
                if (share > 1) {
                    // the first of the waves that share a tile adds up what the others have (in the panel, which is left zero)
                    if (first > t_lo) __syncthreads();
                    f32x4* parts = (f32x4*)(smem + p.off_panel);
                    if (part > 0) {
                        const int at = (slot * (share - 1) + part - 1) * (KT * kWave + kWave / 4);
#pragma unroll
                        for (int u = 0; u < KT; u++) {
                            parts[at + u * kWave + lane] = acc[u];
                            acc[u] = (f32x4){0.f, 0.f, 0.f, 0.f};
                        }
                        ((float*)(parts + at + KT * kWave))[lane] = nrm;
                        nrm = 0.f;
                    }
                    __syncthreads();
                    if (part == 0) {
                        for (int i = 0; i < share - 1; i++) {
                            const int at = (slot * (share - 1) + i) * (KT * kWave + kWave / 4);
#pragma unroll
                            for (int u = 0; u < KT; u++) {
                                acc[u] += parts[at + u * kWave + lane];
                                parts[at + u * kWave + lane] = (f32x4){0.f, 0.f, 0.f, 0.f};
                            }
                            nrm += ((float*)(parts + at + KT * kWave))[lane];
                            ((float*)(parts + at + KT * kWave))[lane] = 0.f;
                        }
                    }
                }
                if (part == 0 && tc < t_hi) finish(prev, row);
                cc = c_lo;
                tc += slots;
            }
            if (BOUNDS) {
                __syncthreads();
                const int pushed = __builtin_amdgcn_readfirstlane(s_misc[3]), qn = pushed < kLoopQueue ? pushed : kLoopQueue;
                for (int e = wave; e < qn; e += kLoopW) {
                    const LoopQueued w = s_queue[e];
                    unsigned long long cand[NC];
                    cand[0] = w.cand[0];
                    if (NC > 1) cand[NC - 1] = w.cand[1];
                    const int first = cand[0] ? __builtin_ctzll(cand[0]) : kWave + __builtin_ctzll(cand[NC - 1]);
                    double dbest;
                    int k = measure((int64_t)w.row, cand, dbest);
                    if (k == 0x7fffffff) k = first;  // (non-finite input: any of them)
                    if (lane == 0) p.expire[w.row] = gnow;  // two centroids within the bound of each other: no margin
                    book(lane == 0, (int64_t)w.row, w.prev, k);
                }
            }
            if (!BOUNDS) {
                in_acc = wave_total(in_acc);
                if (lane == 0) s_in[wave] = in_acc;
            }
            own_memory_done();
            __syncthreads();
            if (!BOUNDS && t == p.iters) break;

            // ---- the rows that changed cluster move between the sums ----
            const int nch = __builtin_amdgcn_readfirstlane(s_misc[2]);
            if (nch > 0 && nch <= p.direct) {
                const unsigned long long ent = BOUNDS && t == kLoopBounds ? list[lane < nch ? lane : 0] : s_list[lane < nch ? lane : 0];
                const uint32_t e_lo = (uint32_t)ent, e_hi = (uint32_t)(ent >> 32);
                const int blocks = (D + kWave - 1) / kWave, items = nch * blocks;
                constexpr int U = BOUNDS ? 8 : 4;  // rows and blocks requested at once
                for (int i0 = wave; i0 < items; i0 += U * kLoopW) {
                    float x[U];
                    int ch[U], nw[U], od[U];
#pragma unroll
                    for (int u = 0; u < U; u++) {
                        const int it = i0 + u * kLoopW < items ? i0 + u * kLoopW : i0;
                        const int e = it / blocks;
                        ch[u] = (it - e * blocks) * kWave + lane;
                        const uint32_t lo = __builtin_amdgcn_readlane(e_lo, e), hi = __builtin_amdgcn_readlane(e_hi, e);
                        const int64_t row = (int64_t)(((unsigned long long)hi << 8) | (lo >> 24));
                        nw[u] = (int)(lo & 0xFFFu);
                        od[u] = (int)((lo >> 12) & 0xFFFu) - 1;
                        x[u] = ld_elem((const T*)p.lq + row * D + (ch[u] < D ? ch[u] : 0));
                    }
#pragma unroll
                    for (int u = 0; u < U; u++) {
                        if (i0 + u * kLoopW >= items) break;
                        if (ch[u] < D) {
                            atomicAdd(sums + nw[u] * D + ch[u], (double)x[u]);
                            if (od[u] >= 0) atomicAdd(sums + od[u] * D + ch[u], -(double)x[u]);
                        }
                    }
                }
            } else if (nch > 0) {
                const int pw = (nch + kLoopW - 1) / kLoopW, ws = wave * pw, we = ws + pw < nch ? ws + pw : nch;
                for (int c0 = 0; c0 < D; c0 += W) {
                    const int wc = D - c0 < W ? D - c0 : W;
                    for (int b = ws; b < we; b += kWave) {
                        const int nb = we - b < kWave ? we - b : kWave;
                        const unsigned long long ent = list[b + (lane < nb ? lane : 0)];
                        const uint32_t e_lo = (uint32_t)ent, e_hi = (uint32_t)(ent >> 32);
                        constexpr int RB = 8, CB = 2;
                        for (int i0 = 0; i0 < nb; i0 += RB)
                            for (int cb = 0; cb < wc; cb += CB * kWave) {
                                float x[RB][CB];
                                int nw[RB], od[RB];
#pragma unroll
                                for (int u = 0; u < RB; u++) {
                                    const int i = i0 + u < nb ? i0 + u : nb - 1;
                                    const uint32_t lo = __builtin_amdgcn_readlane(e_lo, i), hi = __builtin_amdgcn_readlane(e_hi, i);
                                    const int64_t row = (int64_t)(((unsigned long long)hi << 8) | (lo >> 24));
                                    nw[u] = i0 + u < nb ? (int)(lo & 0xFFFu) : -1;
                                    od[u] = i0 + u < nb ? (int)((lo >> 12) & 0xFFFu) - 1 : -1;
                                    const T* xr = (const T*)p.lq + row * D + c0;
#pragma unroll
                                    for (int w = 0; w < CB; w++) {
                                        const int c = cb + w * kWave + lane;
                                        if (cb + w * kWave < wc) x[u][w] = ld_elem(xr + (c < wc ? c : 0));
                                    }
                                }
#pragma unroll
                                for (int u = 0; u < RB; u++)
#pragma unroll
                                    for (int w = 0; w < CB; w++) {
                                        const int c = cb + w * kWave + lane;
                                        if (c < wc) {
                                            if (nw[u] >= 0) atomicAdd(s_panel + nw[u] * W + c, (double)x[u][w]);
                                            if (od[u] >= 0) atomicAdd(s_panel + od[u] * W + c, -(double)x[u][w]);
                                        }
                                    }
                            }
                    }
                    __syncthreads();
                    int k = k_start;  // (the workgroups start at different clusters: not all at one address)
                    for (int i = wave; i < K; i += kLoopW) {
                        for (int c = lane; c < wc; c += kWave) {
                            const double v = s_panel[k * W + c];
                            if (v != 0.0) {
                                atomicAdd(sums + k * D + c0 + c, v);
                                s_panel[k * W + c] = 0.0;
                            }
                        }
                        k += kLoopW;
                        while (k >= K) k -= K;
                    }
                    if (c0 + W < D) __syncthreads();
                }
            }
            if (nch > 0 && tid < K) {
                const int d = s_dn[tid];
                if (d) {
                    atomicAdd(dn + tid, d);
                    s_dn[tid] = 0;
                }
            }
            if (nch > 0) {
                own_memory_done();
                __syncthreads();
            }
            unsigned long long* flags = p.words + 8 + (t & 1) * (NM + 2) * G;
            const int par = t & 1;
            uint32_t exps = 0;
            if (!BOUNDS && t == 0 && wave == 0) exps = (uint32_t)wave_larger(larger_halves(s_exp[lane], s_exp[lane + kWave]));
            if (tid < NM) {
                uint32_t tag = (uint32_t)(t + 1) & kLoopTag;
                if (!BOUNDS && t == 0 && tid == 0) tag |= exps << 16;
                // others have come since (not before the last pass, which nothing follows that would wait for the first workgroup)
                if (tid == 0 && rank == 0 && M < G && t + 1 < p.iters) {
                    const int come = (int)far_load((uint32_t*)p.words);
                    if (come == G || come > M + M / 8) tag |= kLoopRegroup;
                }
                far_store(flags + tid * G + rank, ((unsigned long long)s_mask[tid] << 32) | tag);
                s_mask[tid] = 0;
                s_mask[4 + 4 * (par ^ 1) + tid] = 0;
            }
            if (tid == 0) {
                if (!BOUNDS) {
                    double v = 0.0;
#pragma unroll
                    for (int w = 0; w < kLoopW; w++) v += s_in[w];
                    tagged_store(flags + NM * G + rank, G, v, (uint32_t)(t + 1));
                }
                s_misc[2] = s_misc[3] = s_misc[4] = 0;
            }
            // ---- wait for the others; the first rows (bounds) of the next pass travel meanwhile ----
            if (BOUNDS) bounds_of((uint32_t)wave);
            else restart();
            for (int i0 = wave * kWave; i0 < NM * kLoopMax; i0 += kLoopT) {
                const int w = i0 / kLoopMax, m0 = i0 - w * kLoopMax;
                if (m0 >= M) continue;
                const unsigned long long* f = flags + w * G + (m0 + lane < M ? m0 + lane : M - 1);
                unsigned long long v = far_load(f);
                while (__any(((uint32_t)v & kLoopTag) != ((uint32_t)(t + 1) & kLoopTag))) v = far_load(f);
                if (w == 0 && lane == 0 && ((uint32_t)v & kLoopRegroup)) s_misc[5] = 1;
                if (!BOUNDS && t == 0 && w == 0) {
                    const int x = wave_larger((int)((uint32_t)v >> 16));
                    if (lane == 0) s_misc[8 + wave] = x;
                }
                const uint32_t bits = (uint32_t)(v >> 32);
                if (bits) atomicOr(&s_mask[4 + 4 * par + w], bits);
            }
            __syncthreads();
            if (!BOUNDS && t == 0) {
                const int x = __builtin_amdgcn_readfirstlane(larger_halves(larger_halves(s_misc[8], s_misc[9]), larger_halves(s_misc[10], s_misc[11])));
                full = (x & 0xFF) + (x >> 8) - 255 > kLoopSpread ? 2 : 1;
            }
            if (!BOUNDS && rank == 0 && wave == kLoopW - 1 && p.inertia) {
                double v = 0.0;
                for (int m = lane; m < M; m += kWave) v += tagged_load(flags + NM * G + m, G, (uint32_t)(t + 1));
                v = wave_total(v);
                if (lane == 0) p.inertia[t] = v;
            }
            const uint32_t* mask = s_mask + 4 + 4 * par;
            uint32_t any = mask[0];
#pragma unroll
            for (int w = 1; w < NM; w++) any |= mask[w];
            if (__builtin_amdgcn_readfirstlane(any) == 0u) {
                settled = true;
                break;
            }
            // ---- the next centroids ----
            const bool last = BOUNDS && t == p.iters;
            if (last && rank != 0) break;
            if (z_lo + tid < z_hi && (BOUNDS || t >= full - 1)) carry = far_load(sums + z_lo + tid);
            build(mask, sums, dn, BOUNDS && rank == 0 && p.inertia, last);
            __syncthreads();
            if (BOUNDS && rank == 0 && wave == kLoopW - 1 && p.inertia && t > kLoopBounds) {
                // sum |x|^2 + sum_k c_k . (n_k c_k - 2 S_k), the centroids as they were in this pass
                double v = 0.0;
                for (int k = lane; k < K; k += kWave) v += mask[k >> 5] >> (k & 31) & 1u ? s_term[k] : s_obj[k];
                v = wave_total(v) + sq_total;
                if (lane == 0) p.inertia[t] = v > 0.0 ? v : (v == v ? 0.0 : v);
            }
            if (last) break;
            if (BOUNDS) {
                // how far the centroids have moved in all (select_rows in cat_tile_kernel.h), and the rows that are due
                double v1 = lane < K ? s_mv[lane] : 0.0, v2 = 0.0;
                if (KT > 4) {
                    const double o = lane + kWave < K ? s_mv[lane + kWave] : 0.0;
                    v2 = fmin(v1, o);
                    v1 = fmax(v1, o);
                }
                v1 = fmax(sqrt(v1), 0.0);
                v2 = fmax(sqrt(v2), 0.0);
                two_largest(v1, v2);
                const double g0 = gnow;
                gnow = g0 + (v1 + v2) * (1.0 + 1e-9);
                if (v1 + v2 > 0.0 && gnow == g0) gnow = __longlong_as_double(__double_as_longlong(g0) + 1);  // (drifts are >= 0)
            }
            {
                double* s = sums_prev;
                sums_prev = sums;
                sums = sums_next;
                sums_next = s;
                int32_t* d = dn_prev;
                dn_prev = dn;
                dn = dn_next;
                dn_next = d;
            }
            t++;
            regroup = __builtin_amdgcn_readfirstlane(s_misc[5]) != 0;
            if (regroup) break;
        }
        if (!regroup) break;
        // ---- another group: those who are there now share the rows out anew ----
        // What a row's owner keeps of it (label, bound) is in memory, and the sums are; the first workgroup leaves the rest there: the
        // centroids where they are returned, the rows per cluster in the words of `rep`.
        if (rank == 0) {
            for (int k = wave; k < K; k += kLoopW)
                for (int ch = lane; ch < D; ch += kWave) far_store(p.cent + k * D + ch, s_cent[k * Ds + ch]);
            if (tid < K) far_store(p.rep + tid, (unsigned long long)(uint32_t)s_n[tid]);
            if (tid == 0) {
                far_store(p.words + 2, ((unsigned long long)full << 32) | (uint32_t)t);
                far_store(p.words + 3, (unsigned long long)__double_as_longlong(gnow));
            }
        }
        __threadfence();
        own_memory_done();
        __syncthreads();
        if (tid == 0) {
            s_misc[5] = 0;
            __hip_atomic_fetch_add(p.words + 4, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (rank == 0) {
                while (far_load(p.words + 4) != (unsigned long long)M) __builtin_amdgcn_s_sleep(1);
                far_store(p.words + 4, 0ull);
                far_store(p.words + 5, 0ull);
                own_memory_done();
                const int come = (int)far_load((uint32_t*)p.words), most = M * p.step;
                far_store(p.words + 1, ((unsigned long long)(group + 1) << 32) | (uint32_t)(come < most ? come : most));
            }
        }
        admitted();
        __threadfence();
    }
    if (rank == 0 && tid == 0) {
        __hip_atomic_fetch_or((uint32_t*)p.words, kLoopClosed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        far_store(p.words + 1, kLoopOver);
    }

    // ---- what is returned ----
    if (!BOUNDS && !settled && tid == 0 && p.inertia) {
        double v = 0.0;
#pragma unroll
        for (int w = 0; w < kLoopW; w++) v += s_in[w];
        atomicAdd(p.inertia + p.iters, v);
    }
    if (settled && rank == 0 && wave == kLoopW - 1 && p.inertia) {
        double v = 0.0;
        if (BOUNDS) {
            for (int k = lane; k < K; k += kWave) v += s_obj[k];
            v = wave_total(v) + sq_total;
            v = v > 0.0 ? v : (v == v ? 0.0 : v);
        } else {
            own_memory_done();  // (the entry of this pass, by this wave)
            v = p.inertia[t];
        }
        for (int i = t + (BOUNDS ? 0 : 1) + lane; i <= p.iters; i += kWave) p.inertia[i] = v;
    }
    if (rank == 0 && tid == 0 && p.skipped) *p.skipped = settled && p.iters - 1 > (t > 2 ? t : 2) ? p.iters - 1 - (t > 2 ? t : 2) : 0;
    if (rank == 0 && tid == 0) *p.route = CAT_LOOP_RAN + M;
    int* s_hist = s_dn;
    unsigned long long* s_rep = (unsigned long long*)s_panel;  // (a panel has at least 16 channels)
    if (tid < K) {
        s_hist[tid] = 0;
        s_rep[tid] = ~0ull;
    }
    __syncthreads();
    if (BOUNDS) {
        for (uint32_t i = (uint32_t)wave; i < mine64; i += kLoopW) {
            const int64_t r = (int64_t)kWave * ((int64_t)rank + (int64_t)M * i) + lane;
            if (r < p.N) {
                const int a = p.assign[r];
                atomicAdd(&s_hist[a], 1);
                atomicMin(&s_rep[a], (unsigned long long)r);
            }
        }
    } else {
        const int64_t row_hi = (int64_t)t_hi * kRows < p.N ? (int64_t)t_hi * kRows : p.N;
        for (int64_t i = row_lo + tid; i < row_hi; i += kLoopT) {
            const int a = p.assign[i];
            atomicAdd(&s_hist[a], 1);
            atomicMin(&s_rep[a], (unsigned long long)i);
        }
    }
    __syncthreads();
    if (tid < K && s_hist[tid]) {
        atomicAdd(p.counts + tid, s_hist[tid]);
        atomicMin(p.rep + tid, s_rep[tid]);
    }
    for (int k = rank; k < K; k += M)
        for (int j = tid; j < D; j += kLoopT) p.cent[k * D + j] = s_cent[k * Ds + j];
}

static std::atomic<int> g_loop_members{0};  // cat_debug_loop

// (what concerns the launches of a pass, hooks and the record of their times, keeps two launches a pass)
static bool loops_on(int32_t iters) {
    if (iters >= (int32_t)kLoopTag) return false;  // (a flag has that many numbers for a pass)
    return g_loop_members.load() >= 0 && lloyd_list_capacity() == kListCap && rerank_queue_capacity() == kQueueCap && !profile_on();
}

struct LoopCfg {
    bool ok = false;
    int KT = 0, nsteps = 0, W = 0;
    uint32_t off_cent = 0, off_panel = 0, off_small = 0;
    size_t lds = 0;
};
static LoopCfg loop_config(int64_t N, int64_t D, int32_t K, cat_dtype dt, bool bounds = false) {
    LoopCfg c;
    if (N < 256 || N >= ((int64_t)1 << 31) - 16 || K > 128 || D % (dt == CAT_BF16 ? 8 : 4) || (K + 15) / 16 * 16 * D > 16384) return c;
    c.KT = 1;
    while (c.KT * 16 < K) c.KT *= 2;
    c.nsteps = (int)((D + 31) / 32);
    c.off_cent = (uint32_t)(c.nsteps * c.KT * 2048);
    c.off_panel = c.off_cent + (uint32_t)(K * (D + 4) * 4);
    const size_t small = (size_t)c.KT * 16 * (4 + 4 + 4) + kLoopW * 8 + 24 * 4 + kLoopList * 8 + kLoopQueue * sizeof(LoopQueued) +
                         (size_t)kLoopW * c.KT * 16 * 4 + (bounds ? 3 * (size_t)c.KT * 16 * 8 : 0);
    if (c.off_panel + small + (size_t)K * 16 * 8 > kLdsLimit) return c;
    int64_t W = (int64_t)((kLdsLimit - small - c.off_panel) / ((size_t)K * 8)) / 16 * 16;
    const int64_t Dr = (D + 15) / 16 * 16;
    if (W > Dr) W = Dr;
    if (W > 64 && W < Dr) W = W / 64 * 64;
    c.W = (int)W;
    c.off_small = c.off_panel + (uint32_t)(K * W * 8);
    c.lds = c.off_small + small;
    c.ok = true;
    return c;
}

// Few tiles of long rows: several waves share the channels of a tile (what the others have goes through the panel).  us per cat_fit,
// one wave a tile / as here: 2958 x 984 bf16, K = 14: 159 / 115 (8 waves); 2652 x 640, K = 11: 279 / 187 (4); 7294 x 776, K = 3: 133 / 115 (4);
// 14629 x 998 bf16, K = 4: 273 / 230 (2)
static int loop_share(const LoopCfg& c, int64_t N, int32_t K, int cus, bool bounds) {
    int share = 1;
    while (share < kLoopW && 2 * share <= (c.nsteps + 3) / 4 && (bounds || (N + kRows - 1) / kRows * 2 * share <= (int64_t)cus * kLoopW) &&
           (size_t)(kLoopW - kLoopW / (2 * share)) * (c.KT * 1024 + 256) <= (size_t)K * c.W * 8)
        share *= 2;
    return share;
}
static int loop_groups(int64_t N, int share, int cus, bool bounds) {
    int64_t groups = bounds ? (N + kWave - 1) / kWave : ((N + kRows - 1) / kRows * share + kLoopW - 1) / kLoopW;
    if (groups > cus) groups = cus;
    return (int)(groups < kLoopMax ? groups : kLoopMax);
}

// Below 64 MB, where the passes keep no distance bounds (cat_tile.hip), and the centroids fit LDS twice (loop_config): where one launch
// saves more than it costs.  Against two launches a pass, us per fit, by least squares over 1300 fits (256 .. 700000 rows of 16 .. 1024
// channels, K = 1 .. 128, 1 .. 32 iterations, four kinds of data):
//   saved: 6 a pass (launches, trips) and 4 more in the first four, and 400 per million rows (no sort by cluster for the full sums);
//   lost: 16 per million additions to the sums in memory if every workgroup adds to all of them, once a full pass; 70 per thousand rows
//   of a workgroup for each part of the channels that the panel takes at a time; 1.5 per million entries of bf16 rows (the rows of
//   a tile kernel come faster, and there are twice as many to 64 MB), less with fewer than eight clusters.
// Both sides, two launches / one: 28835 x 1000 bf16, K = 16, 4 iterations 230 / 420 (two here); 60074 x 480 bf16, K = 16, 10: 430 / 525
// (two); 14417 x 1000, K = 16, 4: 222 / 281 (two); 1715 x 136 bf16, K = 98, 2: 116 / 206 (two); 30037 x 480, K = 16, 10: 359 / 283 (one);
// 6291 x 1000 bf16, K = 3, 10: 174 / 132 (one); 89422 x 296 bf16, K = 1, 5: 344 / 196 (one).  Over 1460 other fits of the same ranges: 1.79 times
// as fast on average, 1.0005 times what the faster way takes; three more than 2 % slower than two launches a pass, the worst 266 / 291 (42629 x
// 456 bf16, K = 7, 6 iterations).
bool loop_pays(int64_t N, int64_t D, int32_t K, int32_t iters, cat_dtype dt) {
    if ((double)N * (double)D * (dt == CAT_BF16 ? 2.0 : 4.0) >= 64.0 * 1024 * 1024 || iters < 1 || !loops_on(iters)) return false;
    const LoopCfg c = loop_config(N, D, K, dt);
    if (!c.ok || g_loop_members.load() > 0) return c.ok;
    const double groups = loop_groups(N, loop_share(c, N, K, kLoopMax, false), kLoopMax, false);
    const double saved = 6.0 * iters + 4.0 * (iters < 4 ? iters : 4) + 400e-6 * (double)N;
    const double lost = 16e-6 * groups * (double)K * (double)D + 70e-3 * (double)N / groups * (double)((D + c.W - 1) / c.W) +
                        (dt == CAT_BF16 ? 1.5e-6 * (double)N * (double)D * (K < 8 ? K / 8.0 : 1.0) : 0.0);
    return saved - lost > 10.0;
}

// clears the words and the sums of the first pass
__global__ __launch_bounds__(256) void k_loop_clear(unsigned long long* a, int na, double* b, int nb) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < na) a[i] = 0ull;
    if (i < nb) b[i] = 0.0;
}

template <int KT, bool BF16, bool BOUNDS>
static cat_status launch_loop(const LoopParams& p, const LoopCfg& c, int groups, hipStream_t st) {
    auto kern = k_lloyd_loop<KT, BF16, BOUNDS>;
    // (the most there is, not what this call needs: another thread may launch the same kernel with more meanwhile)
    CAT_HIP_TRY(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsLimit));
    hipLaunchKernelGGL(kern, dim3((unsigned)groups), dim3(kLoopT), c.lds, st, p);
    CAT_LAUNCH_CHECK("k_lloyd_loop");
    return CAT_OK;
}

static cat_status run_loop(const void* lq, cat_dtype dt, int64_t N, int64_t D, int32_t K, int32_t iters, float* cent_io, double* sums,
                           int32_t* assign, int32_t* counts, double* inertia, unsigned long long* rep, int32_t* skipped,
                           const LloydWs& lw, const LoopBounds* lb, hipStream_t st) {
    const LoopCfg c = loop_config(N, D, K, dt, lb != nullptr);
    if (!c.ok) return set_error(CAT_ERR_UNSUPPORTED, "loop in one launch: N=%lld D=%lld K=%d", (long long)N, (long long)D, (int)K);
    LoopParams p = {};
    p.lq = lq;
    p.N = N;
    p.D = (int32_t)D;
    p.K = K;
    p.nsteps = c.nsteps;
    p.iters = iters;
    p.ntiles = (int32_t)((N + kRows - 1) / kRows);
    p.cent = cent_io;
    p.assign = assign;
    p.counts = counts;
    p.inertia = inertia;
    p.rep = rep;
    p.skipped = skipped;
    p.route = lw.skipped;  // (none of the loops here uses that word otherwise)
    p.sums = sums;
    p.list = lw.list;
    if (lb) {
        p.expire = lb->expire;
        p.rows = lb->rows;
        p.list_count = lb->list_count;
        p.counts0 = lb->counts;
        p.sumsq = lw.sumsq;
    }
    p.tau2 = kSplitTau2;
    p.off_cent = c.off_cent;
    p.off_panel = c.off_panel;
    p.off_small = c.off_small;
    p.W = c.W;
    int dev = 0, v = 0;
    static std::atomic<int> ncu[16];
    CAT_HIP_TRY(hipGetDevice(&dev));
    v = dev < 16 ? ncu[dev].load() : 0;
    if (v == 0) {
        CAT_HIP_TRY(hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev));
        if (dev < 16) ncu[dev].store(v);
    }
    p.share = loop_share(c, N, K, v, lb != nullptr);
    // (shared channels are added up once more)
    const int n_acc = (dt == CAT_BF16 ? 2 : 3) * ((c.nsteps + 3) / 4 * 4) + 8 + (p.share - 1);
    p.tau = split_tau(dt, n_acc);
    const int groups = loop_groups(N, p.share, v, lb != nullptr);
    // Rows that go to the sums directly come to 2 rows / K additions an address and workgroup, through the panel to one at most; all
    // workgroups add to the same addresses.  us per cat_fit with up to 2 / 4 / 16 rows directly, as the loop was when this was chosen: 89551 x 128 bf16, K = 7 (256 workgroups)
    // 242 / 268 / 308; 7294 x 776, K = 3 (228) 115 / 115 / 150; 14629 x 998 bf16, K = 4 (229) 249 / 228 / 233; 4096 x 64, K = 4 (32)
    // 194 / 189 / 188; 2652 x 640, K = 11 192 / 185 / 186.
    p.direct = 64 * K / groups * (int)((D + c.W - 1) / c.W);
    if (p.direct < 3) p.direct = 3;
    if (p.direct > kLoopDirect) p.direct = kLoopDirect;
    const int members = g_loop_members.load();
    p.enough = members > 0 && members < groups ? members : groups;
    p.step = members > 0 ? 4 : kLoopMax;
    // A look takes some 0.75 us.  On an idle chip all are there within three; a group that lacks some waits for ten, and for as long as
    // its members would take for a pass (about 40 GB/s each) while that is longer: then the end of another kernel is as likely
    // as not to come first.  us, two launches a pass / this / this with the first group for good: two fits side by side on two streams: 30037 x 480,
    // K = 16, 10 iterations 613 / 662 / 1508 (alone 400 / 345); 1048576 x 256, K = 32, 15: 7555 / 7740 / 14434 (3950 / 3880); 14629 x 998
    // bf16, K = 4, 20: 564 / 700 / 846 (335 / 287); 4096 x 64, K = 4, 20: 542 / 268 / 290 (385 / 208); a fit beside three products of 8192 x 8192 matrices
    // in bf16: 33816 x 80, K = 37, 30: 3409 / 2586 / 3056.
    p.looks = 10;
    p.patience = (int64_t)((double)N * (double)D * (dt == CAT_BF16 ? 2.0 : 4.0) / 30000.0);
    // The words lie in the scratch of the counting sort, 4 N + 8 K + 8 bytes: 64 + 16 (NM + 2) groups + 12 K are needed, NM <= 4, and there are
    // at most N share / 128 + 1 groups of rows that `share` <= 8 waves work on (272 x 112, K = 104: five, 1792 of 1928 bytes, the narrowest)
    const int nm = c.KT < 4 ? 1 : c.KT / 2;
    if (64 + 16 * (int64_t)(nm + 2) * groups + 12 * (int64_t)K > 4 * N + 8 * (int64_t)K + 8)
        return set_error(CAT_ERR_WORKSPACE, "loop in one launch: the scratch of %lld rows does not hold the words of %d workgroups", (long long)N, groups);
    p.words = (unsigned long long*)lw.sort_ws;
    p.dn = (int32_t*)(p.words + 8 + 2 * (nm + 2) * groups);
    const int nwords = 8 + 2 * (nm + 2) * groups + (K + 1) / 2, nsums = lb ? 0 : K * (int)D;
    hipLaunchKernelGGL(k_loop_clear, dim3((unsigned)(((nwords > nsums ? nwords : nsums) + 255) / 256)), dim3(256), 0, st, p.words, nwords, sums, nsums);
    CAT_LAUNCH_CHECK("k_loop_clear");
    const bool bf = dt == CAT_BF16;
#define CAT_LOOP(KT)                                                                                                          \
    (lb ? bf ? launch_loop<KT, true, true>(p, c, groups, st) : launch_loop<KT, false, true>(p, c, groups, st)                  \
        : bf ? launch_loop<KT, true, false>(p, c, groups, st) : launch_loop<KT, false, false>(p, c, groups, st))
    switch (c.KT) {
        case 1: return CAT_LOOP(1);
        case 2: return CAT_LOOP(2);
        case 4: return CAT_LOOP(4);
        default: return CAT_LOOP(8);
    }
#undef CAT_LOOP
}

cat_status loop_lloyd(const void* lq, cat_dtype dt, int64_t N, int64_t D, int32_t K, int32_t iters, float* cent_io, double* sums,
                      int32_t* assign, int32_t* counts, double* inertia, unsigned long long* rep, int32_t* skipped,
                      const LloydWs& lw, hipStream_t st) {
    return run_loop(lq, dt, N, D, K, iters, cent_io, sums, assign, counts, inertia, rep, skipped, lw, nullptr, st);
}

// Fits of 64 to 500 MB, two launches a pass against this, 540 random ones (24 .. 256 channels, K = 1 .. 128, 3 .. 30 iterations, four kinds of
// data).  Where the panel takes whole rows at once: 0.98 to 1.5, 1.12 on average from five iterations on (with four, the one pass in between
// gains nothing: 0.97 to 1.03).  In parts, rows are read again for each, which more passes make up for: up to three parts 1.15 on average from
// eight iterations on, the least 0.96 of 139 (us: 1092872 x 212 bf16, K = 44, 13 iterations 1781 / 1861); more parts 1.13 from twelve on, 69 of
// 76 no slower, skewed clusters down to 0.90 (312223 x 220 bf16, K = 57, 22: 1743 / 1927; 88281 x 221, K = 61, 27, even ones 960 / 633); with
// fewer iterations 649628 x 128 bf16, K = 117, 7: 1335 / 1522; 717591 x 256 bf16, K = 54, 6: 1034 / 1153.  Longer rows: the first passes after the
// full ones list many rows, which k_delta_prep adds faster than the members' atomics, and only a long run of short lists makes up for it: 40000
// x 1000, K = 5, 10 iterations 553 / 670; 117187 x 512, K = 28, 6: 635 / 774; 50000 x 1000, K = 16, 30, skewed clusters 1756 / 1888 (logits 965 /
// 725); 80000 x 1000 bf16, K = 5, 30: 1380 / 1602.  So there fp32, few clusters, 20 iterations: 88 fits of 50 million entries in rows of 300, 600
// and 1000 channels with K = 2, 3, 5, 8 and 20 or 30 iterations, skewed clusters among them: 1.00 to 1.30, the least 83333 x 600, K = 8, 20,
// skewed 1230 / 1235; 123 random ones 0.98 to 1.51.
bool loop_bounds_pays(int64_t N, int64_t D, int32_t K, int32_t iters, cat_dtype dt) {
    if (!loops_on(iters)) return false;
    const LoopCfg c = loop_config(N, D, K, dt, true);
    if (!c.ok || g_loop_members.load() > 0) return c.ok;
    if (D > 256) return dt == CAT_F32 && (int64_t)K * D <= 5120 && iters >= 20;
    const int64_t parts = (D + c.W - 1) / c.W;
    return iters >= (parts == 1 ? 5 : parts <= 3 ? 8 : 12);
}

cat_status loop_lloyd_bounds(const void* lq, cat_dtype dt, int64_t N, int64_t D, int32_t K, int32_t iters, float* cent_io, double* sums,
                             int32_t* assign, int32_t* counts, double* inertia, unsigned long long* rep, const LloydWs& lw,
                             const LoopBounds& lb, hipStream_t st) {
    return run_loop(lq, dt, N, D, K, iters, cent_io, sums, assign, counts, inertia, rep, nullptr, lw, &lb, st);
}

}  // namespace cat

extern "C" cat_status cat_debug_loop(int members) {
    cat::g_loop_members.store(members < 0 ? -1 : members);
    return CAT_OK;
}
