// Fused inference with the centroid operand streamed from L2 (cat_wide_kernel.h): variant selection on the host, launch.
#include "cat_wide_kernel.h"

#include "cat_infer.h"

namespace cat {

// centroid preparation shared with the tile kernels (cat_tile.hip)
cat_status launch_tile_prep_plain(cat_dtype dt, const float* cent, int64_t D, int32_t K, int32_t KT, int32_t P,
                                  int32_t nchunks, int rows_layout, uint16_t* packA, float* cnorm, hipStream_t st,
                                  const FoldAlpha* fold);

namespace {

struct WideInst {
    bool bf16;
    int KT, RG, VPR;  // cluster tiles; 16-row groups per tile; KB per row
    const void* fn;
    const void* fn_ua;
};
#define CAT_WIDE(BF, KT, RG, VPR) \
    {BF, KT, RG, VPR, (const void*)k_wide<BF, KT, RG, VPR, false>, (const void*)k_wide<BF, KT, RG, VPR, true>}
// K <= 16 KT, rows of at most VPR KB; the first in the list that holds a shape is taken.  Tiles of 64, 48
// and 32 rows: 100 .. 150 KB of LDS with the partial products.  The shapes of fewer clusters or shorter rows belong to the
// row-tile kernel (wide_instance).
const WideInst kWideInst[] = {
    CAT_WIDE(false, 4, 2, 3), CAT_WIDE(false, 4, 2, 4),
    CAT_WIDE(false, 8, 2, 3), CAT_WIDE(false, 8, 2, 4),
    CAT_WIDE(false, 16, 2, 2), CAT_WIDE(false, 16, 2, 3),
    CAT_WIDE(true, 2, 2, 3), CAT_WIDE(true, 2, 2, 4),
    CAT_WIDE(true, 4, 3, 2), CAT_WIDE(true, 4, 2, 3), CAT_WIDE(true, 4, 2, 4),
    CAT_WIDE(true, 8, 4, 1), CAT_WIDE(true, 8, 3, 2), CAT_WIDE(true, 8, 2, 3), CAT_WIDE(true, 8, 2, 4),
    CAT_WIDE(true, 16, 2, 2), CAT_WIDE(true, 16, 2, 3),
};
constexpr int kNWide = sizeof(kWideInst) / sizeof(kWideInst[0]);

// -1: none, also where the row-tile kernel has an instance that cat_apply always prefers (two-part ranking, or rows of up to
// 512 channels).
int wide_instance(int64_t D, int32_t K, cat_dtype dt) {
    const bool bf = dt == CAT_BF16;
    if (bf && D % 2) return -1;
    if (infer_supported(1, D, K, dt) && (infer_two_parts(D, K, dt) || D <= 512)) return -1;
    const int64_t row = D * (bf ? 2 : 4);
    for (int i = 0; i < kNWide; i++)
        if (kWideInst[i].bf16 == bf && K <= 16 * kWideInst[i].KT && row <= 1024 * kWideInst[i].VPR) return i;
    return -1;
}

}  // namespace

bool wide_supported(int64_t N, int64_t D, int32_t K, cat_dtype dt) {
    return N < ((int64_t)1 << 40) && wide_instance(D, K, dt) >= 0;
}

int wide_cluster_tiles(int64_t D, int32_t K, cat_dtype dt) {
    const int i = wide_instance(D, K, dt);
    return i >= 0 ? kWideInst[i].KT : 0;
}

cat_status wide_apply(const void* lq, cat_dtype dt, int64_t N, int64_t D, int32_t K, const float* cent, const float* gamma,
                      const float* beta, void* corrected, int32_t* assign, const TileWs& ws, hipStream_t st,
                      const FoldAlpha* fold) {
    const int inst = wide_instance(D, K, dt);
    if (inst < 0 || !corrected)
        return set_error(CAT_ERR_UNSUPPORTED, "streamed-operand inference does not fit D=%lld K=%d", (long long)D, (int)K);
    const WideInst& in = kWideInst[inst];
    const bool bf = dt == CAT_BF16;
    const bool ua = D % (bf ? 8 : 4) != 0;
    const float* cw = cent;
    if (((uintptr_t)cent & 15u) != 0) {
        cat_status s = launch_copy_words(cent, ws.cent, (int64_t)K * D, st);
        if (s != CAT_OK) return s;
        cw = ws.cent;
    }
    const int nchunks = (int)((D + 127) / 128);
    cat_status s = launch_tile_prep_plain(dt, cw, D, K, in.KT, 2, nchunks, 0, ws.packA, ws.cnorm, st, fold);
    if (s != CAT_OK) return s;
    WideParams p = {};
    p.lq = lq;
    p.out = corrected;
    p.assign = assign;
    p.N = N;
    p.D = D;
    p.ntiles = (N + 16 * in.RG - 1) / (16 * in.RG);
    p.K = K;
    p.psteps = 4 * nchunks;
    p.packA = ws.packA;
    p.cnorm = ws.cnorm;
    p.cent = cw;
    p.gamma = gamma;
    p.beta = beta;
    // error bound of the split arithmetic (see the tile kernel): two parts per operand, n_acc fp32 accumulations of partial
    // sums: the products of all steps, the two accumulators and the channel shares
    const float n_acc = (float)((bf ? 2 : 3) * ((int)((D + 31) / 32) + 1) + 8 + 8);
    p.tau = (bf ? 3.1e-5f : 9.4e-5f) + 4.f * n_acc * 5.96e-8f;
    p.tau2 = 4.0e-7f;

    const int SC = in.KT > 8 ? 1 : kInferWaves / in.KT;
    const size_t lds = wide_lds_bytes(in.KT, SC, in.RG, in.VPR);
    if (lds > 160 * 1024) return set_error(CAT_ERR_UNSUPPORTED, "streamed-operand inference: %zu bytes of LDS", lds);
    const void* fn = ua ? in.fn_ua : in.fn;
    static thread_local int cached_key = -1, cached_dev = -1, per_cu = 1, ncu = 256;
    const int key = 2 * inst + (ua ? 1 : 0);
    int dev = 0;
    CAT_HIP_TRY(hipGetDevice(&dev));
    if (cached_key != key || cached_dev != dev) {
        int nb = 0, v = 0;
        CAT_HIP_TRY(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        CAT_HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fn, kInferWaves * kWave, lds));
        CAT_HIP_TRY(hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev));
        per_cu = nb < 1 ? 1 : nb;
        ncu = v > 0 ? v : 256;
        cached_key = key;
        cached_dev = dev;
    }
    const int64_t cap = (int64_t)ncu * per_cu;
    const unsigned blocks = (unsigned)(p.ntiles < cap ? p.ntiles : cap);
    const bool prof = profile_on();
    if (prof) {
        s = profile_mark(true, st);
        if (s != CAT_OK) return s;
    }
    void* args[] = {(void*)&p};
    CAT_HIP_TRY(hipLaunchKernel(fn, dim3(blocks), dim3(kInferWaves * kWave), args, lds, st));
    CAT_LAUNCH_CHECK("k_wide");
    if (prof) return profile_mark(false, st);
    return CAT_OK;
}

}  // namespace cat
