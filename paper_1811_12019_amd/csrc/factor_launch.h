// The matrix-core builders' kernels and their launch, for one dtype to a source file (factor_bf16.hip, factor_f16.hip,
// factor_f32.hip: together they compile for minutes).
#pragma once

#include "common.h"
#include "factor_batch.h"

namespace kfac {

// (256 wide: one workgroup of eight wavefronts per CU.  128 wide: three of four, of fp32 tiles, which have twice the accumulators, two; and
// with them the builds of 64-wide tiles, whose workgroups are of the same size: a launch of their own ended as raggedly as it began.  The
// first convolution's two factors 79.6 -> 71 us, all of ResNet-50 at batch 32 from NCHW bf16 1342 -> 1315.)
// PLANES: with builds that are read as planes among the others.  (A kernel of its own for launches without them: with the form in it
// it cost each launch 0.2 to 0.5 us, the first convolution's two factors 94.1 -> 95.2.  Launches of planes only, beside those of the
// others, leave more ends of launches: all factors of ResNet-50 in bf16 at batch 32 1,639 us instead of 1,514.)
template <int TW, int KIND, bool PLANES>
__global__ __launch_bounds__((tile_threads<TW, KIND == 2 ? 4 : 2>())) __attribute__((amdgpu_waves_per_eu(TW == 256 || KIND == 2 ? 2 : 3, 8)))
void factor_tile_kernel(FBatch b) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    int local;
    const int m = fbatch_locate(b, blockIdx.x, local);
    kfac_factor_item it;
    Unfold u;
    View v;
    fbatch_item<PLANES>(b, m, it, u, v);
    const KFAC_AS1 unsigned char* x = (const KFAC_AS1 unsigned char*)(v.repack ? it.ws : it.x);
    const int turn = b.share[m] >> SHARE_TURN_SHIFT;
    if (v.shared) {
        const SharedPlan p = plan_shared(v, b.share[m]);
        if (TW == 128 && p.tw == 64) shared_tile<TW == 128 ? 64 : TW, KIND>(v, x, p, shared_ws(v, it.ws), local, turn, smem);
        else shared_tile<TW, KIND>(v, x, p, shared_ws(v, it.ws), local, turn, smem);
        return;
    }
    const FactorPlan p = plan_tiles(v, b.share[m]);
    const float scale = it.scale == 0.f ? 1.0f / (float)u.R : it.scale;
    if (TW == 128 && p.tw == 64)
        factor_tile<TW == 128 ? 64 : TW, KIND, PLANES>(v, x, scale, out_spec(it), partial_of(v, p, it.ws), p.rows_per_split, p.tiles_dim,
                                                       p.ntiles, p.nsplit, local, turn, smem);
    else
        factor_tile<TW, KIND, PLANES>(v, x, scale, out_spec(it), partial_of(v, p, it.ws), p.rows_per_split, p.tiles_dim, p.ntiles, p.nsplit,
                                      local, turn, smem);
}

template <int TW, int KIND, bool PLANES>
static int launch_tile_kernel(const char* name, const FBatch& b, hipStream_t stream) {
    constexpr int ES = KIND == 2 ? 4 : 2, LDS = tile_lds_bytes<TW, ES>();
    static_assert(TW != 128 || (tile_threads<64, ES>() == tile_threads<128, ES>() && tile_lds_bytes<64, ES>() <= LDS), "one launch for both widths");
    // More than 64 KB of LDS have to be asked for, on every device anew: the 256-wide kernels' launches do, each for the device it
    // goes to (nothing to remember between calls; their work is milliseconds).
    if constexpr (LDS > 64 * 1024) {
        if (hipFuncSetAttribute((const void*)factor_tile_kernel<TW, KIND, PLANES>, hipFuncAttributeMaxDynamicSharedMemorySize, LDS) != hipSuccess)
            return KFAC_ERR_HIP;
    }
    void* tok = nullptr;
    if (timing_enabled()) timing_begin(name, stream, &tok);
    hipLaunchKernelGGL((factor_tile_kernel<TW, KIND, PLANES>), dim3(b.prefix[b.count]), dim3(tile_threads<TW, ES>()), LDS, stream, b);
    if (tok) timing_end(stream, tok);
    if (hipGetLastError() != hipSuccess) return KFAC_ERR_HIP;
    return KFAC_OK;
}

// Tiles up to `tw` wide (128, or 64 if all are; 16-bit also 256, which are launched apart) of the builds of `b`; planes: some are read as
// planes.
template <int KIND>
int launch_tiles(int tw, bool planes, const FBatch& b, hipStream_t stream) {
#define KFAC_LAUNCH_TILES(TW, name) (planes ? launch_tile_kernel<TW, KIND, true>(name, b, stream) : launch_tile_kernel<TW, KIND, false>(name, b, stream))
    if constexpr (KIND != 2) {
        if (tw == 256) return KFAC_LAUNCH_TILES(256, "factor_tile_kernel<256, 16-bit>");
        return KFAC_LAUNCH_TILES(128, tw == 64 ? "factor_tile_kernel<64, 16-bit>" : "factor_tile_kernel<128, 16-bit>");
    }
    return KFAC_LAUNCH_TILES(128, tw == 64 ? "factor_tile_kernel<64, f32>" : "factor_tile_kernel<128, f32>");
#undef KFAC_LAUNCH_TILES
}

}  // namespace kfac
