// The matrix-core builders' kernels and their launch, for one dtype to a source file (factor_bf16.hip, factor_f16.hip,
// factor_f32.hip: together they compile for minutes).
#pragma once

#include "common.h"
#include "factor_batch.h"

namespace kfac {

// (128 and 64 wide: three workgroups of four wavefronts per CU; 256 wide: one of eight)
// PLANES: with builds that are read as planes among the others.  (A kernel of its own for launches without them: with the form in it
// it cost each launch 0.2 to 0.5 us, the first convolution's two factors 94.1 -> 95.2.  Launches of planes only, beside those of the
// others, leave more ends of launches: all factors of ResNet-50 in bf16 at batch 32 1,639 us instead of 1,514.)
template <int TW, int KIND, bool PLANES>
__global__ __launch_bounds__((tile_threads<TW, KIND == 2 ? 4 : 2>())) __attribute__((amdgpu_waves_per_eu(TW == 256 ? 2 : 3, 8)))
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
        shared_tile<TW, KIND>(v, x, plan_shared(v, b.share[m]), shared_ws(v, it.ws), local, turn, smem);
        return;
    }
    const FactorPlan p = plan_tiles(v, b.share[m]);
    const float scale = it.scale == 0.f ? 1.0f / (float)u.R : it.scale;
    factor_tile<TW, KIND, PLANES>(v, x, scale, out_spec(it), partial_of(v, p, it.ws), p.rows_per_split, p.tiles_dim, p.ntiles, p.nsplit,
                                  local, turn, smem);
}

template <int TW, int KIND, bool PLANES>
static int launch_tile_kernel(const FBatch& b, hipStream_t stream) {
    constexpr int LDS = tile_lds_bytes<TW, KIND == 2 ? 4 : 2>();
    // More than 64 KB of LDS have to be asked for, on every device anew: the 256-wide kernels' launches do, each for the device it
    // goes to (nothing to remember between calls; their work is milliseconds).
    if constexpr (LDS > 64 * 1024) {
        if (hipFuncSetAttribute((const void*)factor_tile_kernel<TW, KIND, PLANES>, hipFuncAttributeMaxDynamicSharedMemorySize, LDS) != hipSuccess)
            return KFAC_ERR_HIP;
    }
    void* tok = nullptr;
    static const char* const name = KIND == 2 ? (TW == 64 ? "factor_tile_kernel<64, f32>" : "factor_tile_kernel<128, f32>")
                                  : TW == 64 ? "factor_tile_kernel<64, 16-bit>"
                                  : TW == 128 ? "factor_tile_kernel<128, 16-bit>" : "factor_tile_kernel<256, 16-bit>";
    if (timing_enabled()) timing_begin(name, stream, &tok);
    hipLaunchKernelGGL((factor_tile_kernel<TW, KIND, PLANES>), dim3(b.prefix[b.count]), dim3(tile_threads<TW, KIND == 2 ? 4 : 2>()), LDS, stream, b);
    if (tok) timing_end(stream, tok);
    if (hipGetLastError() != hipSuccess) return KFAC_ERR_HIP;
    return KFAC_OK;
}

// Tiles `tw` wide (64, 128; 16-bit also 256) of the builds of `b`; planes: some are read as planes.
template <int KIND>
int launch_tiles(int tw, bool planes, const FBatch& b, hipStream_t stream) {
#define KFAC_LAUNCH_TILES(TW) (planes ? launch_tile_kernel<TW, KIND, true>(b, stream) : launch_tile_kernel<TW, KIND, false>(b, stream))
    if (tw == 64) return KFAC_LAUNCH_TILES(64);
    if constexpr (KIND != 2) {
        if (tw == 256) return KFAC_LAUNCH_TILES(256);
    }
    return KFAC_LAUNCH_TILES(128);
#undef KFAC_LAUNCH_TILES
}

}  // namespace kfac
