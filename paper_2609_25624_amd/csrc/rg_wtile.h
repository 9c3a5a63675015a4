// Internal interface of the wave-tile kernel (rg_wtile.hip) for the C-ABI (rg_api.cpp).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rg {

constexpr int kWtileRows = 64;             // output tile of forced launches: 64 rows of x by 64 rows of W
constexpr int64_t kWtileMaxK = (1 << 24) - 1;   // byte offsets within a tile (at most 64 rows of 4 K bytes) fit 32 bits

// waves: 4 or 8 (64 x 64 tiles, forced launches) or 0: tile and waves by the rule in
// rg_wtile.hip, a function of (M, N, K) and the weight type alone.  x [M][K] FP32, w [N][K]
// BF16 bits or FP32, y [M][N]; `aligned`: x and w 16-byte aligned and K % 8 == 0 (BF16) or
// K % 4 == 0 (FP32).  waves = 0 takes any K and alignment, waves = 4 or 8 aligned calls only;
// K <= kWtileMaxK.  hipErrorInvalidValue for what does not fit (nothing is enqueued).
hipError_t launch_wtile(const float* x, const uint16_t* w, const float* bias, float* y, int64_t M, int64_t N,
                        int64_t K, int waves, int reverse, hipStream_t stream);
hipError_t launch_wtile(const float* x, const float* w, const float* bias, float* y, int64_t M, int64_t N,
                        int64_t K, int waves, int reverse, hipStream_t stream);

}  // namespace rg
