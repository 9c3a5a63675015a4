// Wave-tile kernel for the fused-upcast linear layer (rg_wtile.hip): its builds, the rule that chooses
// among them (host code, a function of the shape, the weight type and the alignment alone) and its launch.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rg_kernels.h"

namespace rg {

constexpr int kWtileRows = 64;             // output tile of forced launches (build 0): 64 rows of x by 64 rows of W
constexpr int64_t kWtileMaxK = (1 << 24) - 1;   // byte offsets within a tile (at most 64 rows of 4 K bytes) fit 32 bits
constexpr int kWtileDepth = 2;             // slabs of a wave's LDS ring: one computed, one in flight
constexpr int kWtileLds = 160 * 1024;

// Workgroups of a launch of `tiles` tiles (the same number on every XCD), and whether one of `waves` waves each stays
// within the 2^32 - 1 threads a launch holds.
inline int64_t wtile_grid(int64_t tiles) { return (tiles + 7) / 8 * 8; }
inline bool wtile_grid_ok(int64_t tiles, int waves) { return wtile_grid(tiles) <= 0xffffffffLL / (64 * waves); }

// LDS bytes of one slab of a wave: x then W, each padded to whole 1 KB DMA instructions.
template <int BM, int BN, int KT, typename WT>
struct WtileSlab {
    static constexpr int PX = KT / 4;                         // 16-byte pieces of an x row
    static constexpr int PW = KT * (int)sizeof(WT) / 16;      // ... of a W row
    static constexpr int XI = (BM * PX + 63) / 64;            // DMA instructions for x
    static constexpr int WI = (BN * PW + 63) / 64;            // ... for W
    static constexpr int WOFF = XI * 1024;
    static constexpr int BYTES = (XI + WI) * 1024;
};

// The builds: tile shape (LM, TM, TN, KT, NWMAX, WPE, KB) and `rate`, the multiply-adds per ns one CU
// sustains on it with at least eight waves (measured on an MI355X: the slope between 512 and 1024
// tiles at K = 4096).  Larger tiles run faster per multiply-add; smaller ones fill the CUs of a narrow layer.
#define RG_WTILE_BF16(B)                                                            \
    B(8, 8, 8, 16, 8, 2, 4, 161) /* 64 x 64 */ B(8, 8, 7, 16, 8, 2, 4, 158) /* 64 x 56 */ \
    B(8, 8, 6, 16, 8, 2, 4, 152) /* 64 x 48 */ B(8, 8, 5, 16, 8, 2, 4, 151) /* 64 x 40 */ \
    B(8, 7, 8, 16, 8, 2, 4, 156) /* 56 x 64 */ B(8, 6, 8, 16, 8, 2, 4, 148) /* 48 x 64 */ \
    B(8, 6, 6, 16, 8, 2, 4, 144) /* 48 x 48 */ B(8, 5, 8, 16, 8, 2, 4, 131) /* 40 x 64 */ \
    B(4, 8, 4, 32, 8, 2, 4, 145) /* 32 x 64 */ B(8, 4, 6, 32, 8, 2, 4, 134) /* 32 x 48 */ \
    B(8, 4, 4, 32, 16, 4, 4, 126) /* 32 x 32 */ B(4, 6, 4, 32, 8, 2, 4, 134) /* 24 x 64 */ \
    B(8, 3, 6, 32, 8, 2, 4, 115) /* 24 x 48 */ B(8, 3, 4, 32, 16, 4, 4, 107) /* 24 x 32 */ \
    B(4, 4, 4, 32, 16, 4, 4, 120) /* 16 x 64 */ B(4, 4, 2, 32, 16, 4, 4, 111) /* 16 x 32 */ \
    B(8, 2, 3, 32, 16, 4, 8, 94) /* 16 x 24 */ B(4, 4, 1, 32, 16, 4, 8, 94) /* 16 x 16 */
#define RG_WTILE_F32(B)                                                             \
    B(8, 8, 8, 16, 8, 2, 4, 144) /* 64 x 64 */ B(8, 8, 6, 16, 8, 2, 4, 137) /* 64 x 48 */ \
    B(8, 8, 4, 16, 8, 2, 4, 128) /* 64 x 32 */ B(8, 4, 6, 16, 8, 2, 4, 110) /* 32 x 48 */ \
    B(8, 4, 4, 16, 8, 2, 4, 107) /* 32 x 32 */ B(4, 4, 2, 32, 16, 4, 4, 70) /* 16 x 32 */ \
    B(8, 2, 3, 32, 16, 4, 4, 72) /* 16 x 24 */ \
    B(4, 4, 1, 32, 16, 4, 8, 71) /* 16 x 16 */
#define RG_WTILE_ANY(B)                                                             \
    B(8, 6, 4, 16, 8, 2, 4, 110) /* 48 x 32 */ B(8, 4, 4, 16, 8, 2, 4, 100) /* 32 x 32 */ \
    B(4, 4, 2, 16, 8, 2, 4, 70) /* 16 x 32 */ B(4, 4, 1, 16, 16, 4, 4, 60) /* 16 x 16 */ \
    B(4, 2, 2, 16, 16, 4, 4, 40) /* 8 x 32 */ B(4, 2, 1, 16, 16, 4, 4, 40) /* 8 x 16 */

struct WtileBuild {
    int bm, bn, slab, nwmax, rate;
};

// The builds for a weight type (`f32`: FP32, else BF16) and alignment (`aligned`: x and w 16-byte aligned and
// K % 8 == 0, FP32 K % 4 == 0), in the order of the lists above.
inline const WtileBuild* wtile_builds(bool f32, bool aligned, int* count) {
#define RG_B(WT, LM, TM, TN, KT, NWMAX, RATE) \
    {(LM) * (TM), 64 / (LM) * (TN), WtileSlab<(LM) * (TM), 64 / (LM) * (TN), KT, WT>::BYTES, NWMAX, RATE},
#define RG_B2(LM, TM, TN, KT, NWMAX, WPE, KB, RATE) RG_B(uint16_t, LM, TM, TN, KT, NWMAX, RATE)
#define RG_B4(LM, TM, TN, KT, NWMAX, WPE, KB, RATE) RG_B(float, LM, TM, TN, KT, NWMAX, RATE)
    static const WtileBuild bf16[] = {RG_WTILE_BF16(RG_B2)}, fp32[] = {RG_WTILE_F32(RG_B4)};
    static const WtileBuild any_bf16[] = {RG_WTILE_ANY(RG_B2)}, any_fp32[] = {RG_WTILE_ANY(RG_B4)};
#undef RG_B4
#undef RG_B2
#undef RG_B
    constexpr int kAny = (int)(sizeof any_bf16 / sizeof any_bf16[0]);
    *count = !aligned ? kAny : f32 ? (int)(sizeof fp32 / sizeof fp32[0]) : (int)(sizeof bf16 / sizeof bf16[0]);
    return !aligned ? (f32 ? any_fp32 : any_bf16) : f32 ? fp32 : bf16;
}

inline int64_t wtile_lds(const WtileBuild& b, int64_t J, int nw) {
    return (int64_t)nw * kWtileDepth * b.slab + (J > nw ? (int64_t)b.bm * b.bn * 4 : 0);
}

// Tile and waves for a shape: the least estimated time over the builds and a few wave counts each, a
// function of (M, N, K), the weight type and the alignment.  A wave runs at an eighth of the build's
// rate; a workgroup of nw waves takes as long as the wave with the most k (`path`: whole rounds of
// segments, a short last segment alone in its round counted as short), plus 1 us for its first slabs and
// per round 0.3 us and the fold, which its threads share; a CU works off ceil(tiles / 256) tiles, as many
// at a time as its eight wave slots and LDS hold (builds of sixteen waves share the slots), and never
// faster than W streams (6.2 GB per ms: a constant of this model; the fastest reads measured reach 6.8).  So 1536 = 6 segments run on 2 waves, four workgroups per
// CU, not on 6 waves with two slots empty (2048 x 16384 x 1536 1472 -> 1116 us).
//
// Not ok where no build's tiles fit a launch, and where the 128 x 128 register tiles are the better ones: at
// least 512 of them, and their own time (rounds of 512, 175 multiply-adds per ns and CU) under 0.9 of the estimate
// here, which is pessimistic by that much where tiles are many (2048 x 16384: K = 1024 767 against 785 us, K = 2048 1481
// against 1532; from K = 8192 on the wave tiles lead: 2048 x 57344 x 8192 20.8 against 21.8 ms).
struct WtileChoice {
    bool ok = false;
    int build = 0, waves = 0;      // index into wtile_builds, waves per workgroup
    double us = 0.0;               // estimated time
};

inline WtileChoice wtile_choose(int64_t M, int64_t N, int64_t K, bool f32, bool aligned) {
    WtileChoice c;
    int nb = 0;
    const WtileBuild* bs = wtile_builds(f32, aligned, &nb);
    const int64_t J = (K + kChunk - 1) / kChunk;
    const double last_len = (double)(K - (J - 1) * kChunk);
    const double hbm = (double)N * (double)K * (f32 ? 4 : 2) / 6.2e6;
    for (int i = 0; i < nb; ++i) {
        const WtileBuild& b = bs[i];
        const double tiles = (double)((M + b.bm - 1) / b.bm) * (double)((N + b.bn - 1) / b.bn);
        if (tiles > 2.0e9) continue;
        const int percu = (int)(((int64_t)tiles + 255) / 256);
        // wave counts: the fewest for each of the four smallest numbers of rounds; with one tile per CU a
        // workgroup may bring sixteen waves, with more eight (and four where many tiles have 16 rows: one's
        // folds hide behind the others, the 128256 x 4096 head at M = 16 305 -> 286 us)
        const int most = percu > 2 && b.bm <= 16 ? 4 : percu > 1 && b.nwmax > 8 ? 8 : b.nwmax;
        int64_t rounds = (J + most - 1) / most;
        for (int tries = 0; tries < 4; ++tries, ++rounds) {
            const int nw = (int)((J + rounds - 1) / rounds);
            const int64_t lds = wtile_lds(b, J, nw);
            if (lds > kWtileLds || !wtile_grid_ok((int64_t)tiles, nw)) continue;
            int resident = (int)(kWtileLds / lds);
            if (resident * nw > b.nwmax) resident = b.nwmax / nw > 0 ? b.nwmax / nw : 1;
            if (resident > percu) resident = percu;
            const double share = resident * nw > 8 ? resident * nw / 8.0 : 1.0;
            const double path = (double)(rounds - 1) * kChunk + (J - (rounds - 1) * nw == 1 ? last_len : kChunk);
            const double batches = (double)((percu + resident - 1) / resident);
            const double tile = (double)(b.bm * b.bn);
            double us = batches * (1.0 + (double)rounds * (0.3 + 1.7 / nw * (tile / 4096.0)) +
                                   path * share * tile / (b.rate * 125.0));
            if (us < hbm) us = hbm + 0.05 * us;
            if (!c.ok || us < c.us) {
                c.us = us;
                c.ok = true;
                c.build = i;
                c.waves = nw;
            }
            if (nw == 1) break;
        }
    }
    if (c.ok && aligned && M > 64) {
        const double t128 = (double)((M + 127) / 128) * (double)((N + 127) / 128);
        if (t128 >= 512.0) {
            const double rounds = (double)(((int64_t)t128 + 511) / 512);
            if (rounds * 2.0 * 128.0 * 128.0 * (double)K / 175000.0 < 0.9 * c.us) c.ok = false;
        }
    }
    return c;
}

// x [M][K] FP32, w [N][K] BF16 bits or FP32, y [M][N].  `build`, `aligned`: as wtile_builds; `aligned` false
// takes any K and alignment, true only what it says; waves per workgroup at most the build's; K <= kWtileMaxK.
// hipErrorInvalidValue for arguments that do not fit (nothing is enqueued).
hipError_t launch_wtile(const float* x, const uint16_t* w, const float* bias, float* y, int64_t M, int64_t N,
                        int64_t K, int build, int waves, bool aligned, int reverse, hipStream_t stream);
hipError_t launch_wtile(const float* x, const float* w, const float* bias, float* y, int64_t M, int64_t N,
                        int64_t K, int build, int waves, bool aligned, int reverse, hipStream_t stream);

}  // namespace rg
