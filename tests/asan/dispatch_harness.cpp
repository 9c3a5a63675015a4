// What rg_linear, rg_linear_bias and rg_linear_f32w launch, against what rg_plan and rg_plan_f32w report: the
// library's own rg_api.cpp with stubs in place of the kernel launchers (each notes what it was asked for) and of the
// three HIP queries on the way to a launch, so that every call reaches its launcher without a device.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include "../../include/rg.h"
#include "../../include/rg_attn.h"
#include "../../paper_2609_25624_amd/csrc/rg_attn_rule.h"
#include "../../paper_2609_25624_amd/csrc/rg_kernels.h"
#include "../../paper_2609_25624_amd/csrc/rg_wtile.h"

extern "C" {
hipError_t hipGetDevice(int* d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) {
    memset(p, 0, sizeof *p);
    strcpy(p->gcnArchName, "gfx950");
    p->multiProcessorCount = 256;
    return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
}

static struct Seen {
    int calls, kernel, tm, tn, waves, reverse;
    int64_t grid;             // 0: not compared
    hipError_t answer;        // what the launcher returns
} seen;

static hipError_t saw(int kernel, int tm, int tn, int waves, int64_t grid) {
    ++seen.calls;
    seen.kernel = kernel;
    seen.tm = tm;
    seen.tn = tn;
    seen.waves = waves;
    seen.grid = grid;
    return seen.answer;
}

namespace rg {
template <bool F32>
static hipError_t saw_wtile(int64_t M, int64_t N, int build, int waves, bool aligned, int reverse) {
    seen.reverse = reverse;
    int nb = 0;
    const WtileBuild* bs = wtile_builds(F32, aligned, &nb);
    if (build < 0 || build >= nb) return saw(-1, 0, 0, 0, 0);
    const int64_t tiles = (M + bs[build].bm - 1) / bs[build].bm * ((N + bs[build].bn - 1) / bs[build].bn);
    if ((tiles + 7) / 8 * 8 * 64 * waves > 0xffffffffLL) return saw(-2, 0, 0, 0, 0);   // more threads than a launch holds
    return saw(RG_KERNEL_WTILE, bs[build].bm, bs[build].bn, waves, tiles);
}
hipError_t launch_attn(const AttnArgs&, int, hipStream_t) { return saw(-1, 0, 0, 0, 0); }
hipError_t launch_cast(const uint16_t*, float*, int64_t, hipStream_t) { return saw(-1, 0, 0, 0, 0); }
hipError_t launch_argmax(const float*, int64_t*, int64_t, int64_t, hipStream_t) { return saw(-1, 0, 0, 0, 0); }
hipError_t launch_gemv(const GemvArgs&, int grid, int nw, hipStream_t) { return saw(RG_KERNEL_GEMV, 0, 0, nw, grid); }
hipError_t launch_decode(const DecodeArgs& a, int, int, int nw, int, hipStream_t) {
    return saw(RG_KERNEL_DECODE, 0, 0, nw, a.groups);
}
hipError_t launch_decode1(const DecodeArgs&, int grid, int nw, int, hipStream_t) {
    return saw(RG_KERNEL_DECODE_XS, 0, 0, nw, grid);
}
hipError_t launch_skinny(const SkinnyArgs& a, int mt, int, int nw, int, hipStream_t) {
    return saw(RG_KERNEL_SKINNY, mt, 16, nw, a.groups * a.mslices);
}
hipError_t launch_stream(const StreamArgs&, bool, int, int grid, hipStream_t) {
    return saw(RG_KERNEL_STREAM, 0, 0, 4, grid);
}
hipError_t launch_ktile(const float*, const uint16_t*, const float*, float*, int64_t, int64_t, int64_t, int bm, int bn,
                        int nt, int, int, hipStream_t) { return saw(RG_KERNEL_KTILE, bm, bn, nt / 64, 0); }
hipError_t launch_ktile(const float*, const float*, const float*, float*, int64_t, int64_t, int64_t, int bm, int bn,
                        int nt, int, int, hipStream_t) { return saw(RG_KERNEL_KTILE, bm, bn, nt / 64, 0); }
hipError_t launch_tiled(const float*, const uint16_t*, const float*, float*, int64_t, int64_t, int64_t, int bm, int bn,
                        int, int, hipStream_t) { return saw(RG_KERNEL_TILED, bm, bn, 4, 0); }
hipError_t launch_tiled(const float*, const float*, const float*, float*, int64_t, int64_t, int64_t, int bm, int bn,
                        int, int, hipStream_t) { return saw(RG_KERNEL_TILED, bm, bn, 4, 0); }
hipError_t launch_wtile(const float*, const uint16_t*, const float*, float*, int64_t M, int64_t N, int64_t, int build,
                        int waves, bool aligned, int reverse, hipStream_t) {
    return saw_wtile<false>(M, N, build, waves, aligned, reverse);
}
hipError_t launch_wtile(const float*, const float*, const float*, float*, int64_t M, int64_t N, int64_t, int build,
                        int waves, bool aligned, int reverse, hipStream_t) {
    return saw_wtile<true>(M, N, build, waves, aligned, reverse);
}
hipError_t launch_generic(const float*, const uint16_t*, const float*, float*, int64_t, int64_t, int64_t, int grid, int,
                          hipStream_t) { return saw(RG_KERNEL_GENERIC, 0, 0, 4, grid); }
hipError_t launch_generic(const float*, const float*, const float*, float*, int64_t, int64_t, int64_t, int grid, int,
                          hipStream_t) { return saw(RG_KERNEL_GENERIC, 0, 0, 4, grid); }
}  // namespace rg

// pointers far enough apart for every size below, never read
static float* const X = reinterpret_cast<float*>((uintptr_t)1 << 58);
static uint16_t* const W = reinterpret_cast<uint16_t*>((uintptr_t)2 << 58);
static float* const Y = reinterpret_cast<float*>((uintptr_t)3 << 58);
static float* const BIAS = reinterpret_cast<float*>((uintptr_t)4 << 58);

static int call(int entry, int64_t M, int64_t N, int64_t K) {
    if (entry == 0) return rg_linear(X, W, Y, M, N, K, nullptr);
    if (entry == 1) return rg_linear_bias(X, W, BIAS, Y, M, N, K, nullptr);
    return rg_linear_f32w(X, reinterpret_cast<float*>(W), Y, M, N, K, nullptr);
}

int main() {
    const int64_t Ms[] = {1, 2, 4, 5, 8, 9, 16, 17, 33, 48, 64, 65, 100, 333, 2048, 65536, 1 << 20};
    const int64_t Ns[] = {1, 16, 300, 1030, 4096, 6144, 28672, 128256, 1048579, 1 << 28};
    const int64_t Ks[] = {1, 7, 8, 255, 264, 1000, 1001, 4096, 14336, 28672, 32776, 1 << 20, (1 << 24) - 8, 1 << 24,
                          (1 << 26) + 8};
    rg_launch_t cfgs[24] = {};
    int nc = 1;                                                   // cfgs[0]: the defaults
    for (int k = 1; k <= 9; ++k) cfgs[nc++].kernel = k;           // every kernel forced
    cfgs[nc++].grid_order = 1;
    cfgs[nc++].waves_per_wg = 4;
    cfgs[nc++].waves_per_wg = 8;
    cfgs[nc++].tile_n = 32;
    cfgs[nc++].slice_m = 2;
    cfgs[nc++].depth = 3;
    long compared = 0;
    for (int c = 0; c < nc; ++c) {
        if (rg_linear_set_launch(&cfgs[c]) != RG_OK) return 2;
        for (int64_t M : Ms)
            for (int64_t N : Ns)
                for (int64_t K : Ks)
                    for (int entry = 0; entry < 3; ++entry) {
                        rg_plan_t p;
                        const int ps = entry == 2 ? rg_plan_f32w(M, N, K, &p) : rg_plan(M, N, K, &p);
                        seen = Seen{};
                        const int st = call(entry, M, N, K);
                        if (ps != RG_OK) {
                            if (st == ps && seen.calls == 0) continue;
                            printf("refused by the plan only: entry %d (%ld,%ld,%ld)\n", entry, (long)M, (long)N, (long)K);
                            return 3;
                        }
                        if (st == RG_ERR_RANGE && seen.calls == 0 && p.kernel == RG_KERNEL_DECODE) continue;   // its grid
                        const bool tiles = p.kernel == RG_KERNEL_WTILE || p.kernel == RG_KERNEL_KTILE ||
                                           p.kernel == RG_KERNEL_TILED || p.kernel == RG_KERNEL_SKINNY;
                        if (st != RG_OK || seen.calls != 1 || seen.kernel != p.kernel || seen.waves != p.waves_per_wg ||
                            (tiles && (seen.tm != p.tile_m || seen.tn != p.tile_n)) ||
                            (seen.grid != 0 && seen.grid != p.grid_wgs)) {
                            printf("config %d entry %d (%ld,%ld,%ld): plan kernel %d %d x %d waves %d grid %d, launched "
                                   "%d %d x %d waves %d grid %ld (%d calls, status %d)\n",
                                   c, entry, (long)M, (long)N, (long)K, p.kernel, p.tile_m, p.tile_n, p.waves_per_wg,
                                   p.grid_wgs, seen.kernel, seen.tm, seen.tn, seen.waves, (long)seen.grid, seen.calls, st);
                            return 4;
                        }
                        ++compared;
                    }
    }
    // the grid order alone reverses the default's own kernel, tile and waves
    for (int64_t M : Ms)
        for (int64_t N : Ns)
            for (int64_t K : Ks)
                for (int entry = 0; entry < 3; ++entry) {
                    rg_plan_t a, b;
                    rg_launch_t rev = {};
                    rev.grid_order = 1;
                    rg_linear_set_launch(nullptr);
                    const int sa = entry == 2 ? rg_plan_f32w(M, N, K, &a) : rg_plan(M, N, K, &a);
                    rg_linear_set_launch(&rev);
                    const int sb = entry == 2 ? rg_plan_f32w(M, N, K, &b) : rg_plan(M, N, K, &b);
                    if (sa != RG_OK || a.kernel != RG_KERNEL_WTILE) continue;
                    seen = Seen{};
                    const int st = call(entry, M, N, K);
                    if (sb != RG_OK || memcmp(&a, &b, sizeof a) != 0 || st != RG_OK || seen.reverse != 1) {
                        printf("reversed: entry %d (%ld,%ld,%ld) kernel %d %d x %d, forward %d x %d\n", entry, (long)M,
                               (long)N, (long)K, b.kernel, b.tile_m, b.tile_n, a.tile_m, a.tile_n);
                        return 7;
                    }
                }
    // outputs in numbers whose tiles come near a launch's 2^32 threads: a kernel that can be launched is chosen
    rg_linear_set_launch(nullptr);
    for (int64_t MN : {(int64_t)1 << 30, (int64_t)1 << 31, ((int64_t)1 << 31) + 12345, (int64_t)1 << 33, (int64_t)1 << 35,
                       (int64_t)1 << 38})
        for (int64_t M : {1, 3, 17, 333, 1 << 17, 1 << 19})
            for (int64_t K : {1, 8, 255, 256, 1001, 2048, 4096})
                for (int entry = 0; entry < 3; ++entry) {
                    if (K % 8 == 0 && MN > ((int64_t)1 << 37)) continue;      // (the register tiles' own limit)
                    if (K % 8 == 0 && M <= 8) continue;                       // (not the wave tiles' shapes)
                    seen = Seen{};
                    const int st = call(entry, M, MN / M, K);
                    if (st != RG_OK || seen.calls != 1 || seen.kernel < 0) {
                        printf("entry %d (%ld,%ld,%ld): status %d, launched %d\n", entry, (long)M, (long)(MN / M), (long)K,
                               st, seen.kernel);
                        return 6;
                    }
                }
    // attention: the one-launch kernel only where its threads fit a launch
    for (int64_t pairs : {(int64_t)1, (int64_t)1 << 22, ((int64_t)1 << 23) - 1, (int64_t)1 << 23, (int64_t)1 << 24, (int64_t)1 << 28})
        for (int D : {64, 128, 256})
            for (int G = 1; G <= 8; ++G)
                for (int64_t L : {1, 256, 512, 2048}) {
                    if (pairs * ((L + 255) / 256) > 0x3fffffff) continue;
                    const rg::AttnRoute r = rg::attn_route(pairs, 1, L, D, G, 256);
                    if (r.fused && pairs * rg::kAttnFusedThreads > 0xffffffffLL) {
                        printf("fused: %ld pairs D %d G %d L %ld\n", (long)pairs, D, G, (long)L);
                        return 8;
                    }
                }
    // and only where it was measured ahead of one launch per pass: a round of the CUs, short caches of heavy groups
    const struct { int64_t pairs, L; int D, G; bool fused; } short_caches[] = {
        {8, 512, 64, 1, true}, {256, 512, 64, 1, true}, {512, 512, 64, 1, false}, {2048, 64, 64, 1, false},
        {8192, 256, 64, 1, false}, {300, 200, 64, 1, true}, {400, 200, 64, 1, false}, {256, 2048, 64, 1, true}, {2048, 1024, 64, 1, false}, {2048, 2048, 64, 1, true},
        {512, 1100, 64, 1, true}, {256, 512, 128, 2, true}, {512, 128, 128, 2, false}, {512, 128, 128, 1, true},
        {512, 128, 256, 1, false}, {64, 200, 256, 2, true}, {64, 400, 256, 2, false}, {8, 256, 64, 4, true},
        {8, 300, 64, 4, false}, {200, 300, 64, 4, true}, {257, 64, 128, 4, false}, {64, 128, 64, 8, true}, {64, 150, 64, 8, true}, {64, 200, 64, 8, false},
        {64, 129, 64, 5, false}, {4, 100, 128, 8, false}};
    for (const auto& c : short_caches)
        if (rg::attn_route(c.pairs, 1, c.L, c.D, c.G, 256).fused != c.fused) {
            printf("fused %d: %ld pairs x %ld, D %d, G %d\n", !c.fused, (long)c.pairs, (long)c.L, c.D, c.G);
            return 9;
        }
    // workgroup partials: D = 64, three and more heads, at most three segments per CU
    const struct { int64_t pairs, L; int G; bool group; } groups[] = {
        {8, 1024, 8, true}, {192, 1024, 8, true}, {256, 1024, 8, false}, {64, 1024, 5, true}, {8, 1024, 3, true},
        {64, 2048, 4, true}, {128, 1024, 4, true}, {129, 1024, 4, false}, {512, 64, 8, false}, {8, 1024, 2, false}, {257, 300, 6, true}};
    for (const auto& c : groups)
        if (rg::attn_route(c.pairs, 1, c.L, 64, c.G, 256).group != c.group) {
            printf("group %d: %ld pairs x %ld, G %d\n", !c.group, (long)c.pairs, (long)c.L, c.G);
            return 10;
        }
    // value waves: split, whole or light
    const struct { int64_t pairs, L; int D, G, split, light; } waves[] = {
        {16, 1024, 128, 4, 1, 0}, {256, 1024, 128, 4, 1, 0}, {257, 1024, 128, 4, 0, 0}, {256, 1024, 128, 1, 1, 0},
        {257, 1024, 128, 1, 0, 0}, {256, 1024, 128, 8, 0, 0}, {512, 1024, 128, 8, 0, 0}, {513, 1024, 128, 5, 0, 1},
        {2048, 1024, 128, 4, 0, 0}, {320, 1024, 256, 5, 1, 0}, {321, 1024, 256, 5, 0, 1}, {384, 1024, 256, 8, 1, 0}, {385, 1024, 256, 8, 0, 1},
        {224, 1024, 128, 8, 1, 0}, {225, 1024, 128, 8, 0, 0}, {257, 1024, 256, 4, 0, 0},
        {256, 1024, 256, 1, 1, 0}, {16, 1024, 64, 8, 0, 0}, {2048, 1024, 64, 8, 0, 0}};
    for (const auto& c : waves) {
        const rg::AttnRoute r = rg::attn_route(c.pairs, 1, c.L, c.D, c.G, 256);
        if (r.fused || r.split != (c.split != 0) || r.light != (c.light != 0)) {
            printf("split %d light %d: %ld pairs x %ld, D %d, G %d\n", r.split, r.light, (long)c.pairs, (long)c.L, c.D, c.G);
            return 11;
        }
    }
    // row maxima by a launch of their own: long caches
    const struct { int64_t pairs, L; int D, G; bool maxima; } rows[] = {
        {1, 32768, 128, 4, false}, {8, 65536, 128, 8, false}, {8, 131072, 128, 8, true}, {8, 1 << 20, 128, 8, true},
        {8, 262144, 128, 4, false}, {8, 524288, 64, 1, true}, {1, 1 << 20, 64, 4, false}, {1, 262144, 256, 8, false}, {1, 524288, 256, 8, true},
        {16, 4096, 128, 4, false}, {2048, 1024, 64, 8, false}};
    for (const auto& c : rows)
        if (rg::attn_route(c.pairs, 1, c.L, c.D, c.G, 256).maxima != c.maxima) {
            printf("maxima %d: %ld pairs x %ld, D %d, G %d\n", !c.maxima, (long)c.pairs, (long)c.L, c.D, c.G);
            return 12;
        }
    // a launch that the runtime refuses, with whatever code, is reported and not tried on another kernel
    rg_linear_set_launch(nullptr);
    for (hipError_t err : {hipErrorInvalidValue, hipErrorInvalidConfiguration, hipErrorOutOfMemory})
        for (int64_t M : {1, 4, 16, 333, 2048})
            for (int entry = 0; entry < 3; ++entry)
                for (int64_t K : {1001, 4096}) {
                    seen = Seen{};
                    seen.answer = err;
                    const int st = call(entry, M, 4096, K);
                    if (st != RG_ERR_HIP || seen.calls != 1 || rg_last_hip_error() != (int)err) {
                        printf("launch error %d at entry %d (%ld,4096,%ld): status %d after %d launches\n", (int)err, entry,
                               (long)M, (long)K, st, seen.calls);
                        return 5;
                    }
                }
    printf("ok: %ld launches as planned\n", compared);
    return 0;
}
