// Which kernels a decode-attention call of head dim 64, 128 or 256 launches (rg_attn.hip): host code, a function of
// the call's sizes and the number of compute units.
#pragma once
#include <stdint.h>

namespace rg {

struct AttnRoute {
    bool fused;    // one launch: a workgroup of eight waves per (sequence, kv head)
    bool group;    // partials by a workgroup per segment (D = 64), after the maximum kernel
    bool split;    // partials by two waves per segment, half the value columns each; one wave otherwise
};

// Lanes (of a position) that a group of G query heads takes: the power of two it fits.
constexpr int attn_lanes(int G) { return G <= 1 ? 1 : G <= 2 ? 2 : G <= 4 ? 4 : 8; }

constexpr int kAttnFusedThreads = 512;

// Fused (one launch) where the cache holds at most two segments per sequence, so that launches and their gaps are most of
// the time, or eight with the lightest heads; one launch per pass otherwise: a workgroup per (sequence, kv head)
// takes as long as its longest sequence, which the passes spread over the device.  Whole calls, us, fused
// against one launch per pass (4 sequences, 2 kv heads, 400 positions): D = 128, 1 / 2 / 4 heads per kv head 12.6 / 16.9 /
// 22.6 against 16.2 / 20.5 / 24.5 and their two gaps, 8 heads level; D = 256, 1 / 2 / 4 heads 18.0 / 25.0 / 36.7
// against 26 / 27 / 34.7; D = 64, 1 / 2 / 4 / 8 heads 10.7 / 13.8 / 17.7 / 24.4 against 15 / 17 / 19 / 24.
// Its launch must hold its threads (a launch has at most 2^32 - 1).
//
// Partials: one wave per segment, or two with half its value columns each where there are at most four segments per CU
// (64 of D = 64 fill a wave as they are; the heaviest waves, D = 256 with more than four heads, are always split).
// Against the persistent wave kernel they replaced, with the maximum kernel where it was launched, us: 64 x 32 heads,
// 2048 positions 51.4 -> 46.3; 32 x 64 heads 72.9 -> 63.7; 16 x 32 heads, 4096 positions 27.2 -> 27.0; 4 x 32 heads,
// 2000 positions 14.0 -> 12.3; D = 64, 60 x 32 heads, 3000 positions 74.3 -> 39.0 (a workgroup per segment before; that
// kernel stays for four and more heads and at most 1.25 segments per CU: eight heads 11.8 against 15.9, four heads 11.2
// against 12.0).
inline AttnRoute attn_route(int64_t B, int64_t Hkv, int64_t Lmax, int D, int G, int64_t cus) {
    const int GP = attn_lanes(G);
    const int64_t J = (Lmax + 255) / 256, pairs = B * Hkv, items = pairs * J;
    AttnRoute r = {};
    r.fused = D * GP <= 512 && (J <= 2 || (D * GP == 64 && J <= 8)) && pairs <= 0xffffffffLL / kAttnFusedThreads;
    r.group = !r.fused && D == 64 && G >= 4 && 4 * items <= 5 * cus;
    r.split = D > 64 && ((D == 256 && GP == 8) || items <= 4 * cus);
    return r;
}

}  // namespace rg
