// Which kernels a decode-attention call of head dim 64, 128 or 256 launches (rg_attn.hip): host code, a function of
// the call's sizes and the number of compute units.
#pragma once
#include <stdint.h>

namespace rg {

struct AttnRoute {
    bool fused;    // one launch: a workgroup of eight waves per (sequence, kv head)
    bool group;    // partials by a workgroup per segment (D = 64), after the maximum kernel
    bool split;    // partials by two waves per segment, half the value columns each; one wave otherwise
    bool maxima;   // the whole-row wave partials' row maxima from a launch of their own
    bool light;    // ... by one wave with less LDS (five to eight heads), so that a CU holds sixteen
};

// Lanes (of a position) that a group of G query heads takes: the power of two it fits.
constexpr int attn_lanes(int G) { return G <= 1 ? 1 : G <= 2 ? 2 : G <= 4 ? 4 : 8; }

constexpr int kAttnFusedThreads = 512;

// Fused (one launch) for short caches, where launches and their gaps are most of the time; one launch per pass otherwise.
// A CU holds one of its workgroups (115 to 147 KB of LDS), each as slow as its longest sequence and with half its waves
// idle at two segments, so it leads only while the pairs run in one round of the CUs.  Whole calls, us, fused against one
// launch per pass (ragged batches, pairs of sequence and kv head x longest length; D and query heads per kv head):
//   one or two heads, at most two segments      D = 64, 1: 256 x 512 11.7 / 16.3, 512 x 512 21.0 / 18.6, 2048 x 256 64 / 26;
//                                               D = 128, 2: 256 x 512 18.5 / 23, 512 x 256 28 / 22; D = 256, 1: 256 x 512
//                                               23.3 / 26.9; D = 256, 2, two segments: 64 x 512 29.7 / 26.1 (one only)
//   one head, D = 64, up to eight segments      256 x 2048 20 / 31; above a round of the CUs 512 x 1024 25.8 / 27.0,
//                                               2048 x 1024 99 / 82, 2048 x 2048 145 / 171
//   one head, at most 128 positions             two rounds too: D = 128, 512 x 128 16.0 / 16.4; D = 64, 288 x 164
//                                               12.3 / 13.8, 384 x 256 15.9 / 15.9 (one segment, 1.5 rounds)
//   three or four heads, one segment            D = 64: 64 x 256 17.4 / 17.8 (the group kernel), 128 x 128 12.0 / 15.7;
//   or two on more than half the CUs            D = 128: 64 x 256 21.1 / 21.9, 64 x 512 24.1 / 22.6, 256 x 512 24.7 / 27.1
//   five to eight heads, D = 64                 64 x 128 16.6 / 21.1, 64 x 256 24 / 21; eight 64 x 131 18.5 / 21.6
//                                               (at most 128 positions, eight heads 176)
// Its launch must hold its threads (a launch has at most 2^32 - 1).
//
// Partials: one wave per segment, or two with half its value columns each where there are few segments (64 of D = 64 fill a
// wave as they are): at most four per CU (1024 segments, us, split / whole: D = 128, four heads 1 x 8 pairs of 32768
// positions 38.7 / 40.1 with the cache's rows in the memory-side cache, 40.0 / 39.8 without, 32 x 8 of 1000 38 / 35 and
// 40 / 38; one head 28 / 30; five heads 44.5 / 39.9, eight 55.9 / 54.4, hence 3.5 from five heads on).  With five to
// eight heads many segments want waves more than bytes in flight per wave (8 KB of rows and the e of 64 positions in
// place of 12 KB and 128): from eight segments per CU at D = 128, from five (seven and eight heads six) at D = 256, where
// both halves of a split segment compute all its e.  Whole calls, us, heavy / light: D = 128, eight heads, 256 x 8 pairs of
// 384 positions 138 / 126, 64 x 8 of 2048 155 / 144, of 384 (1024 segments) 55 / 59; D = 256, eight heads (split / light),
// 256 x 8 of 384 250 / 218, 64 x 8 of 1024 150 / 146, of 384 (1024 segments) 80 / 88, 65 x 4 of 1188 (1300 segments)
// 93 / 100; seven heads 28 x 8 of 1156 (1120 segments) 76 / 84.
// Against the persistent wave kernel they replaced, with the maximum kernel where it was launched, us: 64 x 32 heads,
// 2048 positions 51.4 -> 46.3; 32 x 64 heads 72.9 -> 63.7; 16 x 32 heads, 4096 positions 27.2 -> 27.0; 4 x 32 heads,
// 2000 positions 14.0 -> 12.3; D = 64, 60 x 32 heads, 3000 positions 74.3 -> 39.0.
//
// D = 64 with three and more heads: a workgroup per segment while a CU holds them all (three of 40 to 45 KB; with three and
// four heads, whose waves run fewer chains, two per CU) and the segments are more than half full; its four waves share the
// heads that one wave would run alone.  Whole calls, us, group against wave partials (pairs x longest length): eight heads
// 8 x 1024 22.7 / 27.6, 256 x 512 25.8 / 30.7, 192 x 1024 (768 segments) 31.3 / 34.0, 256 x 1024 (1024 segments) 39.9 /
// 37.6; five heads 64 x 1024 20.0 / 25.3; four heads 64 x 2048 22.8 / 23.1, 256 x 512 20.6 / 21.3, 144 x 840 (all full)
// 26.1 / 24.7; three heads 8 x 1024 18.5 / 19.4; eight heads 512 x 64 25.2 / 22.2.
//
// Row maxima of the wave partials: each wave reduces the segment maxima of its whole sequence, work that grows with the
// square of the length; from the line below on (segments x segments / 64; split segments never get there) a launch of
// 2 us takes it over.  Whole calls, us, in the waves / by the launch: eight heads, D = 128, 1 x 8 pairs of 262144 positions
// 332 / 316, of 1048576 1501 / 1216 (1346 with the maximum kernel of one thread per row); D = 64, one head, 1 x 8 of 524288
// 244 / 227, of 262144 114 / 113; D = 128, four heads, 1 x 8 of 524288 456 / 441, of 131072 113 / 116.
inline AttnRoute attn_route(int64_t B, int64_t Hkv, int64_t Lmax, int D, int G, int64_t cus) {
    const int GP = attn_lanes(G);
    const int64_t J = (Lmax + 255) / 256, pairs = B * Hkv, items = pairs * J;
    AttnRoute r = {};
    const bool round = pairs <= cus;
    if (D * GP > 512) r.fused = false;
    else if (GP == 8) r.fused = round && Lmax <= (G == 8 ? 176 : 128);
    else if (GP == 4) r.fused = round && (J == 1 || (J == 2 && 2 * pairs > cus));
    else if (GP == 2) r.fused = round && J <= (D == 256 ? 1 : 2);
    else if (D == 64 && J > 2) r.fused = J <= 8 && (round || J >= 7 || (J >= 4 && pairs <= 2 * cus));
    else r.fused = J <= 2 && (round || (Lmax <= 128 && D < 256 && pairs <= 2 * cus) ||
                              (D == 64 && J == 1 && 2 * pairs <= 3 * cus));
    if (pairs > 0xffffffffLL / kAttnFusedThreads) r.fused = false;
    r.group = !r.fused && D == 64 && G >= 3 && Lmax > 128 && items <= (G <= 4 ? 2 : 3) * cus;
    const int64_t heavy = G >= 7 ? 12 : 10;              // D = 256, five to eight heads: half segments per CU
    r.split = D > 64 && 2 * items <= (GP < 8 ? 8 : D == 256 ? heavy : 7) * cus;
    r.light = D > 64 && GP == 8 && 2 * items > (D == 256 ? heavy : 16) * cus;
    r.maxima = !r.fused && !r.group && !r.split && items * ((J + 63) / 64) >= (GP == 8 ? 32768 : 393216);
    return r;
}

}  // namespace rg
