// Wave-tile kernel for the fused-upcast linear layer (gfx950): the default for M > 8, for FP32
// weights at M > 4 and for every K or alignment the 16-byte kernels do not take, but for the shapes
// where the planner finds another kernel ahead: narrow BF16 layers of up to 64 rows (skinny), register
// tiles of a short K (tiled), a few unaligned k (generic).
//
// Same order as every kernel of the library (include/rg.h, RG-ORDER-1; paper: Design,
// eq. 2 and rules R1-R4): 256-wide K segments, each a chain of fmaf from +0 in ascending
// k, the segment partials folded left to right in ascending segment order.
//
// Work split.  A workgroup owns a BM x BN output tile and all of K.  Each of its NW waves holds
// the whole tile for one segment at a time (wave g runs segments g, g + NW, ...): lane
// (mi, ni) = (lane % LM, lane / LM) runs the TM x TN chains of x rows r LM + mi and W rows
// c (64 / LM) + ni.  A wave stages the KT-wide slabs of its own segment through its own
// double-buffered LDS region, so a segment runs without any barrier.
//
// Data path.  Slabs go from memory to LDS by 16-byte DMA as they are, x rows [row][k] in FP32 and
// W rows [row][k] in their own type: no registers, no transposing stores.  The 16-byte pieces of a row
// are XOR-swizzled (on the global side of the DMA) so that neighbouring rows reach different
// banks.  A lane reads four k of a row at once (16 bytes of x, 8 bytes of BF16 W) and
// widens W in registers.  x or W that are not 16-byte aligned, and K that is not a multiple of the
// vector, go through registers instead (AL = false: loads of any alignment one slab ahead, then
// 16-byte LDS stores); the k past K are staged as x = +0 and w = -0, for which
// fmaf(+0, -0, p) = p for every p.
//
// Fold.  After each round of NW segments the waves put their partials in the LDS slot they have
// just computed from and, after a barrier, every thread adds the round's partials of its
// outputs in ascending segment order to the running total (LDS); the last round stores
// y (+ b).  No atomics, no workspace, no second launch.
//
// What bounds it.  A SIMD issues one FMA per 2 cycles over two waves (one wave: one per 4).  A lane's
// TM x TN chains read 4 / TN + 2 / TM bytes of LDS per FMA (FP32 weights 4 / TN + 4 / TM) and widen TN values of W
// per k, so the fewer chains the slower a multiply-add (the builds' rates in rg_wtile.h).  Counters on 28672 x 4096 give
// about 0.6 of the FMA issue limit to 64 x 56 tiles at M = 64 and 0.35 to 16 x 64 at M = 16, with no bank conflict and
// nearly every wave slot taken at M = 64 (about 7 of 8; 6 at M = 16); what the rest waits for, they do not show.
// W is widened into register pairs such that an FMA's x and W never share a register parity (widen2): these kernels
// run faster so; why is not measured apart.
// 28672 x 4096 at M = 64: 183 us (82 TFLOP/s) against 223 with the transposing wave tile this
// replaced; 4096 x 14336: 109 against 219; 6144 x 4096: 47 against 74.
//
// Arithmetic: only v_fmac_f32 / v_fma_f32 and v_add_f32 (the library is built with
// -ffp-contract=off and packed FP32 disabled), binary32 denormals preserved.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "rg_kernels.h"
#include "rg_wtile.h"

namespace rg {
namespace {

struct WtileArgs {
    const float* x;
    const void* w;        // uint16_t bfloat16 bits or float, [N][K]
    const float* bias;    // b[N] added after the fold, or null
    float* y;
    int64_t M, N, K;
    int J;                // ceil(K / kChunk)
    int tiles_m, tiles_n;
    int reverse;          // 1: reversed workgroup-to-tile mapping
};

constexpr int kGroupM = 8;            // m tiles that share an n tile before the next n tile (large M)

__device__ __forceinline__ uint32_t lds_addr32(const void* p) {
    return (uint32_t)(uintptr_t)((const __attribute__((address_space(3))) void*)p);
}

// One or two 16-byte global -> LDS DMA instructions (lane l writes LDS [base + 16 l, +16), the
// second 1 KB further on).  M0 is saved and restored, and never read in the cycle after a write.
__device__ __forceinline__ void dma_1(const void* sbase, uint32_t v0, uint32_t lds_base) {
    uint32_t saved;
    asm volatile(
        "s_mov_b32 %0, m0\n\t"
        "s_mov_b32 m0, %2\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %1, %3\n\t"
        "s_mov_b32 m0, %0\n\t"
        : "=&s"(saved)
        : "v"(v0), "s"(lds_base), "s"(sbase)
        : "memory");
}
__device__ __forceinline__ void dma_2(const void* sbase, uint32_t v0, uint32_t v1, uint32_t lds_base) {
    uint32_t saved;
    asm volatile(
        "s_mov_b32 %0, m0\n\t"
        "s_mov_b32 m0, %3\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %1, %4\n\t"
        "s_add_u32 m0, m0, 0x400\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %2, %4\n\t"
        "s_mov_b32 m0, %0\n\t"
        : "=&s"(saved)
        : "v"(v0), "v"(v1), "s"(lds_base), "s"(sbase)
        : "memory", "scc");
}
template <int N>
__device__ __forceinline__ void dma_n(const void* sbase, const uint32_t (&v)[N], uint32_t lds_base) {
#pragma unroll
    for (int u = 0; u + 1 < N; u += 2) dma_2(sbase, v[u], v[u + 1], lds_base + 1024u * u);
    if constexpr (N % 2) dma_1(sbase, v[N - 1], lds_base + 1024u * (N - 1));
}

// Every DMA of this wave has landed (the only vector memory operations in flight are its DMA).
__device__ __forceinline__ void dma_wait() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void lds_wait() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
// Barrier that leaves the DMA in flight (a wave's LDS operations are waited for).
__device__ __forceinline__ void wg_barrier() {
    lds_wait();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// The two bfloat16 of a packed dword (even k in the low half), widened exactly.  The odd k's value is
// placed in the even register of a pair and the even k's in the odd one: x arrives by 16-byte LDS reads,
// whose k-th register has the parity of k, so an FMA's x and W never share a register
// parity (64 x 56 tiles 185 -> 180 us at M = 64 on 28672 x 4096, 64 x 64 tiles
// 10.77 -> 10.28 ms on 8192 x 28672 at M = 2048).
__device__ __forceinline__ void widen2(uint32_t d, float& even_k, float& odd_k) {
    uint64_t pair = ((uint64_t)(d << 16) << 32) | (d & 0xffff0000u);
    asm("" : "+v"(pair));
    even_k = __uint_as_float((uint32_t)(pair >> 32));
    odd_k = __uint_as_float((uint32_t)pair);
}

}  // namespace

// LM: lanes along m; TM x TN: chains per lane; KT: k per slab; NWMAX: waves per workgroup at most;
// WPE: waves per SIMD the registers are held to; KB: k per operand read (4 or 8); AL: DMA staging.
template <int LM, int TM, int TN, int KT, int NWMAX, int WPE, int KB, typename WT, bool AL>
__global__ void __launch_bounds__(64 * NWMAX, WPE) wtile_kernel(WtileArgs a) {
    constexpr int LN = 64 / LM, BM = LM * TM, BN = LN * TN;
    using SL = WtileSlab<BM, BN, KT, WT>;
    constexpr int PX = SL::PX, PW = SL::PW, XI = SL::XI, WI = SL::WI;
    constexpr int SLOT = SL::BYTES, RING = kWtileDepth * SLOT;
    constexpr bool BF = sizeof(WT) == 2;
    constexpr int NSL = kChunk / KT;                // slabs per segment
    constexpr int NB = KT / KB;                     // operand reads per slab
    constexpr int NA = TM * TN;                     // chains per lane
    // chains per lane that a fold pass moves through a slot
    constexpr int QC = NA * 256 <= SLOT ? NA
                       : (NA % 2 == 0 && NA / 2 * 256 <= SLOT) ? NA / 2
                       : (NA % 3 == 0 && NA / 3 * 256 <= SLOT) ? NA / 3
                       : (NA % 4 == 0 && NA / 4 * 256 <= SLOT) ? NA / 4 : NA / 8;
    static_assert(QC >= 1 && NA % QC == 0 && QC * 256 <= SLOT, "fold pass");
    static_assert(KT % KB == 0 && KB % 4 == 0 && kChunk % KT == 0 && kWtileDepth == 2, "slab split");
    extern __shared__ __attribute__((aligned(16))) uint8_t wt_lds[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int g = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int NT = blockDim.x, NW = NT >> 6;
    const int mi = lane % LM, ni = lane / LM;
    const int64_t M = a.M, N = a.N, K = a.K;
    const int J = a.J;

    // workgroup -> tile.  Workgroups b, b + 8, b + 16, ... run on one XCD and take one contiguous range of the
    // tiles, in the order: the m tiles of a group of at most kGroupM for one n tile, then the next n tile, then
    // the next group.  So an XCD's L2 holds what its tiles share, and every XCD has as many (same box, against
    // tiles dealt round the XCDs one by one: 28672 x 4096 at M = 16 / 333 82 / 960 -> 75 / 931 us, 8192 x 28672
    // at M = 2048 11.03 -> 10.76 ms).
    int tm, tn;
    {
        const uint32_t b0 = a.reverse ? gridDim.x - 1 - blockIdx.x : blockIdx.x;
        const uint32_t total = (uint32_t)a.tiles_m * (uint32_t)a.tiles_n;
        const uint32_t i = (b0 & 7) * (gridDim.x >> 3) + (b0 >> 3);
        if (i >= total) return;                                     // padding workgroup: no tile
        const uint32_t gsz = min((uint32_t)kGroupM, (uint32_t)a.tiles_m);
        const uint32_t per = gsz * (uint32_t)a.tiles_n;             // tiles of a whole m group
        const uint32_t gm = i / per, j = i % per;
        const uint32_t gs = min(gsz, (uint32_t)a.tiles_m - gm * gsz);
        tm = __builtin_amdgcn_readfirstlane((int)(gm * gsz + j % gs));
        tn = __builtin_amdgcn_readfirstlane((int)(j / gs));
    }
    const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
    uint8_t* ring = wt_lds + g * RING;
    const uint32_t ring_base = lds_addr32(ring);
    float* tots = reinterpret_cast<float*>(wt_lds + NW * RING);     // [NA][64], when there are several rounds

    // swizzle of a row's pieces: eight rows in a row reach eight different 16-byte bank groups
    auto fx = [](int row) { return PX >= 8 ? (row & 7) : ((row * PX / 8) & (PX - 1)); };
    auto fw = [](int row) { return PW >= 8 ? (row & 7) : ((row * PW / 8) & (PW - 1)); };
    // staging roles: instruction u of this lane brings 16-byte position 64 u + lane of the slab image, which
    // holds piece (position % P) ^ f(row) of row position / P (rows past M or N: the last one again, never stored)
    int kx[XI], kw[WI];                 // first k of the piece within the slab
    uint32_t vx[XI], vw[WI];            // byte offset of row and piece from the tile's first row
#pragma unroll
    for (int u = 0; u < XI; ++u) {
        const int p = 64 * u + lane, row = min(p / PX, BM - 1);
        kx[u] = 4 * ((p % PX) ^ fx(p / PX));
        vx[u] = (uint32_t)(min((int64_t)row, M - 1 - m0) * K * 4) + 4u * kx[u];
    }
#pragma unroll
    for (int u = 0; u < WI; ++u) {
        const int p = 64 * u + lane, row = min(p / PW, BN - 1);
        kw[u] = (16 / (int)sizeof(WT)) * ((p % PW) ^ fw(p / PW));
        vw[u] = (uint32_t)(min((int64_t)row, N - 1 - n0) * K * (int)sizeof(WT)) + (uint32_t)sizeof(WT) * kw[u];
    }
    const char* xb = reinterpret_cast<const char*>(a.x + m0 * K);
    const char* wb = reinterpret_cast<const char*>(a.w) + n0 * K * (int)sizeof(WT);

    const int last_len = (int)(K - (int64_t)(J - 1) * kChunk);
    const int last_slabs = (last_len + KT - 1) / KT;
    const int nseg = g < J ? (J - 1 - g) / NW + 1 : 0;             // this wave's segments, and their slabs
    const bool has_last = nseg > 0 && g + (nseg - 1) * NW == J - 1;
    const int S = nseg * NSL - (has_last ? NSL - last_slabs : 0);
    auto slab_k = [&](int s) { return (int64_t)(g + s / NSL * NW) * kChunk + s % NSL * KT; };

    // AL: slab s by DMA into slot s % 2.  Pieces past K (a short last slab) repeat the row's first piece of
    // the slab and are never multiplied.
    auto issue = [&](int s) {
        const int64_t k0 = slab_k(s);
        const uint32_t slot = ring_base + (uint32_t)(s % kWtileDepth * SLOT);
        const char* sx = xb + k0 * 4;
        const char* sw = wb + k0 * (int)sizeof(WT);
        if (k0 + KT <= K) {
            dma_n(sw, vw, slot + SL::WOFF);
            dma_n(sx, vx, slot);
        } else {
            const int kl = (int)(K - k0);
            uint32_t tx[XI], tw[WI];
#pragma unroll
            for (int u = 0; u < XI; ++u) tx[u] = kx[u] < kl ? vx[u] : vx[u] - 4u * kx[u];
#pragma unroll
            for (int u = 0; u < WI; ++u) tw[u] = kw[u] < kl ? vw[u] : vw[u] - (uint32_t)sizeof(WT) * kw[u];
            dma_n(sw, tw, slot + SL::WOFF);
            dma_n(sx, tx, slot);
        }
    };
    // !AL: slab s into registers (any alignment; k past K as x = +0, w = -0), and from there into its slot
    uint4 rx[AL ? 1 : XI], rw[AL ? 1 : WI];
    auto load_regs = [&](int s) {
        const int64_t k0 = slab_k(s);
        const char* sx = xb + k0 * 4;
        const char* sw = wb + k0 * (int)sizeof(WT);
        constexpr int EW = 16 / (int)sizeof(WT);
        if (k0 + KT <= K) {
#pragma unroll
            for (int u = 0; u < XI; ++u) __builtin_memcpy(&rx[AL ? 0 : u], sx + vx[u], 16);
#pragma unroll
            for (int u = 0; u < WI; ++u) __builtin_memcpy(&rw[AL ? 0 : u], sw + vw[u], 16);
        } else {
            const int kl = (int)(K - k0);
#pragma unroll
            for (int u = 0; u < XI; ++u) {
                uint32_t e[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    uint32_t v = 0u;                                            // +0
                    if (kx[u] + i < kl) __builtin_memcpy(&v, sx + vx[u] + 4 * i, 4);
                    e[i] = v;
                }
                rx[AL ? 0 : u] = make_uint4(e[0], e[1], e[2], e[3]);
            }
#pragma unroll
            for (int u = 0; u < WI; ++u) {
                uint32_t e[4] = {0u, 0u, 0u, 0u};
#pragma unroll
                for (int i = 0; i < EW; ++i) {
                    if constexpr (BF) {
                        uint16_t v = 0x8000u;                                   // -0
                        if (kw[u] + i < kl) __builtin_memcpy(&v, sw + vw[u] + 2 * i, 2);
                        e[i / 2] |= (uint32_t)v << (16 * (i & 1));
                    } else {
                        uint32_t v = 0x80000000u;                               // -0
                        if (kw[u] + i < kl) __builtin_memcpy(&v, sw + vw[u] + 4 * i, 4);
                        e[i] = v;
                    }
                }
                rw[AL ? 0 : u] = make_uint4(e[0], e[1], e[2], e[3]);
            }
        }
    };
    int arrived = 0;                    // slabs made readable so far
    // make slab s readable (in order, once each)
    auto arrive = [&](int s) {
        if constexpr (AL) {
            dma_wait();
        } else {
            if (s < arrived || s >= S) return;
            uint4* slot = reinterpret_cast<uint4*>(ring + s % kWtileDepth * SLOT);
#pragma unroll
            for (int u = 0; u < XI; ++u) slot[64 * u + lane] = rx[AL ? 0 : u];
#pragma unroll
            for (int u = 0; u < WI; ++u) slot[SL::WOFF / 16 + 64 * u + lane] = rw[AL ? 0 : u];
            if (s + 1 < S) load_regs(s + 1);
            arrived = s + 1;
        }
    };

    float acc[TM][TN];
    using WV = typename std::conditional<BF, uint2, float4>::type;
    struct Ops {
        float4 x[KB / 4][TM];
        WV w[KB / 4][TN];
    };
    // four k of this lane's rows: 16 bytes of x, 8 bytes of BF16 W or 16 of FP32 W
    auto read4 = [&](const uint8_t* slot, int q, float4 (&ox)[TM], WV (&ow)[TN]) {
        // rows r LM + mi share the swizzle of row mi where LM rows are whole swizzle periods
        constexpr bool wper = PW >= 8 ? LN % 8 == 0 : LN * PW >= 8 && LN * PW / 8 % PW == 0;
        constexpr bool xper = PX >= 8 ? LM % 8 == 0 : LM * PX >= 8 && LM * PX / 8 % PX == 0;
#pragma unroll
        for (int c = 0; c < TN; ++c) {
            const int f = wper ? fw(ni) : fw(c * LN + ni);
            const uint8_t* p = slot + SL::WOFF + ni * (KT * (int)sizeof(WT)) + c * (LN * KT * (int)sizeof(WT));
            if constexpr (BF) ow[c] = *reinterpret_cast<const uint2*>(p + 16 * ((q >> 1) ^ f) + 8 * (q & 1));
            else ow[c] = *reinterpret_cast<const float4*>(p + 16 * (q ^ f));
        }
#pragma unroll
        for (int r = 0; r < TM; ++r) {
            const int f = xper ? fx(mi) : fx(r * LM + mi);
            ox[r] = *reinterpret_cast<const float4*>(slot + mi * (KT * 4) + 16 * (q ^ f) + r * (LM * KT * 4));
        }
    };
    auto fma4 = [&](const float4 (&ox)[TM], const WV (&ow)[TN]) {
#pragma unroll
        for (int kp = 0; kp < 2; ++kp) {
            float wv[2][TN];
#pragma unroll
            for (int c = 0; c < TN; ++c) {
                if constexpr (BF) {
                    widen2(kp == 0 ? ow[c].x : ow[c].y, wv[0][c], wv[1][c]);
                } else {
                    wv[0][c] = kp == 0 ? ow[c].x : ow[c].z;
                    wv[1][c] = kp == 0 ? ow[c].y : ow[c].w;
                }
            }
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
                for (int r = 0; r < TM; ++r) {
                    const float xv = kp == 0 ? (kk == 0 ? ox[r].x : ox[r].y) : (kk == 0 ? ox[r].z : ox[r].w);
#pragma unroll
                    for (int c = 0; c < TN; ++c) acc[r][c] = __builtin_fmaf(xv, wv[kk][c], acc[r][c]);
                }
            }
        }
    };
    auto read = [&](const uint8_t* slot, int b) {
        Ops o;
#pragma unroll
        for (int h = 0; h < KB / 4; ++h) read4(slot, b * (KB / 4) + h, o.x[h], o.w[h]);
        return o;
    };
    auto fma_ops = [&](const Ops& o) {
#pragma unroll
        for (int h = 0; h < KB / 4; ++h) fma4(o.x[h], o.w[h]);
    };

    if (S > 0) {
        if constexpr (AL) issue(0);
        else load_regs(0);
    }
    Ops cur;
    int s = 0;                                             // this wave's next slab
    const int rounds = (J + NW - 1) / NW;
    for (int t = 0; t < rounds; ++t) {
        const int j = t * NW + g;
#pragma unroll
        for (int r = 0; r < TM; ++r)
#pragma unroll
            for (int c = 0; c < TN; ++c) acc[r][c] = 0.0f;
        if (j < J) {
            const int len = j == J - 1 ? last_len : kChunk;
            const int nfull = len / KT;
            if (nfull > 0) {
                arrive(s);
                cur = read(ring + s % kWtileDepth * SLOT, 0);
            }
            for (int sl = 0; sl < nfull; ++sl, ++s) {
                const uint8_t* slot = ring + s % kWtileDepth * SLOT;
                // the other slot's reads are done: fill it with the next slab while this one is computed
                if constexpr (AL) {
                    lds_wait();
                    if (s + 1 < S) issue(s + 1);
                }
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    // the next operands are read while the current ones are multiplied (after the wave's
                    // last slab: bytes that are never used)
                    Ops nxt;
                    if (b + 1 < NB) {
                        nxt = read(slot, b + 1);
                    } else {
                        arrive(s + 1);
                        nxt = read(ring + (s + 1) % kWtileDepth * SLOT, 0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    fma_ops(cur);
                    __builtin_amdgcn_sched_barrier(0);
                    cur = nxt;
                }
            }
            if (nfull * KT < len) {                        // the short last slab of K
                arrive(s);
                const uint8_t* slot = ring + s % kWtileDepth * SLOT;
                const int nq = (len - nfull * KT + 3) / 4;
                for (int q = 0; q < nq; ++q) {
                    float4 ox[TM];
                    WV ow[TN];
                    read4(slot, q, ox, ow);
                    fma4(ox, ow);
                }
                ++s;
            }
            lds_wait();
        }
        // fold: partials through the slot of the last computed slab (the other one may be filling), QC
        // chains per lane at a time
        const int nact = min(NW, J - t * NW);
        const bool last = t == rounds - 1;
        float* part = reinterpret_cast<float*>(ring + (s + kWtileDepth - 1) % kWtileDepth * SLOT);
        const float* pfull =
            reinterpret_cast<const float*>(wt_lds + ((t + 1) * NSL + kWtileDepth - 1) % kWtileDepth * SLOT);
        const float* plast =
            reinterpret_cast<const float*>(wt_lds + (t * NSL + last_slabs + kWtileDepth - 1) % kWtileDepth * SLOT);
        const int nfold = last ? nact - 1 : nact;          // waves with whole segments this round
#pragma unroll
        for (int ch = 0; ch < NA / QC; ++ch) {
            if (j < J) {
#pragma unroll
                for (int q = 0; q < QC; ++q) part[64 * q + lane] = acc[(ch * QC + q) / TN][(ch * QC + q) % TN];
            }
            wg_barrier();
            // four neighbouring outputs per thread
            const float4* pf = reinterpret_cast<const float4*>(pfull);
            const float4* pl = reinterpret_cast<const float4*>(plast);
            float4* tt = reinterpret_cast<float4*>(tots + ch * QC * 64);
            auto add = [](const float4& u, const float4& v) { return make_float4(u.x + v.x, u.y + v.y, u.z + v.z, u.w + v.w); };
            for (int o = tid; o < 16 * QC; o += NT) {
                float4 v;
                int w = 0;
                if (t > 0) {
                    v = tt[o];
                } else {
                    v = nfold > 0 ? pf[o] : pl[o];         // the first partial starts the sum
                    w = 1;
                }
                for (; w + 4 <= nfold; w += 4) {
                    float4 pv[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) pv[u] = pf[(w + u) * (RING / 16) + o];
#pragma unroll
                    for (int u = 0; u < 4; ++u) v = add(v, pv[u]);
                }
                for (; w < nfold; ++w) v = add(v, pf[w * (RING / 16) + o]);
                if (w < nact) v = add(v, pl[w * (RING / 16) + o]);
                if (last) {
                    const int q = ch * QC + o / 16;
                    const float e[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int ln = (4 * o + i) % 64;
                        const int64_t gm = m0 + (q / TN) * LM + ln % LM, gn = n0 + (q % TN) * LN + ln / LM;
                        if (gm < M && gn < N) a.y[gm * N + gn] = a.bias ? e[i] + a.bias[gn] : e[i];
                    }
                } else {
                    tt[o] = v;
                }
            }
            wg_barrier();
        }
    }
}

namespace {

using WtileKernel = void (*)(WtileArgs);

// The kernels of wtile_builds, in its order.
template <typename WT, bool AL>
const WtileKernel* wtile_kernels() {
#define RG_B(LM, TM, TN, KT, NWMAX, WPE, KB, RATE) wtile_kernel<LM, TM, TN, KT, NWMAX, WPE, KB, WT, AL>,
    if constexpr (!AL) {
        static const WtileKernel k[] = {RG_WTILE_ANY(RG_B)};
        return k;
    } else if constexpr (sizeof(WT) == 2) {
        static const WtileKernel k[] = {RG_WTILE_BF16(RG_B)};
        return k;
    } else {
        static const WtileKernel k[] = {RG_WTILE_F32(RG_B)};
        return k;
    }
#undef RG_B
}

template <typename WT>
hipError_t launch_wtile_t(const float* x, const WT* w, const float* bias, float* y, int64_t M, int64_t N,
                          int64_t K, int build, int waves, bool aligned, int reverse, hipStream_t stream) {
    int nb = 0;
    const WtileBuild* bs = wtile_builds(sizeof(WT) == 4, aligned, &nb);
    if (build < 0 || build >= nb || waves < 1 || waves > bs[build].nwmax || K > kWtileMaxK) return hipErrorInvalidValue;
    if (aligned && ((((uintptr_t)x | (uintptr_t)w) & 15) != 0 || K % (16 / (int)sizeof(WT)) != 0))
        return hipErrorInvalidValue;
    const WtileBuild& b = bs[build];
    const int64_t J = (K + kChunk - 1) / kChunk;
    const int64_t lds = wtile_lds(b, J, waves);
    const int64_t tm = (M + b.bm - 1) / b.bm, tn = (N + b.bn - 1) / b.bn;
    if (lds > kWtileLds || tm > 0x7fffffff || tn > 0x7fffffff || !wtile_grid_ok(tm * tn, waves)) return hipErrorInvalidValue;
    const int64_t grid = wtile_grid(tm * tn);
    const WtileArgs a{x, w, bias, y, M, N, K, (int)J, (int)tm, (int)tn, reverse};
    const WtileKernel kernel = (aligned ? wtile_kernels<WT, true>() : wtile_kernels<WT, false>())[build];
    hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(64 * waves), (size_t)lds, stream, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_wtile(const float* x, const uint16_t* w, const float* bias, float* y, int64_t M, int64_t N,
                        int64_t K, int build, int waves, bool aligned, int reverse, hipStream_t stream) {
    return launch_wtile_t(x, w, bias, y, M, N, K, build, waves, aligned, reverse, stream);
}

hipError_t launch_wtile(const float* x, const float* w, const float* bias, float* y, int64_t M, int64_t N,
                        int64_t K, int build, int waves, bool aligned, int reverse, hipStream_t stream) {
    return launch_wtile_t(x, w, bias, y, M, N, K, build, waves, aligned, reverse, stream);
}

}  // namespace rg
