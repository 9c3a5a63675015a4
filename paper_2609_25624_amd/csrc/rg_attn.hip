// Fixed-order decode attention kernels for gfx950 (MI355X): the order
// RG-ATTN-1 and its exponential EXP1, both defined in include/rg_attn.h.
//
// One launch for short caches, three otherwise, or four where the maximum is a launch of its own
// (attn_route in rg_attn_rule.h; head dims other than 64, 128 and 256 always four), each
// deterministic by construction (no order that depends on the grid):
//   1. scores:   work item (b, g, j) = segment j (positions [256j, 256j + 256))
//                of kv head g of sequence b; its keys are staged in LDS and
//                thread l runs the dot product chain of position l for every
//                query head of the group, scales it, writes t, and the
//                workgroup writes the segment's maximum per head (max is
//                exact, so its tree shape does not matter).
//   2. max:      m[b][h] = the largest segment maximum (exact, so it is the same
//                value when the partials kernel reduces it per item instead).
//   3. partials: per work item, e_l = EXP1(t_l - m), the segment sum S_j (one
//                addition chain per head) and the segment numerators n_j[d]
//                (one fmaf chain per head and d over the positions in
//                ascending order; values and e staged in LDS).
//   4. fold:     workgroup (b, h) folds the S_j and n_j[d] in ascending j and
//                divides.
// The fused kernel runs 1 to 4 in one workgroup per (b, g).
// Kernel 1, and kernel 3 for other head dims, are persistent: a workgroup walks work items it,
// it + grid, ... (kernel 1 in steps of one 32 KB tile), fetching the next step into registers while it
// computes the current one from LDS.  Kernel 3 for head dims 64, 128 and 256 (but where a workgroup per
// segment leads at 64) and the fused kernel stream rows wave by wave through LDS rings by DMA.
// Arithmetic: binary32 fmaf / add / multiply / correctly rounded divide,
// denormals kept, no contraction (the build uses -ffp-contract=off).

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "rg_attn_rule.h"
#include "rg_kernels.h"

namespace rg {

// A 16-byte non-temporal load (key and value rows that a pass reads whole, once per call).
__device__ __forceinline__ uint4 ldnt(const uint4* p) {
    using E = __attribute__((ext_vector_type(4))) uint32_t;
    const E e = __builtin_nontemporal_load(reinterpret_cast<const E*>(p));
    return make_uint4(e.x, e.y, e.z, e.w);
}

namespace {

constexpr int kAttnSeg = 256;                 // positions per segment

// EXP1 of include/rg_attn.h.
__device__ __forceinline__ float exp1(float u) {
    if (u != u) return u;
    if (u < -87.0f) return 0.0f;
    const float k = __builtin_rintf(u * 0x1.715476p+0f);
    float r = __builtin_fmaf(-k, 0x1.62e4p-1f, u);
    r = __builtin_fmaf(-k, 0x1.7f7d1cp-20f, r);
    float p = 0x1.a01a02p-13f;
    p = __builtin_fmaf(p, r, 0x1.6c16c2p-10f);
    p = __builtin_fmaf(p, r, 0x1.111112p-7f);
    p = __builtin_fmaf(p, r, 0x1.555556p-5f);
    p = __builtin_fmaf(p, r, 0x1.555556p-3f);
    p = __builtin_fmaf(p, r, 0.5f);
    p = __builtin_fmaf(p, r, 1.0f);
    p = __builtin_fmaf(p, r, 1.0f);
    return p * __uint_as_float((uint32_t)((int)k + 127) << 23);
}

// The same without branches (the discarded 2^k of u < -87 is any value).
__device__ __forceinline__ float exp1_select(float u) {
    const float k = __builtin_rintf(u * 0x1.715476p+0f);
    float r = __builtin_fmaf(-k, 0x1.62e4p-1f, u);
    r = __builtin_fmaf(-k, 0x1.7f7d1cp-20f, r);
    float p = 0x1.a01a02p-13f;
    p = __builtin_fmaf(p, r, 0x1.6c16c2p-10f);
    p = __builtin_fmaf(p, r, 0x1.111112p-7f);
    p = __builtin_fmaf(p, r, 0x1.555556p-5f);
    p = __builtin_fmaf(p, r, 0x1.555556p-3f);
    p = __builtin_fmaf(p, r, 0.5f);
    p = __builtin_fmaf(p, r, 1.0f);
    p = __builtin_fmaf(p, r, 1.0f);
    const float k0 = u >= -87.0f ? k : 0.0f;          // a k the conversion is defined for
    const float e = p * __uint_as_float((uint32_t)((int)k0 + 127) << 23);
    return u != u ? u : (u < -87.0f ? 0.0f : e);
}

__device__ __forceinline__ int clamp_len(const int32_t* lens, int64_t b, int64_t Lmax) {
    const int64_t L = lens[b];
    return (int)(L < 0 ? 0 : (L > Lmax ? Lmax : L));
}

// A step's tile: `rows` rows of VPR 16-byte vectors (8 bf16 each) taken from a
// [*, D] bf16 block at row stride D, staged in LDS at a row stride of
// 8 * VPR + 8 (16 bytes of pad: lanes that read one row each hit different
// banks).  It is fetched into registers one step ahead (every load issued
// before the first use) and stored to LDS between barriers; rows past the
// sequence are +0.  Thread t holds vectors t, t + 256, ...; the row of vector i
// is i / VPR (a shift for the fixed shapes, else a multiply by `vmagic` =
// ceil(2^32 / vpr), exact for i < 8192).
template <int NV, int VPR>   // VPR > 0: fixed vectors per row; 0: vpr at run time
struct Tile {
    uint4 r[NV];
    __device__ __forceinline__ static int row_of(int i, int vpr, uint32_t vmagic) {
        if constexpr (VPR > 0) return i / VPR;
        return vpr == 1 ? i : (int)__umulhi((uint32_t)i, vmagic);
    }
    __device__ __forceinline__ void fetch(const uint16_t* __restrict__ src, int64_t stride, int rows, int vpr,
                                          uint32_t vmagic) {
        if constexpr (VPR > 0) vpr = VPR;
        const int limit = rows * vpr;
#pragma unroll
        for (int u = 0; u < NV; ++u) {
            const int i = (int)threadIdx.x + 256 * u;
            const int row = row_of(i, vpr, vmagic);
            r[u] = i < limit ? ldnt(reinterpret_cast<const uint4*>(src + row * stride + 8 * (i - row * vpr)))
                             : make_uint4(0u, 0u, 0u, 0u);
        }
    }
    __device__ __forceinline__ void store(uint16_t* dst, int rows_total, int vpr, uint32_t vmagic) const {
        if constexpr (VPR > 0) vpr = VPR;
#pragma unroll
        for (int u = 0; u < NV; ++u) {
            const int i = (int)threadIdx.x + 256 * u;
            if (VPR > 0 || i < rows_total * vpr) {
                const int row = row_of(i, vpr, vmagic);
                *reinterpret_cast<uint4*>(dst + 8 * (i + row)) = r[u];   // row * (8 vpr + 8) + 8 (i % vpr)
            }
        }
    }
};

// Work item it = (b * Hkv + g) * J + j: segment j of kv head g of sequence b.
struct Item {
    int b, g, j;
    int L, l0, rows;
};

__device__ __forceinline__ Item item_of(const AttnArgs& a, int it) {
    Item w;
    const int J = (int)a.J, Hkv = (int)a.Hkv;
    const int bg = it / J;
    w.j = it - bg * J;
    w.b = bg / Hkv;
    w.g = bg - w.b * Hkv;
    w.L = clamp_len(a.lens, w.b, a.Lmax);
    w.l0 = w.j * kAttnSeg;
    w.rows = w.L - w.l0 < kAttnSeg ? w.L - w.l0 : kAttnSeg;
    return w;
}

// The first item at or after `it`, stepping by the grid, that holds positions.
__device__ __forceinline__ int next_item(const AttnArgs& a, int it, int items) {
    while (it < items && item_of(a, it).rows <= 0) it += (int)gridDim.x;
    return it;
}

typedef const __attribute__((address_space(4))) float cfloat;   // read-only: uniform loads go to SGPRs

// Exact maximum over the workgroup of one value per thread: lanes by xor
// shuffles, then the four waves through LDS (fmaxf is exact and NaN never
// wins, so any tree gives the same value).
template <int G>
__device__ __forceinline__ void block_max(float (&v)[G], float (*wred)[G]) {
#pragma unroll
    for (int sh = 32; sh > 0; sh >>= 1)
#pragma unroll
        for (int i = 0; i < G; ++i) v[i] = __builtin_fmaxf(v[i], __shfl_xor(v[i], sh, 64));
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int i = 0; i < G; ++i) wred[threadIdx.x >> 6][i] = v[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < G; ++i)
        v[i] = __builtin_fmaxf(__builtin_fmaxf(wred[0][i], wred[1][i]), __builtin_fmaxf(wred[2][i], wred[3][i]));
}

// 1. scores and segment maxima.  Work item = segment; its NC steps take the keys'
// columns [c DC, c DC + DC) in turn (DC = 64 for the fixed head dims, else DC = D
// in one step), so each thread's dot product chain of position l continues across
// the steps in ascending d.  G query heads per kv head, their chains interleaved;
// q is read with uniform (scalar) loads.
template <int G, int DC, int NC, bool EXACT>
__global__ void __launch_bounds__(256) attn_scores_kernel(AttnArgs a) {
    constexpr int VPR = EXACT ? DC / 8 : 0;
    constexpr int NV = DC / 8;                                                // vectors per thread (256 rows)
    __shared__ __attribute__((aligned(16))) uint16_t ks[kAttnSeg * (DC + 8)]; // [256][DC + 8]
    __shared__ float wred[4][G];
    const int D = EXACT ? DC * NC : (int)a.D, l = threadIdx.x;
    const int dc = EXACT ? DC : D;                    // columns per step
    const int vpr = dc / 8;
    const int items = (int)(a.B * a.Hkv * a.J);
    cfloat* q4 = (cfloat*)a.q;
    Tile<NV, VPR> tile;
    auto fetch = [&](const Item& w, int c) {
        tile.fetch(a.k + (((int64_t)w.b * a.Hkv + w.g) * a.Lmax + w.l0) * D + c * dc, D, w.rows, vpr, a.vmagic);
    };
    int it = next_item(a, (int)blockIdx.x, items);
    Item w;
    int c = 0;
    if (it < items) {
        w = item_of(a, it);
        fetch(w, 0);
    }
    float z[G];
    while (it < items) {
        __syncthreads();                              // the previous step's reads of LDS are done
        tile.store(ks, kAttnSeg, vpr, a.vmagic);
        __syncthreads();
        const Item cur = w;
        const int cc = c;
        if (c + 1 < NC) {
            ++c;
        } else {
            c = 0;
            it = next_item(a, it + (int)gridDim.x, items);
            if (it < items) w = item_of(a, it);
        }
        if (it < items) fetch(w, c);                  // in flight during this step's chains
        if (cc == 0) {
#pragma unroll
            for (int i = 0; i < G; ++i) z[i] = 0.0f;
        }
        const int64_t h0 = (int64_t)cur.g * G;
        const int64_t qbase = ((int64_t)cur.b * a.H + h0) * D + cc * dc;
        if (l < cur.rows) {
            const uint16_t* kr = ks + l * (dc + 8);
#pragma unroll 1
            for (int d = 0; d < DC; d += 8) {
                if (!EXACT && d >= dc) break;
                const uint4 kv = *reinterpret_cast<const uint4*>(kr + d);
                const uint32_t w4[4] = {kv.x, kv.y, kv.z, kv.w};
                float kf[8];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    kf[2 * e] = __uint_as_float(w4[e] << 16);
                    kf[2 * e + 1] = __uint_as_float(w4[e] & 0xffff0000u);
                }
#pragma unroll
                for (int i = 0; i < G; ++i)
#pragma unroll
                    for (int e = 0; e < 8; ++e) z[i] = __builtin_fmaf(q4[qbase + i * D + d + e], kf[e], z[i]);
            }
        }
        if (cc == NC - 1) {
            float t[G];
#pragma unroll
            for (int i = 0; i < G; ++i) {
                t[i] = l < cur.rows ? z[i] * a.scale : -__builtin_inff();
                if (l < cur.rows) a.t[(((int64_t)cur.b * a.H + h0 + i) * a.Lmax) + cur.l0 + l] = t[i];
            }
            block_max<G>(t, wred);
            float mine = t[0];                        // thread l < G writes head l's maximum
#pragma unroll
            for (int i = 1; i < G; ++i) mine = (l == i) ? t[i] : mine;
            if (l < G) a.segmax[((int64_t)cur.b * a.H + h0 + l) * a.J + cur.j] = mine;
        }
    }
}

// 1'. the same scores with 128 threads per workgroup, thread l holding positions
// l and l + 128 (head dims 64, 128, 256; 32-column key steps).  Each q value
// (read with uniform loads) then feeds two FMAs per thread, which halves the
// scalar-load traffic per FMA of the 256-thread kernel.
template <int G, int D>
__global__ void __launch_bounds__(128) attn_scores2_kernel(AttnArgs a) {
    constexpr int DC = 32, NC = D / DC, PAD = DC + 8;
    constexpr int NV = kAttnSeg * DC / 8 / 128;       // 16-byte vectors per thread per step (8)
    __shared__ __attribute__((aligned(16))) uint16_t ks[kAttnSeg * PAD];   // [256][DC + 8]
    __shared__ float wred[2][G];
    const int tid = threadIdx.x;
    const int items = (int)(a.B * a.Hkv * a.J);
    cfloat* q4 = (cfloat*)a.q;
    uint4 kr[NV];
    auto fetch = [&](const Item& w, int c) {
        const uint16_t* src = a.k + (((int64_t)w.b * a.Hkv + w.g) * a.Lmax + w.l0) * D + c * DC;
#pragma unroll
        for (int u = 0; u < NV; ++u) {
            const int i = tid + 128 * u;               // vector i: row i / 4, columns 8 (i % 4)
            const int row = i >> 2;
            // a normal load: each pass reads 64 bytes of a row whose other bytes the next
            // passes read (non-temporal here measured slower on the 70B-shaped heads)
            kr[u] = row < w.rows ? *reinterpret_cast<const uint4*>(src + (int64_t)row * D + 8 * (i & 3))
                                 : make_uint4(0u, 0u, 0u, 0u);
        }
    };
    int it = next_item(a, (int)blockIdx.x, items);
    Item w;
    int c = 0;
    if (it < items) {
        w = item_of(a, it);
        fetch(w, 0);
    }
    float z0[G], z1[G];
    while (it < items) {
        __syncthreads();                              // the previous step's reads of LDS are done
#pragma unroll
        for (int u = 0; u < NV; ++u) {
            const int i = tid + 128 * u;
            *reinterpret_cast<uint4*>(ks + (i >> 2) * PAD + 8 * (i & 3)) = kr[u];
        }
        __syncthreads();
        const Item cur = w;
        const int cc = c;
        if (c + 1 < NC) {
            ++c;
        } else {
            c = 0;
            it = next_item(a, it + (int)gridDim.x, items);
            if (it < items) w = item_of(a, it);
        }
        if (it < items) fetch(w, c);                  // in flight during this step's chains
        if (cc == 0) {
#pragma unroll
            for (int i = 0; i < G; ++i) z0[i] = z1[i] = 0.0f;
        }
        const int64_t h0 = (int64_t)cur.g * G;
        const int64_t qbase = ((int64_t)cur.b * a.H + h0) * D + cc * DC;
        const uint16_t* kp0 = ks + tid * PAD;
        const uint16_t* kp1 = ks + (tid + 128) * PAD;
#pragma unroll 1
        for (int d = 0; d < DC; d += 8) {
            const uint4 k0 = *reinterpret_cast<const uint4*>(kp0 + d);
            const uint4 k1 = *reinterpret_cast<const uint4*>(kp1 + d);
            const uint32_t a4[4] = {k0.x, k0.y, k0.z, k0.w}, b4[4] = {k1.x, k1.y, k1.z, k1.w};
            float f0[8], f1[8];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                f0[2 * e] = __uint_as_float(a4[e] << 16);
                f0[2 * e + 1] = __uint_as_float(a4[e] & 0xffff0000u);
                f1[2 * e] = __uint_as_float(b4[e] << 16);
                f1[2 * e + 1] = __uint_as_float(b4[e] & 0xffff0000u);
            }
#pragma unroll
            for (int i = 0; i < G; ++i)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float qv = q4[qbase + i * D + d + e];
                    z0[i] = __builtin_fmaf(qv, f0[e], z0[i]);
                    z1[i] = __builtin_fmaf(qv, f1[e], z1[i]);
                }
        }
        if (cc == NC - 1) {
            // t for the valid positions; the segment maximum per head over them (exact)
            const int l0 = tid, l1 = tid + 128;
            float t[G];
#pragma unroll
            for (int i = 0; i < G; ++i) {
                const float t0 = l0 < cur.rows ? z0[i] * a.scale : -__builtin_inff();
                const float t1 = l1 < cur.rows ? z1[i] * a.scale : -__builtin_inff();
                float* tp = a.t + (((int64_t)cur.b * a.H + h0 + i) * a.Lmax) + cur.l0;
                if (l0 < cur.rows) tp[l0] = t0;
                if (l1 < cur.rows) tp[l1] = t1;
                t[i] = __builtin_fmaxf(t0, t1);
            }
#pragma unroll
            for (int sh = 32; sh > 0; sh >>= 1)
#pragma unroll
                for (int i = 0; i < G; ++i) t[i] = __builtin_fmaxf(t[i], __shfl_xor(t[i], sh, 64));
            if ((tid & 63) == 0) {
#pragma unroll
                for (int i = 0; i < G; ++i) wred[tid >> 6][i] = t[i];
            }
            __syncthreads();
            if (tid < G) {
                float mine = wred[0][0];
#pragma unroll
                for (int i = 0; i < G; ++i) mine = (tid == i) ? __builtin_fmaxf(wred[0][i], wred[1][i]) : mine;
                a.segmax[((int64_t)cur.b * a.H + h0 + tid) * a.J + cur.j] = mine;
            }
        }
    }
}

// 2. m[b][h] = the largest segment maximum (exact).  One thread per (b, h) for up to
// kMaxThreadSegs segments.
__global__ void __launch_bounds__(256) attn_max_kernel(AttnArgs a) {
    const int64_t bh = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (bh >= a.B * a.H) return;
    const int L = clamp_len(a.lens, bh / a.H, a.Lmax);
    const int Jb = (L + kAttnSeg - 1) / kAttnSeg;
    const float* sm = a.segmax + bh * a.J;
    float m = -__builtin_inff();
    int jj = 0;
    for (; jj + 8 <= Jb; jj += 8) {
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = sm[jj + i];
#pragma unroll
        for (int i = 0; i < 8; ++i) m = __builtin_fmaxf(m, v[i]);
    }
    for (; jj < Jb; ++jj) m = __builtin_fmaxf(m, sm[jj]);
    a.mmax[bh] = m;
}

// The same with one wave per (b, h), its lanes over the segments: with one thread a row of 512 segments is a chain of 64
// batches of loads (D = 64, eight heads, one sequence of 131072 positions: the call 42.0 -> 35.4 us; a short row's wave
// takes 0.7 us more than its thread).
__global__ void __launch_bounds__(256) attn_max_rows_kernel(AttnArgs a) {
    const int64_t bh = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (bh >= a.B * a.H) return;
    const int L = clamp_len(a.lens, bh / a.H, a.Lmax);
    const int Jb = (L + kAttnSeg - 1) / kAttnSeg;
    const float* sm = a.segmax + bh * a.J;
    float m = -__builtin_inff();
    for (int j = threadIdx.x & 63; j < Jb; j += 64) m = __builtin_fmaxf(m, sm[j]);
#pragma unroll
    for (int sh = 32; sh > 0; sh >>= 1) m = __builtin_fmaxf(m, __shfl_xor(m, sh, 64));
    if ((threadIdx.x & 63) == 0) a.mmax[bh] = m;
}

constexpr int64_t kMaxThreadSegs = 16;

hipError_t launch_max(const AttnArgs& a, hipStream_t stream) {
    const int64_t rows = a.B * a.H;
    if (a.J <= kMaxThreadSegs)
        hipLaunchKernelGGL(attn_max_kernel, dim3((unsigned)((rows + 255) / 256)), dim3(256), 0, stream, a);
    else
        hipLaunchKernelGGL(attn_max_rows_kernel, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, stream, a);
    return hipGetLastError();
}

// 3. exponentials and the segment partials S_j and n_j[d] (head dim 64, and the head dims without wave
// passes).  Work item = segment, all its 256 value rows staged at once.  e for the segment is computed
// into LDS ([head][position], -0 past the sequence).  Unit u =
// (head, pair of adjacent d): two fmaf chains over the positions; threads tid < G
// also run the segment sum of head tid (an addition chain).  Chains run over all
// 256 positions of the segment: past the sequence e = -0 and the values are +0,
// so a padded step is fmaf(-0, +0, n) = -0 + n = n and s + (-0) = s for every n and
// s, including a numerator that is -0 (a negative product e * v that underflows).
// (A +0 pad would turn such a -0 numerator into +0.)
template <int G, int DM, bool EXACT>
__global__ void __launch_bounds__(256) attn_partials_kernel(AttnArgs a) {
    constexpr int RS = kAttnSeg;                      // value rows staged
    constexpr int VPR = EXACT ? DM / 8 : 0;
    constexpr int NV = RS * DM / 8 / 256;             // vectors per thread
    constexpr int UPT = (G * DM / 2 + 255) / 256;     // units per thread
    __shared__ __attribute__((aligned(16))) float es[G * kAttnSeg];           // [G][256]
    __shared__ __attribute__((aligned(16))) uint16_t vs[RS * (DM + 8)];       // [RS][D + 8]
    const int D = EXACT ? DM : (int)a.D, tid = threadIdx.x;
    const int vpr = D / 8;
    const int items = (int)(a.B * a.Hkv * a.J);
    Tile<NV, VPR> tile;
    float tr[G], mr[G];
    auto fetch = [&](const Item& w) {
        tile.fetch(a.v + (((int64_t)w.b * a.Hkv + w.g) * a.Lmax + w.l0) * D, D, w.rows < RS ? w.rows : RS, vpr, a.vmagic);
        const int64_t h0 = (int64_t)w.g * G;
#pragma unroll
        for (int i = 0; i < G; ++i) {
            tr[i] = tid < w.rows ? a.t[((int64_t)w.b * a.H + h0 + i) * a.Lmax + w.l0 + tid] : 0.0f;
            mr[i] = a.mmax[(int64_t)w.b * a.H + h0 + i];
        }
    };
    int it = next_item(a, (int)blockIdx.x, items);
    Item w;
    if (it < items) {
        w = item_of(a, it);
        fetch(w);
    }
    const int npd = D / 2;
    const int nunits = G * npd;
    while (it < items) {
        __syncthreads();
        tile.store(vs, RS, vpr, a.vmagic);
#pragma unroll
        for (int i = 0; i < G; ++i) es[i * kAttnSeg + tid] = tid < w.rows ? exp1(tr[i] - mr[i]) : -0.0f;
        __syncthreads();
        const Item cur = w;
        it = next_item(a, it + (int)gridDim.x, items);
        if (it < items) {
            w = item_of(a, it);
            fetch(w);                                 // in flight during this item's chains
        }
#pragma unroll
        for (int k = 0; k < UPT; ++k) {
            const int u = tid + 256 * k;
            if (u < nunits) {
                const int hh = u / npd, d = 2 * (u - hh * npd);
                const bool sums = k == 0 && tid < G;
                const float* ep = es + hh * kAttnSeg;
                const float* sp = es + (tid < G ? tid : 0) * kAttnSeg;
                const uint16_t* vp = vs + d;
                float x0 = 0.0f, x1 = 0.0f, sm = 0.0f;
#pragma unroll 2
                for (int l = 0; l < RS; l += 8) {
                    const float4 e0 = *reinterpret_cast<const float4*>(ep + l);
                    const float4 e1 = *reinterpret_cast<const float4*>(ep + l + 4);
                    const float ev[8] = {e0.x, e0.y, e0.z, e0.w, e1.x, e1.y, e1.z, e1.w};
                    uint32_t vv[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) vv[i] = *reinterpret_cast<const uint32_t*>(vp + (l + i) * (D + 8));
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        x0 = __builtin_fmaf(ev[i], __uint_as_float(vv[i] << 16), x0);
                        x1 = __builtin_fmaf(ev[i], __uint_as_float(vv[i] & 0xffff0000u), x1);
                    }
                    if (sums) {
                        const float4 s0 = *reinterpret_cast<const float4*>(sp + l);
                        const float4 s1 = *reinterpret_cast<const float4*>(sp + l + 4);
                        sm = sm + s0.x; sm = sm + s0.y; sm = sm + s0.z; sm = sm + s0.w;
                        sm = sm + s1.x; sm = sm + s1.y; sm = sm + s1.z; sm = sm + s1.w;
                    }
                }
                float* np = a.npart + (((int64_t)cur.b * a.H + cur.g * G + hh) * a.J + cur.j) * D + d;
                np[0] = x0;
                np[1] = x1;
                if (sums) a.spart[((int64_t)cur.b * a.H + cur.g * G + tid) * a.J + cur.j] = sm;
            }
        }
    }
}

// One 16-byte global -> LDS DMA per lane (lane l writes LDS [lds_base + 16 l, +16)), non-temporal: key and value rows are
// read once, in whole 128-byte lines.  M0 is saved and restored and never read in the cycle after a write.
__device__ __forceinline__ void attn_dma16(const void* sbase, uint32_t voff, uint32_t lds_base) {
    uint32_t saved;
    asm volatile(
        "s_mov_b32 %0, m0\n\t"
        "s_mov_b32 m0, %2\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %1, %3 nt\n\t"
        "s_mov_b32 m0, %0\n\t"
        : "=&s"(saved)
        : "v"(voff), "s"(lds_base), "s"(sbase)
        : "memory");
}
template <int N>
__device__ __forceinline__ void attn_vm_wait() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ void attn_lds_wait() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// The two bfloat16 of a dword, widened exactly; the odd element in the even register of a pair and the even
// element in the odd one (the other operand's registers have the parity of the element, and an FMA whose operands
// all have one parity holds up the SIMD's other wave).
__device__ __forceinline__ void attn_widen2(uint32_t d, float& even, float& odd) {
    uint64_t pair = ((uint64_t)(d << 16) << 32) | (d & 0xffff0000u);
    asm volatile("" : "+v"(pair));                    // volatile: kept in order, so that few pairs are live at a time
    even = __uint_as_float((uint32_t)(pair >> 32));
    odd = __uint_as_float((uint32_t)pair);
}

// ---------------------------------------------------------------------------
// Wave passes (head dims 64, 128 and 256).  Each wave streams its own rows by DMA through its own LDS ring
// and meets no barrier inside a pass.
// ---------------------------------------------------------------------------
template <int GP, int D>
struct KeySteps {
    static constexpr int DC = D < 128 ? D : 128;                // columns whose q a lane holds at a time
    static constexpr int NCK = D / DC;                          // passes over the keys
    static constexpr int P = 64 / GP;                           // positions a wave's lanes hold at a time
    static constexpr int CC = GP == 1 && DC == 128 ? 64 : DC;   // columns per step
    static constexpr int NSUB = DC / CC;                        // steps per row group
    // row groups per step (chains per lane, two where a step then stays within 8 KB: a lone chain waits for itself)
    static constexpr int NCH = P * CC * 2 >= 8192 ? 1 : P * CC * 2 >= 2048 ? 2 : 4;
    static constexpr int RS = P * NCH;                          // key rows per step
    static constexpr int STEP = RS * CC * 2;                    // bytes: 4 or 8 KB
    static constexpr int RING = STEP > 4096 ? 2 * STEP : 12288;
    static constexpr int NS = RING / STEP;                      // steps in the ring
    static constexpr int UNIT = 128;                            // positions per unit
};
template <int GP, int D, int CS, int RINGB = 12288, int ECP = GP >= 4 ? 128 : 256>
struct ValueSteps {
    static constexpr int DH = D / CS;                           // value columns of a unit
    static constexpr int RS = 4096 / (DH * 2);                  // value rows per 4 KB step
    static constexpr int EC = ECP;                              // positions whose e are in LDS at a time
    static constexpr int RING = RINGB;
};

// Scores of units first, first + stride, ... (128 positions each) of kv head g of sequence b, `nu` of them.  Lane
// (position p, head h) = (lane / GP, lane % GP) runs the whole dot product chain of its position and head
// with its head's q in registers; key rows are XOR-swizzled in 16-byte pieces.  t goes to the workspace; returns the
// lane's largest t (its head's; -inf if it has none).
template <int GP, int D>
__device__ __forceinline__ float key_pass(const AttnArgs& a, int b, int g, int G, int L, int first, int stride, int nu,
                                          uint8_t* ring) {
    using KS = KeySteps<GP, D>;
    constexpr int CC = KS::CC, NCH = KS::NCH, P = KS::P, NSUB = KS::NSUB, NS = KS::NS, STEP = KS::STEP;
    constexpr int NI = STEP / 1024;                   // DMA instructions per step
    constexpr int SPU = KS::UNIT / KS::RS * NSUB;     // steps per unit
    constexpr int PCK = CC / 8;                       // 16-byte pieces per row of a step
    constexpr int LOGGP = GP == 1 ? 0 : GP == 2 ? 1 : GP == 4 ? 2 : 3;
    static_assert(KS::RS <= KS::UNIT && PCK % 8 == 0 && KS::UNIT % KS::RS == 0, "key step");
    const int lane = threadIdx.x & 63;
    const uint32_t ring_base = (uint32_t)(uintptr_t)((const __attribute__((address_space(3))) void*)ring);
    const int64_t h0 = (int64_t)b * a.H + (int64_t)g * G;
    float* tb = a.t + h0 * a.Lmax;
    const int hq = lane & (GP - 1), pos = lane >> LOGGP;
    const int hh = hq < G ? hq : G - 1;               // lanes past the group's heads repeat the last one
    const int S = nu * SPU;
    float mymax = -__builtin_inff();
#pragma unroll 1
    for (int ck = 0; ck < KS::NCK; ++ck) {
        const char* kb = reinterpret_cast<const char*>(a.k + ((int64_t)b * a.Hkv + g) * a.Lmax * D + ck * KS::DC);
        auto issue = [&](int s) {
            const int u = s / SPU, r = s - u * SPU;
            const int l0 = (first + stride * u) * KS::UNIT + r / NSUB * KS::RS;   // the step's first position
            const int from = min(l0, L - 1), rmax = L - 1 - from;               // past L: the last row again
            const char* sb = kb + (int64_t)from * (D * 2) + (r % NSUB) * (CC * 2);
            const uint32_t slot = ring_base + (uint32_t)(s % NS * STEP);
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int p = 64 * i + lane, row = p / PCK, pc = (p % PCK) ^ (row & 7);
                attn_dma16(sb, (uint32_t)(min(row, rmax) * (D * 2) + 16 * pc), slot + 1024u * i);
            }
        };
#pragma unroll
        for (int s = 0; s < NS - 1; ++s)
            if (s < S) issue(s);
        float q[KS::DC];
        const float4* qp = reinterpret_cast<const float4*>(a.q + (h0 + hh) * D + ck * KS::DC);
#pragma unroll
        for (int i = 0; i < KS::DC / 4; ++i) {
            const float4 v = qp[i];
            q[4 * i] = v.x; q[4 * i + 1] = v.y; q[4 * i + 2] = v.z; q[4 * i + 3] = v.w;
        }
        float z[NCH];
#pragma unroll 1
        for (int s0 = 0; s0 < S; s0 += NSUB) {
            const int u = s0 / SPU, r = s0 - u * SPU;
            const int l0 = (first + stride * u) * KS::UNIT + r / NSUB * KS::RS + pos;   // this lane's first position
#pragma unroll
            for (int c = 0; c < NCH; ++c) {
                z[c] = 0.0f;
                if (KS::NCK > 1 && ck > 0 && l0 + c * P < L) z[c] = tb[(int64_t)hh * a.Lmax + l0 + c * P];
            }
#pragma unroll
            for (int sub = 0; sub < NSUB; ++sub) {
                const int s = s0 + sub;
                if (NS > 2 && s + NS - 2 < S) attn_vm_wait<(NS - 2) * NI>();
                else attn_vm_wait<0>();
                attn_lds_wait();
                if (s + NS - 1 < S) issue(s + NS - 1);
                const uint8_t* slot = ring + s % NS * STEP;
                // the next piece of each row is read while the current ones are multiplied
                auto piece = [&](int pc, uint4 (&kv)[NCH]) {
#pragma unroll
                    for (int c = 0; c < NCH; ++c) {
                        const int row = c * P + pos;
                        kv[c] = *reinterpret_cast<const uint4*>(slot + row * (CC * 2) + 16 * (pc ^ (row & 7)));
                    }
                };
                uint4 kv[NCH], kn[NCH];
                piece(0, kv);
#pragma unroll
                for (int pc = 0; pc < PCK; ++pc) {
                    if (pc + 1 < PCK) piece(pc + 1, kn);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        float k0[NCH], k1[NCH];
#pragma unroll
                        for (int c = 0; c < NCH; ++c) {
                            const uint32_t w = e == 0 ? kv[c].x : e == 1 ? kv[c].y : e == 2 ? kv[c].z : kv[c].w;
                            attn_widen2(w, k0[c], k1[c]);
                        }
                        const float q0 = q[sub * CC + 8 * pc + 2 * e], q1 = q[sub * CC + 8 * pc + 2 * e + 1];
#pragma unroll
                        for (int c = 0; c < NCH; ++c) z[c] = __builtin_fmaf(q0, k0[c], z[c]);
#pragma unroll
                        for (int c = 0; c < NCH; ++c) z[c] = __builtin_fmaf(q1, k1[c], z[c]);
                    }
#pragma unroll
                    for (int c = 0; c < NCH; ++c) asm volatile("" : "+v"(z[c]));   // this piece's FMAs end here
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int c = 0; c < NCH; ++c) kv[c] = kn[c];
                }
            }
#pragma unroll
            for (int c = 0; c < NCH; ++c) {
                const float t = ck == KS::NCK - 1 ? z[c] * a.scale : z[c];
                if (l0 + c * P < L) {
                    if (ck == KS::NCK - 1) mymax = __builtin_fmaxf(mymax, t);
                    if (hq < G) tb[(int64_t)hq * a.Lmax + l0 + c * P] = t;
                }
            }
        }
        attn_lds_wait();
    }
    return mymax;
}

// Segment partials of units first, first + stride, ... below Jb * CS (segment unit / CS, value columns part unit % CS) of
// kv head g of sequence b.  The value stream starts, then row_max(m) brings the group's row maxima;
// the wave turns t into e (LDS, [position][head], EC positions at a time) and lane p runs the numerator chains of its
// columns for GH heads (the group's G where the kernel is built for them, else GP).  Lanes < G sum e.
template <int GH, typename VS, int GP, int D, int CS, typename F>
__device__ __forceinline__ void value_pass(const AttnArgs& a, int b, int g, int G, int L, int Jb, int first, int stride,
                                           uint8_t* ring, float* es, F row_max) {
    constexpr int DH = VS::DH, RS = VS::RS, EC = VS::EC, NS = VS::RING / 4096, NI = 4;
    constexpr int SEG = kAttnSeg / RS;                // steps of a whole segment
    constexpr int SVC = EC / RS;                      // steps per chunk of e
    constexpr int NT = EC * GH / 64;                  // scores per lane per chunk
    constexpr int PPL = DH >= 128 ? DH / 128 : 0;     // value pairs per lane (0: one column)
    constexpr int NC = PPL > 0 ? PPL : 1;
    static_assert(EC % RS == 0 && kAttnSeg % EC == 0, "value step");
    const int lane = threadIdx.x & 63;
    const uint32_t ring_base = (uint32_t)(uintptr_t)((const __attribute__((address_space(3))) void*)ring);
    const int64_t h0 = (int64_t)b * a.H + (int64_t)g * G;
    const float* tb = a.t + h0 * a.Lmax;
    const char* vb = reinterpret_cast<const char*>(a.v + ((int64_t)b * a.Hkv + g) * a.Lmax * D);
    const int units = Jb * CS;
    const int nv = first < units ? (units - 1 - first) / stride + 1 : 0;
    // steps of this wave's units: whole segments but for the last one of the sequence
    const int last_rows = L - (Jb - 1) * kAttnSeg;
    const bool has_last = nv > 0 && (first + stride * (nv - 1)) / CS == Jb - 1;
    const int S = nv * SEG - (has_last ? (kAttnSeg - last_rows) / RS : 0);
    auto issue = [&](int s) {
        const int u = s / SEG, r = s - u * SEG;
        const int unit = first + stride * u;
        const int l0 = unit / CS * kAttnSeg + r * RS;                           // < L
        const char* sb = vb + ((int64_t)l0 * D + unit % CS * DH) * 2;
        const int rmax = L - 1 - l0;
        const uint32_t slot = ring_base + (uint32_t)(s % NS * 4096);
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int p = 64 * i + lane, row = p / (DH / 8), pc = p % (DH / 8);
            attn_dma16(sb, (uint32_t)(min(row, rmax) * (D * 2) + 16 * pc), slot + 1024u * i);
        }
    };
    float tr[NT];                                     // score (position lane + 64 i, head h) at GH i + h
    auto tload = [&](int s) {                         // the chunk that begins at step s
        const int u = s / SEG, r = s - u * SEG;
        const int l0 = (first + stride * u) / CS * kAttnSeg + r * RS;
#pragma unroll
        for (int i = 0; i < EC / 64; ++i)
#pragma unroll
            for (int h = 0; h < GH; ++h) {
                // (past L the last score again: its e is never used)
                const int l = min(l0 + lane + 64 * i, L - 1);
                tr[GH * i + h] = tb[(int64_t)(h < G ? h : G - 1) * a.Lmax + l];
            }
    };
#pragma unroll
    for (int s = 0; s < NS - 1; ++s)
        if (s < S) issue(s);
    float m[GH];
    row_max(m);
    if (S > 0) tload(0);
    float n0[NC][GH], n1[NC][GH], ssum = 0.0f;
#pragma unroll 1
    for (int s = 0; s < S; ++s) {
        const int u = s / SEG, r = s - u * SEG;
        const int unit = first + stride * u;
        const int j = unit / CS, part = unit % CS;
        const int rows = min(kAttnSeg, L - j * kAttnSeg);
        if (r % SVC == 0) {
            attn_lds_wait();                          // the previous chunk's reads are done
#pragma unroll
            for (int i = 0; i < EC / 64; ++i)
#pragma unroll
                for (int h = 0; h < GH; ++h) es[(lane + 64 * i) * GP + h] = exp1_select(tr[GH * i + h] - m[h]);
            // the next chunk's scores: of this unit if it has more rows, else of the next unit
            const int next = (r + SVC) * RS < rows ? s + SVC : (u + 1) * SEG;
            if (next < S) tload(next);
            if (r == 0) {
#pragma unroll
                for (int k = 0; k < NC; ++k)
#pragma unroll
                    for (int h = 0; h < GH; ++h) n0[k][h] = n1[k][h] = 0.0f;
                ssum = 0.0f;
            }
        }
        if (NS > 2 && s + NS - 2 < S) attn_vm_wait<(NS - 2) * NI>();
        else attn_vm_wait<0>();
        attn_lds_wait();
        if (s + NS - 1 < S) issue(s + NS - 1);
        const uint16_t* vw = reinterpret_cast<const uint16_t*>(ring + s % NS * 4096);
        const float* er = es + (r % SVC) * (RS * GP);
        const float* eo = er + (lane < GH ? lane : 0);
        auto row_step = [&](int l) {
            float ev[GH];
#pragma unroll
            for (int h = 0; h < GH; ++h) ev[h] = er[l * GP + h];
            if constexpr (PPL == 0) {
                const float v1 = __uint_as_float((uint32_t)vw[l * DH + lane] << 16);
#pragma unroll
                for (int h = 0; h < GH; ++h) n0[0][h] = __builtin_fmaf(ev[h], v1, n0[0][h]);
            } else {
#pragma unroll
                for (int k = 0; k < PPL; ++k) {
                    const uint32_t v2 = *reinterpret_cast<const uint32_t*>(vw + l * DH + 128 * k + 2 * lane);
                    const float vlo = __uint_as_float(v2 << 16), vhi = __uint_as_float(v2 & 0xffff0000u);
#pragma unroll
                    for (int h = 0; h < GH; ++h) {
                        n0[k][h] = __builtin_fmaf(ev[h], vlo, n0[k][h]);
                        n1[k][h] = __builtin_fmaf(ev[h], vhi, n1[k][h]);
                    }
                }
            }
            ssum = ssum + eo[l * GP];
        };
        const int nrow = min(RS, rows - r * RS);
        if (nrow == RS) {
#pragma unroll 8
            for (int l = 0; l < RS; ++l) row_step(l);
        } else {
            for (int l = 0; l < nrow; ++l) row_step(l);
        }
        if (r * RS + RS >= rows) {                    // the unit's last step
#pragma unroll
            for (int h = 0; h < GH; ++h) {
                if (h >= G) break;
                float* nb = a.npart + ((h0 + h) * a.J + j) * D + part * DH;
                if constexpr (PPL == 0) {
                    nb[lane] = n0[0][h];
                } else {
#pragma unroll
                    for (int k = 0; k < PPL; ++k)
                        *reinterpret_cast<float2*>(nb + 128 * k + 2 * lane) = make_float2(n0[k][h], n1[k][h]);
                }
            }
            if (lane < G && part == 0) a.spart[(h0 + lane) * a.J + j] = ssum;
        }
    }
}

// out of head h0 + h, column d: the ascending folds of its Jb segment partials and the division.
template <int BATCH>
__device__ __forceinline__ void fold_out(const AttnArgs& a, int64_t bh, int d, int D, int Jb) {
    const float* sp = a.spart + bh * a.J;
    const float* np = a.npart + bh * a.J * D + d;
    float S = 0.0f, N = 0.0f;
    int jj = 0;
    auto batch = [&](auto nb) {
        constexpr int NB = decltype(nb)::value;
        for (; jj + NB <= Jb; jj += NB) {             // loads issued in groups, additions in order
            float sv[NB], nv[NB];
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                sv[i] = sp[jj + i];
                nv[i] = np[(int64_t)(jj + i) * D];
            }
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                S = (jj + i == 0) ? sv[i] : S + sv[i];
                N = (jj + i == 0) ? nv[i] : N + nv[i];
            }
        }
    };
    if constexpr (BATCH > 8) batch(std::integral_constant<int, BATCH>{});
    batch(std::integral_constant<int, 8>{});
    for (; jj < Jb; ++jj) {
        S = (jj == 0) ? sp[0] : S + sp[jj];
        N = (jj == 0) ? np[0] : N + np[(int64_t)jj * D];
    }
    a.out[bh * D + d] = N / S;
}

// 3'. the same partials with one wave per (segment, value columns part); each takes the group's row maxima from the
// segment maxima itself (exact, so no launch of the maximum kernel), or from that kernel (MAXIMA: a
// build of its own; as an argument it cost the other one 0.5 us of 23).  One unit per workgroup (more only beyond the
// largest grid): the waves of a CU are then at different points of their units, and a short sequence's
// waves leave at once.
template <int GH, int D, int CS, int RINGB, int EC, bool MAXIMA>
__global__ void __launch_bounds__(64) attn_values_kernel(AttnArgs a) {
    constexpr int GP = attn_lanes(GH);
    __shared__ __attribute__((aligned(16))) uint8_t ring[RINGB];
    __shared__ __attribute__((aligned(16))) float es[EC * GP];
    const int lane = threadIdx.x;
    const int G = (int)(a.H / a.Hkv);
    const uint32_t units = (uint32_t)(a.B * a.Hkv * a.J) * CS;
    for (uint32_t it = blockIdx.x; it < units; it += gridDim.x) {
        const Item w = item_of(a, (int)(it / CS));
        if (w.rows <= 0) continue;
        const int b = __builtin_amdgcn_readfirstlane(w.b), g = __builtin_amdgcn_readfirstlane(w.g);
        const int j = __builtin_amdgcn_readfirstlane(w.j), L = __builtin_amdgcn_readfirstlane(w.L);
        const int Jb = (L + kAttnSeg - 1) / kAttnSeg;
        value_pass<GH, ValueSteps<GP, D, CS, RINGB, EC>, GP, D, CS>(a, b, g, G, L, Jb, j * CS + (int)(it % CS), Jb * CS, ring, es, [&](float (&m)[GH]) {
            if constexpr (MAXIMA) {
#pragma unroll
                for (int h = 0; h < GH; ++h) m[h] = a.mmax[(int64_t)b * a.H + (int64_t)g * G + (h < G ? h : G - 1)];
            } else {
                const float* sm = a.segmax + ((int64_t)b * a.H + (int64_t)g * G) * a.J;
#pragma unroll
                for (int h = 0; h < GH; ++h) m[h] = -__builtin_inff();
                for (int j0 = lane; j0 < Jb; j0 += 64)
#pragma unroll
                    for (int h = 0; h < GH; ++h)
                        m[h] = __builtin_fmaxf(m[h], sm[(int64_t)(h < G ? h : G - 1) * a.J + j0]);
#pragma unroll
                for (int sh = 32; sh > 0; sh >>= 1)
#pragma unroll
                    for (int h = 0; h < GH; ++h) m[h] = __builtin_fmaxf(m[h], __shfl_xor(m[h], sh, 64));
            }
        });
        attn_lds_wait();                              // before the next unit's rows arrive
    }
}

// The whole call for one (sequence, kv head) in one workgroup of eight waves, with barriers in place of launches.
template <int GP, int D, int CS>
__global__ void __launch_bounds__(kAttnFusedThreads, 2) attn_fused_kernel(AttnArgs a) {
    using KS = KeySteps<GP, D>;
    using VS = ValueSteps<GP, D, CS>;
    constexpr int RING = KS::RING > VS::RING ? KS::RING : VS::RING;
    __shared__ __attribute__((aligned(16))) uint8_t ring[8][RING];
    __shared__ __attribute__((aligned(16))) float es[8][VS::EC * GP];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int Hkv = (int)a.Hkv, G = (int)(a.H / a.Hkv);
    const int b = __builtin_amdgcn_readfirstlane((int)blockIdx.x / Hkv);
    const int g = __builtin_amdgcn_readfirstlane((int)blockIdx.x - b * Hkv);
    const int L = clamp_len(a.lens, b, a.Lmax);
    const int Jb = (L + kAttnSeg - 1) / kAttnSeg;
    const int nunits = (L + KS::UNIT - 1) / KS::UNIT;
    float mymax = key_pass<GP, D>(a, b, g, G, L, wave, 8, wave < nunits ? (nunits - 1 - wave) / 8 + 1 : 0, ring[wave]);
    value_pass<GP, VS, GP, D, CS>(a, b, g, G, L, Jb, wave, 8, ring[wave], es[wave], [&](float (&m)[GP]) {
        // the maxima over the lanes of each head, then over the waves (through the e region, free until then)
        float v = mymax;
#pragma unroll
        for (int sh = 32; sh >= GP; sh >>= 1) v = __builtin_fmaxf(v, __shfl_xor(v, sh, 64));
        if (lane < GP) es[wave][lane] = v;
        __syncthreads();
#pragma unroll
        for (int h = 0; h < GP; ++h) {
            m[h] = es[0][h];
#pragma unroll
            for (int w = 1; w < 8; ++w) m[h] = __builtin_fmaxf(m[h], es[w][h]);
        }
        __syncthreads();
    });
    attn_vm_wait<0>();
    __syncthreads();
    for (int o = tid; o < G * D; o += 512) {
        const int h = o / D;
        fold_out<8>(a, (int64_t)b * a.H + (int64_t)g * G + h, o - h * D, D, Jb);
    }
}

// 4. out = N / S after the ascending folds of the segment partials.  Workgroup (b, h),
// thread d.
__global__ void __launch_bounds__(256) attn_fold_kernel(AttnArgs a) {
    const int64_t bh = blockIdx.x;
    const int L = clamp_len(a.lens, bh / a.H, a.Lmax);
    const int Jb = (L + kAttnSeg - 1) / kAttnSeg;
    for (int d = threadIdx.x; d < a.D; d += blockDim.x) fold_out<32>(a, bh, d, (int)a.D, Jb);
}

// Workgroups each kernel keeps resident per CU: LDS-limited (160 KB per CU).
constexpr int64_t kLdsPerCU = 160 * 1024;

// Persistent grids: as many workgroups as the LDS of the device keeps resident.
template <typename K1, typename K3>
hipError_t launch_pair(K1 k1, int64_t lds1, K3 k3, int64_t lds3, const AttnArgs& a, int cus, hipStream_t stream) {
    const int64_t items = a.B * a.Hkv * a.J;
    const int64_t g1 = items < (kLdsPerCU / lds1) * cus ? items : (kLdsPerCU / lds1) * cus;
    const int64_t g3 = items < (kLdsPerCU / lds3) * cus ? items : (kLdsPerCU / lds3) * cus;
    hipLaunchKernelGGL(k1, dim3((unsigned)g1), dim3(256), 0, stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    e = launch_max(a, stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k3, dim3((unsigned)g3), dim3(256), 0, stream, a);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(attn_fold_kernel, dim3((unsigned)(a.B * a.H)), dim3(256), 0, stream, a);
    return hipGetLastError();
}

// Fixed head dims (64, 128, 256), by attn_route.
//
// Scores: 64-column key steps (32 KB tiles, four workgroups per CU); with eight query heads per kv head the
// two-positions-per-thread kernel (32-column steps, 128 threads, about 20 KB of LDS; measured 111 -> 90 us
// for the scores of a 32 x 64-head, 4096-position batch, and 0-22 % slower than the 64-column kernel with six or fewer heads).
template <int G, int D>
hipError_t launch_fixed(const AttnArgs& a, int cus, hipStream_t stream) {
    // heads of a values wave: five and six their own number, three and seven the next power of two (their e are then
    // read as whole vectors: 32 x 8 pairs of 4096 positions at D = 64 with three heads 58 us, 62 with chains for three)
    constexpr int GP = attn_lanes(G), GH = G == 5 || G == 6 ? G : GP;
    const AttnRoute route = attn_route(a.B, a.Hkv, a.Lmax, D, G, cus);
    // bytes in flight of a whole-row wave and of one with half the columns, and positions whose e it holds (more per wave
    // costs waves: slower but for the heaviest rows)
    constexpr int RING1 = GP == 8 ? 12288 : 8192, RING2 = GP == 8 || (D == 256 && GP < 4) ? 12288 : 8192;
    constexpr int EC = GP >= 4 ? 128 : 256;
    const int64_t items = a.B * a.Hkv * a.J;
    if constexpr (D * GP <= 512) {
        if (route.fused) {
            constexpr int CS = D == 64 ? 1 : 2;
            hipLaunchKernelGGL((attn_fused_kernel<GP, D, CS>), dim3((unsigned)(a.B * a.Hkv)), dim3(kAttnFusedThreads), 0,
                               stream, a);
            return hipGetLastError();
        }
    }
    if constexpr (G == 8) {
        const int64_t lds1 = (int64_t)kAttnSeg * (32 + 8) * 2 + 8 * G;
        const int64_t g1 = items < (kLdsPerCU / lds1) * cus ? items : (kLdsPerCU / lds1) * cus;
        hipLaunchKernelGGL((attn_scores2_kernel<G, D>), dim3((unsigned)g1), dim3(128), 0, stream, a);
    } else {
        const int64_t lds1 = (int64_t)kAttnSeg * (64 + 8) * 2 + 16 * G;
        const int64_t g1 = items < (kLdsPerCU / lds1) * cus ? items : (kLdsPerCU / lds1) * cus;
        hipLaunchKernelGGL((attn_scores_kernel<G, 64, D / 64, true>), dim3((unsigned)g1), dim3(256), 0, stream, a);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (route.group) {
        e = launch_max(a, stream);
        if (e != hipSuccess) return e;
        if constexpr (D == 64 && G >= 3)
            hipLaunchKernelGGL((attn_partials_kernel<G, D, true>), dim3((unsigned)items), dim3(256), 0, stream, a);
    } else {
        if (route.maxima) {
            e = launch_max(a, stream);
            if (e != hipSuccess) return e;
        }
        const int64_t units = items * (route.split ? 2 : 1);
        const dim3 grid((unsigned)(units < (1 << 24) ? units : (1 << 24)));
        if constexpr (D > 64) {
            if (route.split)
                hipLaunchKernelGGL((attn_values_kernel<GH, D, 2, RING2, EC, false>), grid, dim3(64), 0, stream, a);
        }
        auto whole = [&](auto ring, auto ec) {
            if (route.maxima)
                hipLaunchKernelGGL((attn_values_kernel<GH, D, 1, decltype(ring)::value, decltype(ec)::value, true>), grid,
                                   dim3(64), 0, stream, a);
            else
                hipLaunchKernelGGL((attn_values_kernel<GH, D, 1, decltype(ring)::value, decltype(ec)::value, false>), grid,
                                   dim3(64), 0, stream, a);
        };
        if constexpr (D > 64 && GP == 8) {
            if (route.light) whole(std::integral_constant<int, 8192>{}, std::integral_constant<int, 64>{});
        }
        if (!route.split && !route.light) {
            if constexpr (!(D == 256 && GP == 8))
                whole(std::integral_constant<int, RING1>{}, std::integral_constant<int, EC>{});
        }
    }
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(attn_fold_kernel, dim3((unsigned)(a.B * a.H)), dim3(256), 0, stream, a);
    return hipGetLastError();
}

template <int G, int DM>
hipError_t launch_any(const AttnArgs& a, int cus, hipStream_t stream) {
    const int64_t lds1 = (int64_t)kAttnSeg * (DM + 8) * 2 + 16 * G;
    const int64_t lds3 = (int64_t)G * kAttnSeg * 4 + (int64_t)kAttnSeg * (DM + 8) * 2;
    return launch_pair(attn_scores_kernel<G, DM, 1, false>, lds1, attn_partials_kernel<G, DM, false>, lds3,
                       a, cus, stream);
}

template <int G>
hipError_t launch_dm(const AttnArgs& a, int cus, hipStream_t stream) {
    if (a.D == 64) return launch_fixed<G, 64>(a, cus, stream);
    if (a.D == 128) return launch_fixed<G, 128>(a, cus, stream);
    if (a.D == 256) return launch_fixed<G, 256>(a, cus, stream);
    if (a.D <= 64) return launch_any<G, 64>(a, cus, stream);
    if (a.D <= 128) return launch_any<G, 128>(a, cus, stream);
    return launch_any<G, 256>(a, cus, stream);
}

}  // namespace

hipError_t launch_attn(const AttnArgs& a, int cus, hipStream_t stream) {
    if (cus < 1) cus = 1;
    if (a.D < 8 || a.D > 256 || a.D % 8 != 0 || a.Hkv < 1 || a.H % a.Hkv != 0) return hipErrorInvalidValue;
    switch (a.H / a.Hkv) {
        case 1: return launch_dm<1>(a, cus, stream);
        case 2: return launch_dm<2>(a, cus, stream);
        case 3: return launch_dm<3>(a, cus, stream);
        case 4: return launch_dm<4>(a, cus, stream);
        case 5: return launch_dm<5>(a, cus, stream);
        case 6: return launch_dm<6>(a, cus, stream);
        case 7: return launch_dm<7>(a, cus, stream);
        case 8: return launch_dm<8>(a, cus, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace rg
