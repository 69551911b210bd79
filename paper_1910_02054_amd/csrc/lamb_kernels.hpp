// lamb_kernels.hpp -- gfx950 kernels of the LAMB shard step.
//
// LAMB (You et al., layer-wise adaptive large-batch optimization; one of the
// adaptive optimizers ZeRO's related work lists as made affordable by
// partitioning optimizer state) keeps Adam's fp32 moments but scales each
// layer's update direction u by the trust ratio phi(||theta||)/||u||.  The
// layer norms couple every element of a layer, so the step takes two
// streaming passes after the gradient statistics:
//   k_lamb_moments  reads g16, theta, m, v; writes m, v; one fp64 partial
//                   (sum theta^2, sum u^2) per work item (22 bytes/element).
//   k_lamb_sums     fixed-order two-level sum of each layer's partials.
//   k_lamb_apply    reads theta, m, v; recomputes u from the stored moments
//                   (the same fp32 operations, so the same bits); writes
//                   theta - step*u and its fp16 copy (18 bytes/element).
// A work item is a tile's piece inside one layer: the host cuts the shard's
// tiles at the layer boundaries.  Each workgroup owns one tile and computes its
// addresses from its index alone; it reads the tile's items (almost always
// one) only to attribute its partial sums and step sizes to layers.
#pragma once

#include "shard_kernels.hpp"

namespace zs {

// Elements [start, next item's start) of layer `layer`.  The list ends with a
// sentinel item whose start is n.
struct alignas(16) LambItem {
    int64_t start;
    int32_t layer;
    int32_t unused;
};

// Sum of theta^2 and sum of u^2 (fp64) of one work item or one layer.
struct alignas(16) LayerSums {
    double wsq;
    double usq;
};

// The layer's fp32 step size lr * phi(||theta||) / ||u|| (1 for the ratio when
// either norm is zero), computed in double and rounded once.
__device__ __forceinline__ float lamb_step_size(LayerSums s, double lr, double phi_lo, double phi_hi) {
    double trust = 1.0;
    if (s.wsq > 0.0 && s.usq > 0.0) {
        double wn = __builtin_sqrt(s.wsq);
        if (wn < phi_lo)
            wn = phi_lo;
        if (wn > phi_hi)
            wn = phi_hi;
        trust = wn / __builtin_sqrt(s.usq);
    }
    return (float)(lr * trust);
}

// Fixed-order workgroup sum of two doubles per thread; thread 0 receives the
// totals.  Ends with a barrier so that a following call may reuse the LDS.
template <int BLOCK>
__device__ __forceinline__ void block_sum2(double& a, double& b) {
    a = wave_sum(a);
    b = wave_sum(b);
    if constexpr (BLOCK > 64) {
        __shared__ double lds[2][BLOCK / 64];
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        if (lane == 0) {
            lds[0][wave] = a;
            lds[1][wave] = b;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            double sa = 0.0, sb = 0.0;
#pragma unroll
            for (int w = 0; w < BLOCK / 64; ++w) {
                sa += lds[0][w];
                sb += lds[1][w];
            }
            a = sa;
            b = sb;
        }
        __syncthreads();
    }
}

// Tiles of the shard: with head h (0..kMaxHead) the 4-element vectors begin at
// indices congruent to h mod 4; tile 0 is [0, h) when h > 0, and the other
// tiles are T = 4*BLOCK*U elements long, from h on.  Returns the tile's first
// vector's element index (which lies before the shard when tile 0 begins with
// part of a vector) and the tile's element range [ts, te).
template <int BLOCK, int U>
__device__ __forceinline__ int64_t tile_range(int64_t b, int64_t head, int64_t n, int64_t* ts, int64_t* te) {
    constexpr int64_t T = 4 * (int64_t)BLOCK * U;
    const int64_t hs = head > 0 ? 1 : 0;
    if (b < hs) {
        *ts = 0;
        *te = head < n ? head : n;
        return head - (head + 3) / 4 * 4;
    }
    const int64_t base = head + (b - hs) * T;
    *ts = base;
    *te = base + T < n ? base + T : n;
    return base;
}

// ---------------------------------------------------------------------------
// Work items: [0, n) cut at the tile boundaries and at the layer boundaries
// off[0..n_seg].  One thread per tile: its items come after one item per earlier
// tile and per earlier layer that begins inside a tile (inner[s]: how many of the
// layers 1..s do), and are the tile's start and the layers that begin inside it.
// The thread after the last tile writes the end sentinels.  Runs once per plan
// and alignment: the binary search over the layers is all that it waits for.
// ---------------------------------------------------------------------------
constexpr int kItemsBlock = 256;

[[maybe_unused]] static __global__ __launch_bounds__(kItemsBlock) void k_lamb_items(
    const int64_t* __restrict__ off, const int64_t* __restrict__ inner, int32_t n_seg, int64_t head, int64_t ntiles,
    int64_t tile, LambItem* __restrict__ items, int64_t* __restrict__ tile_first) {
    const int64_t b = (int64_t)blockIdx.x * kItemsBlock + threadIdx.x;
    if (b > ntiles)
        return;
    const int64_t n = off[n_seg];
    if (b == ntiles) {
        const int64_t k = ntiles + inner[n_seg - 1];
        tile_first[b] = k;
        items[k] = LambItem{n, -1, 0};
        return;
    }
    const int64_t hs = head > 0 ? 1 : 0;
    const int64_t ts = b < hs ? 0 : head + (b - hs) * tile;
    const int64_t end = b < hs ? head : ts + tile, te = end < n ? end : n;
    int32_t s = 0, hi = n_seg;  // off[s] <= ts < off[hi]
    while (hi - s > 1) {
        const int32_t mid = s + (hi - s) / 2;
        if (off[mid] <= ts)
            s = mid;
        else
            hi = mid;
    }
    int64_t k = b + inner[s];
    tile_first[b] = k;
    items[k] = LambItem{ts, s, 0};
    for (++s; s < n_seg && off[s] < te; ++s)
        items[++k] = LambItem{off[s], s, 0};
}

// ---------------------------------------------------------------------------
// Moments pass.  Workgroup b (grid-strided over the tiles; with XCD, remapped so
// that each XCD walks a contiguous run of tiles and the tiles' descriptors,
// which neighbouring tiles share cache lines of, stay in one L2) owns tile b: thread
// t covers the U vectors base + 4*(t + u*BLOCK) .. +3.  The data addresses
// depend on b only, so the loads are issued before the tile's work items
// (its layer pieces, [tile_first[b], tile_first[b+1]) of the item list) are
// read; the items are needed only to attribute each element's theta^2 and u^2
// to its layer piece.  A vector inside the tile is one 16-byte fp32 access per
// array and one 8-byte fp16 access: `head` brings the master array's vectors
// to cache lines, the other arrays' may be unaligned (as k_adam_vec's);
// the partial vectors at the shard's ends go element by element.
// ---------------------------------------------------------------------------
template <int BLOCK, int U, bool NTL, bool NTS, bool XCD, typename SRC>
__global__ __launch_bounds__(BLOCK) void k_lamb_moments(const uint16_t* __restrict__ g, const float* __restrict__ th,
                                                        float* __restrict__ m, float* __restrict__ v,
                                                        const LambItem* __restrict__ items,
                                                        const int64_t* __restrict__ tile_first, int64_t ntiles,
                                                        int64_t n, int64_t head, SRC src,
                                                        LayerSums* __restrict__ part) {
    float mult;
    AdamConst c;
    if (!src.get(mult, c))
        return;
    for (int64_t b = logical_block<XCD>(); b < ntiles; b += gridDim.x) {
        int64_t ts, te;
        const int64_t base = tile_range<BLOCK, U>(b, head, n, &ts, &te);
        double w2[U][4], u2[U][4];
        int64_t e0s[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t e0 = base + 4 * ((int64_t)threadIdx.x + (int64_t)u * BLOCK);
            e0s[u] = e0;
            if (e0 >= ts && e0 + 4 <= te) {
                const u32x2 gq = ld4<NTL>(g + e0);
                const f32x4 tq = ld4<NTL>(th + e0);
                f32x4 mq = ld4<NTL>(m + e0);
                f32x4 vq = ld4<NTL>(v + e0);
                const uint32_t gw[4] = {gq.x & 0xFFFFu, gq.x >> 16, gq.y & 0xFFFFu, gq.y >> 16};
                const float t4[4] = {tq.x, tq.y, tq.z, tq.w};
                float m4[4] = {mq.x, mq.y, mq.z, mq.w};
                float v4[4] = {vq.x, vq.y, vq.z, vq.w};
                float d4[4];
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    moments_elem(gw[j], mult, m4[j], v4[j], c);
                direction4(m4, v4, c, d4);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const double ud = (double)decayed(d4[j], t4[j], c);
                    const double td = (double)t4[j];
                    w2[u][j] = td * td;
                    u2[u][j] = ud * ud;
                }
                st4<NTS>(f32x4{m4[0], m4[1], m4[2], m4[3]}, m + e0);
                st4<NTS>(f32x4{v4[0], v4[1], v4[2], v4[3]}, v + e0);
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int64_t i = e0 + j;
                    w2[u][j] = 0.0;
                    u2[u][j] = 0.0;
                    if (i >= ts && i < te) {
                        float mm = m[i], vv = v[i];
                        const float t = th[i];
                        moments_elem(g[i], mult, mm, vv, c);
                        const double ud = (double)decayed(direction(mm, vv, c), t, c);
                        const double td = (double)t;
                        w2[u][j] = td * td;
                        u2[u][j] = ud * ud;
                        m[i] = mm;
                        v[i] = vv;
                    }
                }
            }
        }
        // one partial per layer piece of the tile (almost always one piece)
        const int64_t f = tile_first[b], l = tile_first[b + 1];
        for (int64_t k = f; k < l; ++k) {
            const int64_t s0 = items[k].start, s1 = items[k + 1].start;
            double aw = 0.0, au = 0.0;
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int64_t i = e0s[u] + j;
                    if (i >= s0 && i < s1) {
                        aw += w2[u][j];
                        au += u2[u][j];
                    }
                }
            block_sum2<BLOCK>(aw, au);
            if (threadIdx.x == 0)
                part[k] = LayerSums{aw, au};
        }
    }
}

// ---------------------------------------------------------------------------
// Layer sums, two levels in a fixed order.  Workgroup c adds the partials of
// item chunk c, items [chunk[c], chunk[c+1]) (a chunk never spans two layers);
// the workgroups of a layer bring their chunks' sums together through two slots
// each (close_slots: neither sum is negative) and the one that closes them, the
// last as a rule, writes the layer's.  The second level in a kernel of its own
// cost 4.7 us a step.
// ---------------------------------------------------------------------------
constexpr int kChunkBlock = 256;
constexpr int kChunkItems = 1024;   // items per chunk (4 per thread)

__global__ __launch_bounds__(kChunkBlock) void k_lamb_sums(const LayerSums* __restrict__ part,
                                                           const int64_t* __restrict__ chunk,
                                                           const int32_t* __restrict__ chunk_layer,
                                                           const int64_t* __restrict__ chunk_first,
                                                           uint64_t* __restrict__ slots, LayerSums* __restrict__ sums,
                                                           const Result* __restrict__ res) {
    if (res && res->skip)
        return;
    const int64_t cb = blockIdx.x;
    const int64_t a = chunk[cb], e = chunk[cb + 1];
    const int32_t s = chunk_layer[cb];  // read ahead of the sums: two dependent reads
    const int64_t first = chunk_first[s];
    const int count = (int)(chunk_first[s + 1] - first);
    double w = 0.0, u = 0.0;
    for (int64_t i = a + threadIdx.x; i < e; i += kChunkBlock) {
        const LayerSums p = part[i];
        w += p.wsq;
        u += p.usq;
    }
    block_sum2<kChunkBlock>(w, u);
    if (threadIdx.x >= 64)
        return;
    if (count > 1) {
        const double mine[2] = {w, u};
        double share[2];
        if (!close_slots<2, true>(slots + 2 * first, count, (int)(cb - first), mine, share))
            return;
        w = wave_sum(share[0]);
        u = wave_sum(share[1]);
    }
    if (threadIdx.x == 0)
        sums[s] = LayerSums{w, u};
}

// ---------------------------------------------------------------------------
// Apply pass: same tile walk as the moments pass; each element moves by its
// layer piece's step size (theta <- theta - step*u) and gets its fp16 copy.
// ---------------------------------------------------------------------------
template <int BLOCK, int U, bool NTL, bool NTS, bool XCD, typename SRC>
__global__ __launch_bounds__(BLOCK) void k_lamb_apply(float* __restrict__ th, const float* __restrict__ m,
                                                      const float* __restrict__ v, uint16_t* __restrict__ p,
                                                      const LambItem* __restrict__ items,
                                                      const int64_t* __restrict__ tile_first, int64_t ntiles,
                                                      int64_t n, int64_t head, const LayerSums* __restrict__ sums,
                                                      SRC src, double lr, double phi_lo, double phi_hi) {
#pragma clang fp contract(off)
    float mult;
    AdamConst c;
    if (!src.get(mult, c))
        return;
    for (int64_t b = logical_block<XCD>(); b < ntiles; b += gridDim.x) {
        int64_t ts, te;
        const int64_t base = tile_range<BLOCK, U>(b, head, n, &ts, &te);
        float t4[U][4], u4[U][4];
        bool full[U];
        int64_t e0s[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t e0 = base + 4 * ((int64_t)threadIdx.x + (int64_t)u * BLOCK);
            e0s[u] = e0;
            full[u] = e0 >= ts && e0 + 4 <= te;
            if (full[u]) {
                const f32x4 tq = ld4<NTL>(th + e0);
                const f32x4 mq = ld4<NTL>(m + e0);
                const f32x4 vq = ld4<NTL>(v + e0);
                const float tt[4] = {tq.x, tq.y, tq.z, tq.w};
                const float mm[4] = {mq.x, mq.y, mq.z, mq.w};
                const float vv[4] = {vq.x, vq.y, vq.z, vq.w};
                float d4[4];
                direction4(mm, vv, c, d4);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    t4[u][j] = tt[j];
                    u4[u][j] = decayed(d4[j], tt[j], c);
                }
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int64_t i = e0 + j;
                    t4[u][j] = 0.0f;
                    u4[u][j] = 0.0f;
                    if (i >= ts && i < te) {
                        t4[u][j] = th[i];
                        u4[u][j] = decayed(direction(m[i], v[i], c), t4[u][j], c);
                    }
                }
            }
        }
        // the step size of every element's layer piece (almost always one piece per tile)
        float step[U][4];
        const int64_t f = tile_first[b], l = tile_first[b + 1];
        {
            const LambItem it = items[f];
            const float s = lamb_step_size(sums[it.layer], lr, phi_lo, phi_hi);
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    step[u][j] = s;
        }
        for (int64_t k = f + 1; k < l; ++k) {
            const LambItem it = items[k];
            const float s = lamb_step_size(sums[it.layer], lr, phi_lo, phi_hi);
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (e0s[u] + j >= it.start)
                        step[u][j] = s;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t e0 = e0s[u];
            float o[4];
            uint32_t h[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                o[j] = t4[u][j] - step[u][j] * u4[u][j];
                h[j] = f32_to_f16(o[j]);
            }
            if (full[u]) {
                st4<NTS>(f32x4{o[0], o[1], o[2], o[3]}, th + e0);
                st4<NTS>(u32x2{h[0] | (h[1] << 16), h[2] | (h[3] << 16)}, p + e0);
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int64_t i = e0 + j;
                    if (i >= ts && i < te) {
                        th[i] = o[j];
                        p[i] = (uint16_t)h[j];
                    }
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Byte-mix probes of the two passes: the same arrays, tile walk (XCD-contiguous
// tiles of 4*BLOCK*U elements, one tile per workgroup), vector width and cache
// policy as k_lamb_moments (PASS 0: reads g16, theta, m, v; writes m, v) and
// k_lamb_apply (PASS 1: reads theta, m, v; writes theta, p16), with one or two
// adds per element in place of the pass's arithmetic and no work lists.  Their
// time is the achievable time of each pass's streams at its launch shape.
// Arrays 16-byte aligned (fp16 8-byte); the last partial vector is scalar.
// ---------------------------------------------------------------------------
template <int BLOCK, int U, bool NTL, bool NTS, bool XCD, int PASS>
__global__ __launch_bounds__(BLOCK) void k_probe_lamb(const uint16_t* __restrict__ g, float* __restrict__ th,
                                                      float* __restrict__ m, float* __restrict__ v,
                                                      uint16_t* __restrict__ p, int64_t ntiles, int64_t n) {
    constexpr int64_t T = 4 * (int64_t)BLOCK * U;
    for (int64_t b = logical_block<XCD>(); b < ntiles; b += gridDim.x) {
        const int64_t te = (b + 1) * T < n ? (b + 1) * T : n;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t e0 = b * T + 4 * ((int64_t)threadIdx.x + (int64_t)u * BLOCK);
            if (e0 + 4 <= te) {
                if constexpr (PASS == 0) {
                    const u32x2 gq = ld<NTL>(reinterpret_cast<const u32x2*>(g + e0));
                    const f32x4 tq = ld<NTL>(reinterpret_cast<const f32x4*>(th + e0));
                    const f32x4 mq = ld<NTL>(reinterpret_cast<const f32x4*>(m + e0));
                    const f32x4 vq = ld<NTL>(reinterpret_cast<const f32x4*>(v + e0));
                    const f32x4 gf = {f16_to_f32(gq.x & 0xFFFFu), f16_to_f32(gq.x >> 16), f16_to_f32(gq.y & 0xFFFFu),
                                      f16_to_f32(gq.y >> 16)};
                    st<NTS>(mq + gf, reinterpret_cast<f32x4*>(m + e0));
                    st<NTS>(vq + tq, reinterpret_cast<f32x4*>(v + e0));
                } else {
                    const f32x4 tq = ld<NTL>(reinterpret_cast<const f32x4*>(th + e0));
                    const f32x4 mq = ld<NTL>(reinterpret_cast<const f32x4*>(m + e0));
                    const f32x4 vq = ld<NTL>(reinterpret_cast<const f32x4*>(v + e0));
                    const f32x4 o = tq + mq + vq;
                    st<NTS>(o, reinterpret_cast<f32x4*>(th + e0));
                    st<NTS>(u32x2{f32_to_f16(o.x) | (f32_to_f16(o.y) << 16), f32_to_f16(o.z) | (f32_to_f16(o.w) << 16)},
                            reinterpret_cast<u32x2*>(p + e0));
                }
            } else {
                for (int64_t i = e0; i < te && i < e0 + 4; ++i) {
                    if constexpr (PASS == 0) {
                        m[i] = m[i] + f16_to_f32(g[i]);
                        v[i] = v[i] + th[i];
                    } else {
                        const float o = th[i] + m[i] + v[i];
                        th[i] = o;
                        p[i] = (uint16_t)f32_to_f16(o);
                    }
                }
            }
        }
    }
}

}  // namespace zs
