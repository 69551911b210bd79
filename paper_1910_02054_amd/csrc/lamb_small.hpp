// lamb_small.hpp -- the one-launch LAMB step for small shards (gfx950): gradient
// statistics, moments, layer norms and the trusted update in a single kernel.
#pragma once

#include "lamb_kernels.hpp"
#include "small_kernels.hpp"

namespace zs {

// ---------------------------------------------------------------------------
// One-launch LAMB step.  The grid, its residency and the exchange of the
// gradient sums (all workgroups, slot_wait, bounded) are k_small_step's.
// Workgroup b owns V * kLambSmallBlock consecutive vectors and each of its waves
// consecutive ones of them, so they meet few layers; the first workgroup also
// takes the head's single elements, the last one the tail's, one per thread.
//   1. Gradient sums, exchanged; theta, m and v are loaded meanwhile.
//   2. Moments (stored) and direction; theta and the direction stay in registers.
//   3. One pair of sums (theta^2, u^2) per layer piece of the workgroup, each
//      put into the piece's two slots; the workgroup then adds the slots of all
//      pieces of its own layers in a fixed order.  (Layers of one piece need no
//      exchange.)  Every workgroup has filled its gradient slot by then, so all
//      are resident, none has given up, and each fills all its pieces' slots
//      before it waits for another's: this wait ends, one exchange deep, and has
//      no limit (the moments are written by then and the total is published, so
//      there is nothing to give up to).  (A wave that waited for its
//      first piece's layer before filling its next piece's slots chained the
//      workgroups where the last of five pieces runs on into the next workgroup:
//      200 workgroups so cut took 260 us a step with its synchronisation, 26 us
//      now and with one layer.)
//   4. Step sizes and the update.
// Latency bounds it: every array is touched once (28 bytes an element, where the
// kernel sequence moves 42) behind two exchanges.  Against the kernel sequence,
// whole synchronous steps: 2000 elements 21.0 -> 14.0 us, 200K 21.2 -> 15.2, 500K
// 21.9 -> 15.9, 1M (65 layers) 23.5 -> 17.9.  256-thread workgroups, because
// at four tiles (121 registers) a quarter of the chip holds 256 of them and so
// 1M elements; the arithmetic of 16 elements a thread, one wave per SIMD, is then
// about half of the kernel's time.  That register limit is the size limit: a step on
// 1,048,576 elements of 64 layers takes 15.2 us, one on 1,048,700, in the kernel
// sequence, 21.4 (1.5M 23.3).
// ---------------------------------------------------------------------------
constexpr int kLambSmallBlock = 256;
constexpr int kLambPieces = 8;          // the most layer pieces of a workgroup
constexpr int kLambSmallItems = 1024;   // the most layer pieces of a shard
constexpr int kLambSmallWords = kSmallSlots + 2 * kLambSmallItems;  // one set of slots

static_assert(kSmallSlots <= kLambSmallBlock, "a thread reads at most one gradient slot");
static_assert(2 * kLambSmallWords * sizeof(uint64_t) == 36 * 1024, "the size that the interface states");

// Waves per SIMD that the registers of k_lamb_small<V> leave: a quarter of the
// chip then holds 256 workgroups at every V.
constexpr int lamb_small_waves(int v) { return v == 1 ? 8 : v == 2 ? 6 : 4; }

template <int V>
__global__ __launch_bounds__(kLambSmallBlock, lamb_small_waves(V)) void k_lamb_small(
    const uint16_t* __restrict__ g, float* __restrict__ th, float* __restrict__ m, float* __restrict__ v,
    uint16_t* __restrict__ p, int n, int head, int nvec, const LambItem* __restrict__ items,
    const int64_t* __restrict__ wg_first, const int64_t* __restrict__ layer_first, uint64_t* __restrict__ set,
    uint64_t* __restrict__ other, uint64_t* __restrict__ host, double loss_scale, double clip, uint32_t seq,
    AdamConst c, double lr, double phi_lo, double phi_hi) {
#pragma clang fp contract(off)
    constexpr int W = kLambSmallBlock / 64;
    __shared__ double lds[W];
    __shared__ Sum2 lds2[kSmallSlots / 64];
    __shared__ LayerSums s_piece[kLambPieces][W];
    __shared__ float s_step[kLambPieces];
    __shared__ int s_abort;
    const int b = (int)blockIdx.x;
    const int G = (int)gridDim.x;
    const int tid = (int)threadIdx.x, wave = tid >> 6, lane = tid & 63;
    // each wave owns V * 64 consecutive vectors, so it meets few of the workgroup's layers
    const int w0 = (b * W + wave) * V * 64, i0 = w0 + lane, e0 = head + 4 * i0;

    // the single element of this thread, if any
    int one = -1;
    if (b == 0 && tid < head)
        one = tid;
    if (b == G - 1 && tid >= kMaxHead && head + 4 * nvec + (tid - kMaxHead) < n)
        one = head + 4 * nvec + (tid - kMaxHead);

    // 1. gradient sums and state
    u32x2 gq[V];
#pragma unroll
    for (int k = 0; k < V; ++k) {
        const int i = i0 + k * 64;
        gq[k] = i < nvec ? ld4<true>(g + head + 4 * i) : u32x2{0u, 0u};
    }
    const uint32_t g1 = one >= 0 ? g[one] : 0u;
    double a0 = sq1(g1), a1 = 0.0;
#pragma unroll
    for (int k = 0; k < V; ++k) {
        a0 = acc_sq2(gq[k].x, a0);
        a1 = acc_sq2(gq[k].y, a1);
    }
    if (tid == 0)
        s_abort = 0;
    double tot = small_block_total<kLambSmallBlock>(a0 + a1, lds);
    if (G > 1 && tid == 0)
        slot_fill(set + b, slot_word(tot));
    f32x4 tq[V] = {}, mq[V] = {}, vq[V] = {};
#pragma unroll
    for (int k = 0; k < V; ++k) {
        const int i = i0 + k * 64;
        if (i < nvec) {
            const int e = head + 4 * i;
            tq[k] = ld4<true>(th + e);
            mq[k] = ld4<true>(m + e);
            vq[k] = ld4<true>(v + e);
        }
    }
    float t1 = 0.0f, m1 = 0.0f, v1 = 0.0f;
    if (one >= 0) {
        t1 = th[one];
        m1 = m[one];
        v1 = v[one];
    }
    for (int k = b * kLambSmallBlock + tid; k < kLambSmallWords; k += G * kLambSmallBlock)
        astore(other + k, 0);
    if (G > 1) {
        tot = small_exchange(set, G, lds2, &s_abort);
        if (s_abort)
            return;
    }
    if (b == 0 && tid == 0)
        publish_sum(host, tot, seq);
    const Result r = make_result(tot, loss_scale, clip, seq);
    if (r.skip)
        return;

    // 2. moments and direction (mq becomes u)
#pragma unroll
    for (int k = 0; k < V; ++k) {
        const int i = i0 + k * 64;
        if (i < nvec) {
            const uint32_t gw[4] = {gq[k].x & 0xFFFFu, gq[k].x >> 16, gq[k].y & 0xFFFFu, gq[k].y >> 16};
            float mm[4], vv[4], d4[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                mm[j] = mq[k][j];
                vv[j] = vq[k][j];
                moments_elem(gw[j], r.mult, mm[j], vv[j], c);
            }
            const int e = head + 4 * i;
            st4<true>(f32x4{mm[0], mm[1], mm[2], mm[3]}, m + e);
            st4<true>(f32x4{vv[0], vv[1], vv[2], vv[3]}, v + e);
            direction4(mm, vv, c, d4);
#pragma unroll
            for (int j = 0; j < 4; ++j)
                mq[k][j] = decayed(d4[j], tq[k][j], c);
        }
        __builtin_amdgcn_sched_barrier(0);  // one vector's arithmetic at a time: registers
    }
    if (one >= 0) {
        moments_elem(g1, r.mult, m1, v1, c);
        m[one] = m1;
        v[one] = v1;
        m1 = decayed(direction(m1, v1, c), t1, c);
    }

    // 3. layer sums of the workgroup's pieces
    const int f = (int)wg_first[b], pieces = (int)wg_first[b + 1] - f;
    for (int q = 0; q < pieces; ++q) {
        const int s0 = (int)items[f + q].start, s1 = (int)items[f + q + 1].start;
        const int d0 = s0 - e0, d1 = s1 - e0;
        const bool single = one >= s0 && one < s1;
        double w = 0.0, u = 0.0;
        if (__any(single) || (s0 < head + 4 * (w0 + V * 64) && s1 > head + 4 * w0)) {
#pragma unroll
            for (int k = 0; k < V; ++k) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int d = 4 * k * 64 + j;
                    const bool in = d >= d0 && d < d1;  // a thread without a vector holds zeros
                    const double td = in ? (double)tq[k][j] : 0.0, ud = in ? (double)mq[k][j] : 0.0;
                    w += td * td;
                    u += ud * ud;
                }
            }
            if (single) {
                w += (double)t1 * (double)t1;
                u += (double)m1 * (double)m1;
            }
            w = wave_sum(w);
            u = wave_sum(u);
        }
        if (lane == 0)
            s_piece[q][wave] = LayerSums{w, u};
    }
    __syncthreads();
    uint64_t* const pair = set + kSmallSlots;
    // every slot of the workgroup's pieces is filled before the first wait, so no wait depends on another
    constexpr int Q = (kLambPieces + W - 1) / W;  // the most pieces of a wave
    LayerSums own[Q];
    int first[Q], end[Q];
#pragma unroll
    for (int j = 0; j < Q; ++j) {
        const int q = wave + j * W;
        own[j] = LayerSums{0.0, 0.0};
        first[j] = end[j] = 0;
        if (q < pieces) {
#pragma unroll
            for (int x = 0; x < W; ++x) {
                own[j].wsq += s_piece[q][x].wsq;
                own[j].usq += s_piece[q][x].usq;
            }
            const int32_t layer = items[f + q].layer;
            first[j] = (int)layer_first[layer];
            end[j] = (int)layer_first[layer + 1];
            if (end[j] - first[j] > 1 && lane == 0) {
                (void)slot_fill(pair + 2 * (f + q), slot_word(own[j].wsq));
                (void)slot_fill(pair + 2 * (f + q) + 1, slot_word(own[j].usq));
            }
        }
    }
#pragma unroll
    for (int j = 0; j < Q; ++j) {
        const int q = wave + j * W;
        if (end[j] - first[j] > 1) {
            double w = 0.0, u = 0.0;
            for (int i = first[j] + lane; i < end[j]; i += 64) {
                w += slot_sum(slot_read(pair + 2 * i));
                u += slot_sum(slot_read(pair + 2 * i + 1));
            }
            own[j].wsq = wave_sum(w);
            own[j].usq = wave_sum(u);
        }
        if (q < pieces && lane == 0)
            s_step[q] = lamb_step_size(own[j], lr, phi_lo, phi_hi);
    }
    __syncthreads();

    // 4. the update
#pragma unroll
    for (int k = 0; k < V; ++k) {
        if (i0 + k * 64 < nvec) {
            const int e = e0 + 4 * k * 64;
            float step[4];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                step[j] = s_step[0];
            for (int q = 1; q < pieces; ++q) {
                const int s0 = (int)items[f + q].start;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (e + j >= s0)
                        step[j] = s_step[q];
            }
            uint32_t h[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                tq[k][j] = tq[k][j] - step[j] * mq[k][j];
                h[j] = f32_to_f16(tq[k][j]);
            }
            st4<true>(tq[k], th + e);
            st4<true>(u32x2{h[0] | (h[1] << 16), h[2] | (h[3] << 16)}, p + e);
        }
    }
    if (one >= 0) {
        float step = s_step[0];
        for (int q = 1; q < pieces; ++q)
            if (one >= items[f + q].start)
                step = s_step[q];
        t1 = t1 - step * m1;
        th[one] = t1;
        p[one] = (uint16_t)f32_to_f16(t1);
    }
}

}  // namespace zs
