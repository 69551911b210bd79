// small_kernels.hpp -- the one-launch small-shard step (gfx950): gradient
// statistics, an exchange of the workgroups' sums and the Adam update of
// shard_kernels.hpp in a single kernel.
#pragma once

#include "shard_kernels.hpp"

namespace zs {

// ---------------------------------------------------------------------------
// One-launch small-shard step.  The grid is small enough to be resident on
// the device at once (the host keeps it to a fraction of the co-resident
// capacity, so a few such steps on concurrent streams also fit together), which
// the exchange below relies on.  The shard's vector layout is k_adam_vec's
// (`head` single elements, `nvec` 4-element vectors, a tail of 0..3); workgroup
// b walks the tiles b, b + G, ... of kSmallBlock vectors.
//   1. The workgroup sums its gradient vectors' exact squares in fp64 (the last
//      workgroup also takes the head and tail elements) and puts the sum into
//      its slot.
//   2. The first tile's loads of theta, m and v are issued (they overlap the
//      wait; a shard of up to 512K elements has no later tile).
//   3. Every workgroup reads every slot until all are filled and adds them in
//      one fixed order, so all hold the same bits; workgroup 0 publishes the
//      total to the host.
//   4. Unless the step is skipped, the update tile by tile.
// Latency bounds it, not bandwidth, so the exchange is one store and one load
// deep and has no atomic counters: on a 1M-element shard the counters, last
// arrival's total and wake flags that it replaced put the total at 4.3 us, the
// host's record at 5.5 us and the updates at 6.1 us into the kernel.  A whole
// synchronous step took 10.7 us on 1000 elements, 12.4 on 400K and 13.2 on 1M;
// now 8.2, 10.3 and 11.5 us.  The slots a workgroup reads grow with the grid:
// 391 workgroups of 256 threads on 400K elements took 12.5 us, hence at most
// kSmallSlots workgroups of kSmallBlock threads.  Loading a second tile's state
// before the wait as well (11.3 us on 1M), or each later tile's before the tile
// in hand (20.3 against 19.5 us on 3M), gained nothing; loading the gradient
// tile by tile instead of at once costs 0.7 us on 600K and more.
//
// A slot (see shard_kernels.hpp) is filled once, by a compare-and-swap.  Two sets
// of slots alternate from launch to launch of a stream, and each launch empties
// the other set.  The wait is bounded: a workgroup that gives up on an empty slot
// fills it with kSlotMark in the owner's place.  Each slot has one final value that
// everybody reads, so either every workgroup updates or none does; then nothing is
// written, the total is not published, and the host, which finds the stream idle
// without it, empties the slots and launches the kernel sequence.
// ---------------------------------------------------------------------------
constexpr int kSmallBlock = 512;
constexpr int kSmallSlots = 256;                       // the largest grid
constexpr int kSmallTiles = 3;                         // the most tiles per workgroup
constexpr int kSlotWords = 2 * kSmallSlots;            // two sets
static_assert(kSmallSlots <= kSmallBlock, "a thread reads at most one slot");

// The value of a slot, waiting until it is filled (with kSlotMark by this
// thread if that takes too long).
__device__ __forceinline__ uint64_t slot_wait(uint64_t* slot) {
    uint32_t polls = 0;
    for (;;) {
        const uint64_t w = aload(slot);
        if (w != 0)
            return w;
        if (++polls >= kSmallPolls)
            (void)slot_fill(slot, kSlotMark);
        __builtin_amdgcn_s_sleep(1);
    }
}

// The value of a slot whose owner is known to be running and to fill it without
// waiting for anybody.
__device__ __forceinline__ uint64_t slot_read(const uint64_t* slot) {
    uint64_t w;
    while ((w = aload(slot)) == 0)
        __builtin_amdgcn_s_sleep(1);
    return w;
}

// Fixed-order sum of one double per thread, returned to every thread.
// `lds`: BLOCK / 64 doubles that no earlier call of the kernel used.
template <int BLOCK>
__device__ __forceinline__ double small_block_total(double x, double* lds) {
    x = wave_sum(x);
    if ((threadIdx.x & 63) == 0)
        lds[threadIdx.x >> 6] = x;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < BLOCK / 64; ++w)
        s += lds[w];
    return s;
}

// The total of the launch's G slots, the same bits in every workgroup; ends
// with a barrier, after which *abort is 1 if some slot holds kSlotMark.
__device__ __forceinline__ double small_exchange(uint64_t* slots, int G, Sum2* lds2, int* abort) {
    const int tid = (int)threadIdx.x;
    if (tid < kSmallSlots) {
        Sum2 x{0.0, 0.0};
        if (tid < G) {
            const uint64_t w = slot_wait(slots + tid);
            if (w == kSlotMark)
                *abort = 1;
            x.hi = slot_sum(w);
        }
        x = wave_sum2(x);
        if ((tid & 63) == 0)
            lds2[tid >> 6] = x;
    }
    __syncthreads();
    Sum2 x = lds2[0];
#pragma unroll
    for (int w = 1; w < kSmallSlots / 64; ++w)
        x = sum2_add(x, lds2[w]);
    return sum2_value(x);
}

[[maybe_unused]] static __global__ __launch_bounds__(kSmallBlock, 8) void k_small_step(
    const uint16_t* __restrict__ g, float* __restrict__ th, float* __restrict__ m, float* __restrict__ v,
    uint16_t* __restrict__ p, int64_t n, int64_t head, int64_t nvec, uint64_t* __restrict__ slots,
    uint64_t* __restrict__ other, uint64_t* __restrict__ host, double loss_scale, double clip, uint32_t seq,
    AdamConst c) {
    __shared__ double lds[kSmallBlock / 64];
    __shared__ Sum2 lds2[kSmallSlots / 64];
    __shared__ int s_abort;
    const int64_t b = blockIdx.x;
    const int G = (int)gridDim.x;
    const int tid = (int)threadIdx.x;
    const int64_t stride = (int64_t)G * kSmallBlock;
    const int64_t i0 = b * kSmallBlock + tid;

    // 1. statistics of this workgroup's gradient vectors, which stay in registers
    u32x2 gq[kSmallTiles] = {};
    if (i0 < nvec)
        gq[0] = ld4<true>(g + head + 4 * i0);
    if (stride < nvec) {
#pragma unroll
        for (int k = 1; k < kSmallTiles; ++k)
            if (i0 + k * stride < nvec)
                gq[k] = ld4<true>(g + head + 4 * (i0 + k * stride));
    }
    double a0 = 0.0, a1 = 0.0;
#pragma unroll
    for (int k = 0; k < kSmallTiles; ++k) {
        a0 = acc_sq2(gq[k].x, a0);
        a1 = acc_sq2(gq[k].y, a1);
    }
    if (b == G - 1) {
        const int64_t tail0 = head + 4 * nvec;
        if (tid < head)
            a0 += sq1(g[tid]);
        if (tid < 4 && tail0 + tid < n)
            a1 += sq1(g[tail0 + tid]);
    }
    if (tid == 0)
        s_abort = 0;
    double tot = small_block_total<kSmallBlock>(a0 + a1, lds);
    if (G > 1 && tid == 0)
        slot_fill(slots + b, slot_word(tot));

    // 2. the first tile's state, overlapping the wait
    f32x4 tq{}, mq{}, vq{};
    if (i0 < nvec) {
        const int64_t e = head + 4 * i0;
        tq = ld4<true>(th + e);
        mq = ld4<true>(m + e);
        vq = ld4<true>(v + e);
    }
    for (int k = (int)b * kSmallBlock + tid; k < kSmallSlots; k += G * kSmallBlock)
        astore(other + k, 0);

    // 3. the total of all workgroups
    if (G > 1) {
        tot = small_exchange(slots, G, lds2, &s_abort);
        if (s_abort)
            return;
    }
    if (b == 0 && tid == 0)
        publish_sum(host, tot, seq);
    const Result r = make_result(tot, loss_scale, clip, seq);
    if (r.skip)
        return;

    // 4. the update (the last workgroup also takes head and tail)
#pragma unroll
    for (int k = 0; k < kSmallTiles; ++k) {
        const int64_t i = i0 + k * stride;
        if (i >= nvec)
            break;
        const int64_t e = head + 4 * i;
        if (k > 0) {
            tq = ld4<true>(th + e);
            mq = ld4<true>(m + e);
            vq = ld4<true>(v + e);
        }
        f32x4 to, mo, vo;
        u32x2 po;
        adam_vec4(gq[k], tq, mq, vq, r.mult, c, to, mo, vo, po);
        st4<true>(to, th + e);
        st4<true>(mo, m + e);
        st4<true>(vo, v + e);
        st4<true>(po, p + e);
    }
    if (b == G - 1)
        adam_ends(g, th, m, v, p, n, head, nvec, r.mult, c);
}

}  // namespace zs
