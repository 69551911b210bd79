// shard_kernels.hpp -- gfx950 kernels of the ZeRO P_os+g shard step.
//
// ZeRO (arXiv 1910.02054) Sec. 5.1-5.2: after the reduce-scatter each
// data-parallel rank holds the fp16 gradients of its 1/N_d partition and
// updates only that partition's fp32 master parameters, momentum and variance
// (Sec. 3.1's mixed-precision Adam), then publishes the fp16 parameters.
//
// Two kernels run per step, all HBM-streaming (no dense contraction, so no
// MFMA):
//   k_stats     one read of the fp16 gradients; per-workgroup fp64 sum of the
//               exact fp32 squares, totalled by one of them (close_slots).  The sum is
//               non-finite iff some gradient is inf or NaN, which is the
//               overflow test (every finite square is below 2^32, so no finite
//               sum over fewer than 2^990 elements overflows fp64).  From it the
//               norm of the unscaled gradient, the global-norm clipping
//               coefficient, the fp32 gradient multiplier and the skip flag go
//               to device memory, and the sum to the host.
//   k_adam_vec  the fused update: unscale+clip, Adam with bias correction, fp16
//               cast; 14 bytes read and 14 bytes written per element.
// Small shards take one launch instead (k_small_step in small_kernels.hpp).
// The other ways of running the same step change what follows the statistics
// total (FinishStep, FinishSum, FinishResident) or where the update's scalars come from:
// the split phase takes the global sum from the host or from device memory, the
// resident step its hyperparameters and loss scale from a state record in device
// memory (FromResult, FromHost, FromSum, FromResident).
//
// Numerics: every fp32 operation of the update is correctly rounded (IEEE
// division and square root, no contraction), in the order Adam's bias-corrected
// form is written, so an element's result depends only on its own inputs and
// the shared scalars.  The bias corrections 1 - beta^t come from one
// definition shared by the host and the device (bias_correction below).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "zero_shard.h"

namespace zs {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// The same vectors at element alignment, for arrays that start anywhere.  gfx950
// runs in unaligned access mode, so they compile to the same single 16-byte
// (fp32) and 8-byte (fp16) loads and stores as the aligned types.
typedef u32x2 u32x2_e __attribute__((aligned(2)));
typedef f32x4 f32x4_e __attribute__((aligned(4)));

constexpr int kLineBytes = 128;        // a cache line
constexpr int kMaxHead = kLineBytes / 4 - 1;  // elements before the first line of an fp32 array
constexpr int kMaxStatsBlocks = 4096;  // partial-sum records in the workspace

// Launch-policy knobs of the streaming kernels are template parameters:
//   BLOCK  threads per workgroup;  U  vectors per thread per tile;
//   NTL/NTS  non-temporal (streaming) loads/stores;
//   XCD    remap workgroups so that each of the 8 XCDs walks a contiguous run of
//          tiles (the dispatcher assigns workgroup b to XCD b mod 8);
//   REV    walk the tiles from the end of the shard to its start.
template <bool NT, typename T>
__device__ __forceinline__ T ld(const T* p) {
    if constexpr (NT)
        return __builtin_nontemporal_load(p);
    else
        return *p;
}

template <bool NT, typename T>
__device__ __forceinline__ void st(T v, T* p) {
    if constexpr (NT)
        __builtin_nontemporal_store(v, p);
    else
        *p = v;
}

// Four consecutive elements at any element alignment.
template <bool NT>
__device__ __forceinline__ f32x4 ld4(const float* p) {
    const f32x4_e* q = reinterpret_cast<const f32x4_e*>(p);
    if constexpr (NT)
        return __builtin_nontemporal_load(q);
    else
        return *q;
}

template <bool NT>
__device__ __forceinline__ u32x2 ld4(const uint16_t* p) {
    const u32x2_e* q = reinterpret_cast<const u32x2_e*>(p);
    if constexpr (NT)
        return __builtin_nontemporal_load(q);
    else
        return *q;
}

template <bool NT>
__device__ __forceinline__ void st4(f32x4 v, float* p) {
    f32x4_e* q = reinterpret_cast<f32x4_e*>(p);
    if constexpr (NT)
        __builtin_nontemporal_store(v, q);
    else
        *q = v;
}

template <bool NT>
__device__ __forceinline__ void st4(u32x2 v, uint16_t* p) {
    u32x2_e* q = reinterpret_cast<u32x2_e*>(p);
    if constexpr (NT)
        __builtin_nontemporal_store(v, q);
    else
        *q = v;
}

template <bool XCD>
__device__ __forceinline__ int64_t logical_block() {
    const unsigned b = blockIdx.x, grid = gridDim.x;
    if constexpr (XCD) {
        if (grid % 8 == 0)
            return (int64_t)(b % 8) * (grid / 8) + b / 8;  // a bijection of [0, grid)
    }
    return b;
}

// The step's shared scalars, produced on the device by k_stats and read by
// the update kernel.
struct alignas(16) Result {
    double sumsq;    // sum of grad16^2 (loss-scaled); non-finite iff overflow
    double norm;     // sqrt(sumsq) / loss_scale
    double coef;     // clipping coefficient
    float mult;      // (float)(coef / loss_scale)
    int32_t skip;    // 1 = overflow: the update kernel writes nothing
    int32_t overflow;
    uint32_t seq;    // call sequence number
    int32_t unused[2];
};

// fp32 constants of the update, each rounded once from a double (on the host,
// or on the device for the resident step).
struct AdamConst {
    float lr, b1, omb1, b2, omb2, bc1, bc2, eps, wd;
    int32_t quick;        // the constants allow direction4's short sequences
    double rbc1, rbc2;    // 1 / bc1 and 1 / bc2 in double
};

// beta^t for an integer t >= 0, as the double nearest the exact power.  Binary
// powering in double-double arithmetic: each product's rounding error is
// recovered exactly with a fused multiply-add, so the pair carries the power to
// about 2^-90 relative error before the one final rounding to double (the
// exact power of a double is never a midpoint between doubles for t >= 2).
// Every operation is a correctly rounded IEEE multiply, add or fused
// multiply-add, so the host and the device compute the same bits.
struct DDouble {
    double hi, lo;
};

__host__ __device__ inline DDouble dd_mul(DDouble a, DDouble b) {
    const double p = a.hi * b.hi;
    double e = __builtin_fma(a.hi, b.hi, -p);
    e = e + (a.hi * b.lo + a.lo * b.hi);
    const double s = p + e;
    return DDouble{s, e - (s - p)};
}

__host__ __device__ inline double pow_int(double b, int64_t t) {
    DDouble r{1.0, 0.0}, x{b, 0.0};
    while (t > 0) {
        if (t & 1)
            r = dd_mul(r, x);
        t >>= 1;
        if (t)
            x = dd_mul(x, x);
    }
    return r.hi;
}

// The fp32 bias correction 1 - beta^t of Adam's moment estimates: the power
// rounded to double, the difference in double, then one rounding to fp32.
__host__ __device__ inline float bias_correction(double beta, int64_t t) {
    return (float)(1.0 - pow_int(beta, t));
}

// The fp32 constants from the hyperparameters (each computed in double and
// rounded once).
__host__ __device__ inline AdamConst make_adam_const(double lr, double beta1, double beta2, double eps, double wd,
                                                     int64_t t) {
    AdamConst c;
    c.lr = (float)lr;
    c.b1 = (float)beta1;
    c.omb1 = (float)(1.0 - beta1);
    c.b2 = (float)beta2;
    c.omb2 = (float)(1.0 - beta2);
    c.bc1 = bias_correction(beta1, t);
    c.bc2 = bias_correction(beta2, t);
    c.eps = (float)eps;
    c.wd = (float)wd;
    c.quick = c.bc1 >= 0x1p-24f && c.bc2 >= 0x1p-24f && c.eps <= 0x1p40f;
    c.rbc1 = 1.0 / (double)c.bc1;
    c.rbc2 = 1.0 / (double)c.bc2;
    return c;
}

// The hyperparameter ranges every step accepts (the synchronous entry points
// check the same on the host): lr, eps >= 0 and finite, weight decay finite,
// beta1, beta2 in [0, 1), t >= 1, loss scale finite and > 0, clip not NaN.
__host__ __device__ inline bool hyper_ok(double lr, double beta1, double beta2, double eps, double wd, int64_t t,
                                         double loss_scale, double clip) {
    return __builtin_isfinite(lr) && lr >= 0.0 && __builtin_isfinite(eps) && eps >= 0.0 && __builtin_isfinite(wd) &&
           beta1 >= 0.0 && beta1 < 1.0 && beta2 >= 0.0 && beta2 < 1.0 && t >= 1 && __builtin_isfinite(loss_scale) &&
           loss_scale > 0.0 && !__builtin_isnan(clip);
}

// A resident state record the step can run from: hyper_ok plus a finite
// min_scale > 0.
__host__ __device__ inline bool resident_record_ok(const zero_resident_state_t& s) {
    return hyper_ok(s.lr, s.beta1, s.beta2, s.eps, s.weight_decay, s.t, s.loss_scale, s.clip) &&
           __builtin_isfinite(s.min_scale) && s.min_scale > 0.0;
}

__device__ __forceinline__ float f16_to_f32(uint32_t bits16) {
    return (float)__builtin_bit_cast(_Float16, (uint16_t)bits16);
}

__device__ __forceinline__ uint32_t f32_to_f16(float x) {
    // v_cvt_f16_f32 in the default round-to-nearest-even mode, fp16 denormals kept.
    return (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)x);
}

// acc + g^2 for both halves of a 32-bit word; the square of a binary16 value
// is exact in fp32 (22 significant bits) and in fp64.
__device__ __forceinline__ double acc_sq2(uint32_t w, double acc) {
    double lo = (double)f16_to_f32(w & 0xFFFFu);
    double hi = (double)f16_to_f32(w >> 16);
    acc = __builtin_fma(lo, lo, acc);
    return __builtin_fma(hi, hi, acc);
}

__device__ __forceinline__ double sq1(uint32_t bits16) {
    double d = (double)f16_to_f32(bits16);
    return d * d;
}

// Cross-lane steps of a 64-lane sum, in the vector ALU: within rows of 16 lanes
// by DPP (the neighbour, the other pair, the other quad, the other half row; the
// last two are mirrors, which serve because by then all lanes of a quad or half
// row hold the same value), across rows by gfx950's row and half-wave swaps.
// Every lane ends with the bits that an exclusive-or butterfly gives.  A shuffle
// through the LDS crossbar takes 2 instructions and some 100 cycles a step, and
// these sums lie on the path to every exchange: with them a LAMB step on 1M
// elements takes 16.9 us where it took 17.7, a resident step 12.65 (13.1), a fused
// step on 5.9M 34.0 (34.4), a LAMB step on 20M 147.5 (148.7).
template <int CTRL>
__device__ __forceinline__ double lane_dpp(double x) {
    const u32x2 w = __builtin_bit_cast(u32x2, x);
    const u32x2 r = {(uint32_t)__builtin_amdgcn_update_dpp(0, (int)w.x, CTRL, 0xF, 0xF, true),
                     (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w.y, CTRL, 0xF, 0xF, true)};
    return __builtin_bit_cast(double, r);
}

// The two values that lanes of this lane's pair of rows (HALF false) or of the
// two half waves (HALF true) hold at this lane's place.
template <bool HALF>
__device__ __forceinline__ void lane_pair(double x, double& a, double& b) {
    const u32x2 w = __builtin_bit_cast(u32x2, x);
    const auto lo = HALF ? __builtin_amdgcn_permlane32_swap(w.x, w.x, false, false)
                         : __builtin_amdgcn_permlane16_swap(w.x, w.x, false, false);
    const auto hi = HALF ? __builtin_amdgcn_permlane32_swap(w.y, w.y, false, false)
                         : __builtin_amdgcn_permlane16_swap(w.y, w.y, false, false);
    a = __builtin_bit_cast(double, u32x2{lo[0], hi[0]});
    b = __builtin_bit_cast(double, u32x2{lo[1], hi[1]});
}

__device__ __forceinline__ double wave_sum(double x) {
    x += lane_dpp<0xB1>(x);   // quad_perm 1, 0, 3, 2
    x += lane_dpp<0x4E>(x);   // quad_perm 2, 3, 0, 1
    x += lane_dpp<0x141>(x);  // row_half_mirror
    x += lane_dpp<0x140>(x);  // row_mirror
    double a, b;
    lane_pair<false>(x, a, b);
    lane_pair<true>(a + b, a, b);
    return a + b;
}

// A sum carried with its rounding error (each addition's error is recovered
// exactly), so that the total of the workgroups' sums is theirs to about 2^-100
// before its one rounding, whatever the order: the one-launch step and the
// statistics pass cut the shard differently and report the same bits (but for a
// tie within the sums' own last bits).
struct Sum2 {
    double hi, lo;
};

__device__ __forceinline__ Sum2 sum2_add(Sum2 a, Sum2 b) {
    const double s = a.hi + b.hi, t = s - a.hi;
    return Sum2{s, (a.lo + b.lo) + ((a.hi - (s - t)) + (b.hi - t))};
}

// An overflowed sum's error term is NaN: the sum itself is the value then.
__device__ __forceinline__ double sum2_value(Sum2 a) { return __builtin_isfinite(a.hi) ? a.hi + a.lo : a.hi; }

template <int CTRL>
__device__ __forceinline__ Sum2 lane_dpp(Sum2 x) {
    return Sum2{lane_dpp<CTRL>(x.hi), lane_dpp<CTRL>(x.lo)};
}

__device__ __forceinline__ Sum2 wave_sum2(Sum2 x) {
    x = sum2_add(x, lane_dpp<0xB1>(x));
    x = sum2_add(x, lane_dpp<0x4E>(x));
    x = sum2_add(x, lane_dpp<0x141>(x));
    x = sum2_add(x, lane_dpp<0x140>(x));
    Sum2 a, b;
    lane_pair<false>(x.hi, a.hi, b.hi);
    lane_pair<false>(x.lo, a.lo, b.lo);
    x = sum2_add(a, b);
    lane_pair<true>(x.hi, a.hi, b.hi);
    lane_pair<true>(x.lo, a.lo, b.lo);
    return sum2_add(a, b);
}

// A workgroup's sum on its way to the others of its launch: a 64-bit slot in
// device memory that is empty (0) before the launch and is filled with the
// sum's bits under a set sign bit (a sum of squares is never negative), so one
// word carries the sum and that it is there.  Slots are accessed with
// agent-scope atomic operations, which the device keeps coherent across its
// XCDs without writing back or invalidating the L2 caches.
//
// Polls of an empty slot (about 0.5-1 us each) after which a workgroup stops
// waiting: a closing workgroup then hands over (close_slots), a workgroup of a
// one-launch step gives the step up (slot_wait).  A build for tests sets both
// low, so that both happen all the time.
#ifndef ZS_CLOSE_POLLS
#define ZS_CLOSE_POLLS (1u << 10)
#endif
#ifndef ZS_SMALL_POLLS
#define ZS_SMALL_POLLS (1u << 22)
#endif
constexpr uint64_t kSlotFilled = (uint64_t)1 << 63;
constexpr uint64_t kSlotMark = ~(uint64_t)0;           // not the bits of a sum of squares
constexpr uint32_t kClosePolls = ZS_CLOSE_POLLS;
constexpr uint32_t kSmallPolls = ZS_SMALL_POLLS;

__device__ __forceinline__ uint64_t slot_word(double x) { return __builtin_bit_cast(uint64_t, x) | kSlotFilled; }
__device__ __forceinline__ double slot_sum(uint64_t w) { return __builtin_bit_cast(double, w & ~kSlotFilled); }

__device__ __forceinline__ uint64_t aload(const uint64_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void astore(uint64_t* p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Fills an empty slot, a filled one keeps its value; returns what it held.
__device__ __forceinline__ uint64_t slot_fill(uint64_t* slot, uint64_t v) {
    uint64_t held = 0;
    (void)__hip_atomic_compare_exchange_strong(slot, &held, v, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
    return held;
}

// The value of a 64-bit word in the wave's first active lane.
__device__ __forceinline__ uint64_t first_lane(uint64_t x) {
    return (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x) |
           (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32)) << 32;
}

// The W sums of each of `count` members, brought together by one of them.  Each
// member calls this once, with one whole wave and its own sums (read from lane
// 0); slots[W * i .. W * i + W) are member i's.  It returns true for exactly one
// member, with sums[k] in every lane: this lane's share (members lane, lane +
// 64, ...) of the k-th sums, added in a fixed order.  All slots are empty again
// then.  MANY: there may be more than 64 members.
//
// The last member closes: it polls the others' slots, which they normally fill
// before it gets there or within microseconds.  It must not rely on that:
// they may not even have been dispatched while other work fills part of the
// device.  So after kClosePolls it leaves its own sums in its slots, puts
// kSlotMark into a slot that is still empty and returns; that slot's owner finds
// the mark when it comes to fill it (the compare-and-swap decides which of the
// two was first) and closes in its place, or hands over to another late member
// in turn.  Nobody waits for longer, every launch's total is produced whatever
// the dispatch order, and no slot is filled after the one that closes emptied
// it, whether or not a host looks on.
template <int W, bool MANY>
__device__ __forceinline__ bool close_slots(uint64_t* slots, int count, int me, const double (&mine)[W],
                                            double (&sums)[W]) {
    const int lane = (int)threadIdx.x & 63;
    uint64_t own[W];
#pragma unroll
    for (int k = 0; k < W; ++k)
        own[k] = slot_word(__builtin_bit_cast(double, first_lane(__builtin_bit_cast(uint64_t, mine[k]))));
    if (me != count - 1) {
        bool mark = false;
        if (lane == 0) {
            uint64_t held[W];
#pragma unroll
            for (int k = 0; k < W; ++k)
                held[k] = slot_fill(slots + W * me + k, own[k]);
#pragma unroll
            for (int k = 0; k < W; ++k)
                mark = mark || held[k] == kSlotMark;
        }
        if (__builtin_expect(!__any(mark), 1))
            return false;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
#pragma unroll
    for (int k = 0; k < W; ++k)
        sums[k] = 0.0;
    int base = 0;
    do {
        const int i = base + lane;
        uint64_t* const theirs = slots + W * i;
        uint64_t w[W];
#pragma unroll
        for (int k = 0; k < W; ++k)
            w[k] = own[k];
        // one exit and branches of the whole wave: this is on the path to every total
        uint64_t late;
        bool handed = false;
        uint32_t polls = 0;
        do {
            bool missing = false;
            if (i < count && i != me) {
#pragma unroll
                for (int k = 0; k < W; ++k)
                    w[k] = aload(theirs + k);
#pragma unroll
                for (int k = 0; k < W; ++k)
                    missing = missing || w[k] == 0;
            }
            late = __ballot(missing);
            if (__builtin_expect(late != 0 && polls++ >= kClosePolls, 0)) {
                if (lane == __builtin_ctzll(late)) {
                    int empty = 0;
#pragma unroll
                    for (int k = W - 1; k >= 0; --k) {
                        astore(slots + W * me + k, own[k]);
                        empty = w[k] == 0 ? k : empty;
                    }
                    // the release: whoever finds the mark finds this member's sums, too
                    uint64_t held = 0;
                    handed = __hip_atomic_compare_exchange_strong(theirs + empty, &held, kSlotMark, __ATOMIC_RELEASE,
                                                                  __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                late = __any(handed) ? 0 : late;
            }
        } while (late != 0);
        if (__any(handed))
            return false;
        if (i < count) {
#pragma unroll
            for (int k = 0; k < W; ++k)
                sums[k] += slot_sum(w[k]);
        }
        base += 64;
    } while (MANY && base < count);
    for (int i = lane; i < count; i += 64) {
#pragma unroll
        for (int k = 0; k < W; ++k)
            astore(slots + W * i + k, 0);
        if (!MANY)
            break;
    }
    return true;
}

// Norm, clipping coefficient, multiplier and skip flag from the global sum of
// squares (all in double; the multiplier rounded once to fp32).  The host
// evaluates it too, from the sum that the device publishes; every operation is
// correctly rounded, so both get the same bits.
__host__ __device__ inline Result make_result(double tot, double loss_scale, double clip, uint32_t seq) {
    Result r;
    r.sumsq = tot;
    r.overflow = __builtin_isfinite(tot) ? 0 : 1;
    r.skip = r.overflow;
    if (r.overflow) {
        r.norm = __builtin_inf();
        r.coef = 1.0;
        r.mult = 0.0f;
    } else {
        r.norm = __builtin_sqrt(tot) / loss_scale;
        r.coef = (clip > 0.0 && r.norm > clip) ? clip / r.norm : 1.0;
        r.mult = (float)(r.coef / loss_scale);
    }
    r.seq = seq;
    r.unused[0] = r.unused[1] = 0;
    return r;
}

// The statistics total to the host's two mapped words, each with the call's
// sequence number in its high half.  Each word is complete in itself, so the
// host needs no order between them and the device neither a release (an L2
// write-back) nor a wait before the sequence number.
__device__ __forceinline__ void publish_sum(uint64_t* __restrict__ host, double tot, uint32_t seq) {
    const uint64_t w = __builtin_bit_cast(uint64_t, tot), tag = (uint64_t)seq << 32;
    __hip_atomic_store(host, tag | (w & 0xFFFFFFFFu), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(host + 1, tag | (w >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// What becomes of the statistics total, by one lane of the workgroup of k_stats
// that closes its sums.  `before` is called once by that workgroup ahead of
// `total`; by the last one, which closes them as a rule, at its start.
// The fused step: the result record, and the sum to the host.
struct FinishStep {
    Result* res;
    uint64_t* host;
    double loss_scale, clip;
    uint32_t seq;
    __device__ __forceinline__ void before() {}
    __device__ __forceinline__ void total(double tot) {
        publish_sum(host, tot, seq);
        *res = make_result(tot, loss_scale, clip, seq);
    }
};

// The asynchronous split phase: the sum into caller device memory.
struct FinishSum {
    double* out;
    __device__ __forceinline__ void before() {}
    __device__ __forceinline__ void total(double tot) { *out = tot; }
};

// The total of the sums of `count` <= 64 members (close_slots), by the one member
// for which this returns true.
__device__ __forceinline__ bool close_total(uint64_t* slots, int count, int me, double& sum) {
    if (count == 1)
        return true;
    const double mine[1] = {sum};
    double share[1];
    if (!close_slots<1, false>(slots, count, me, mine, share))
        return false;
    sum = sum2_value(wave_sum2(Sum2{share[0], 0.0}));
    return true;
}

// ---------------------------------------------------------------------------
// K1: statistics.  `head` leading elements (0..63) lie before the gradient's
// first cache line and `nvec` 8-element vectors follow; elements
// [head + 8*nvec, n) are the tail.  Grid: 1 .. kMaxStatsBlocks workgroups of one
// wave.  The workgroups' sums meet in two levels, each a fixed-order sum
// (bitwise reproducible for a given launch shape): workgroup b fills slot b, one
// workgroup of every 64 closes its group's slots (close_slots: the last one, or
// one that came late) and fills the group's slot, and one of those closes the
// groups' and finishes (FIN).
// Reading the gradient bounds the pass on large shards; the total costs two
// round trips at its end, where a kernel of its own (of one workgroup) took 3.5
// to 4.6 us a step.  (One level, the last workgroup draining all 2047 slots,
// took 4 us more than that kernel.)  Steps before and after: resident 1M 14.9 ->
// 13.3 us and 20K 14.8 -> 11.4, fused 5.9M 36.1 -> 35.3, 94M 420 -> 417.5, 250M
// 1116 -> 1115.  That a late workgroup can take the closing over, where a bounded
// wait was given up with a wrong or missing total, costs 0.3 us (resident 1M
// 12.57 -> 12.86, asynchronous 5.9M 35.3 -> 35.6); the code that is skipped for it
// takes most of that, not the compare-and-swap.
// ---------------------------------------------------------------------------
constexpr int kStatsSlots = kMaxStatsBlocks + kMaxStatsBlocks / 64;  // the workgroups', then the groups'
static_assert(kMaxStatsBlocks <= 64 * 64, "one wave drains the groups");

template <int U, bool NTL, bool XCD, typename FIN>
__global__ __launch_bounds__(64) void k_stats(const uint16_t* __restrict__ g, int64_t n, int64_t head, int64_t nvec,
                                              uint64_t* __restrict__ part, FIN fin) {
    if (blockIdx.x == gridDim.x - 1)
        fin.before();
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
    const u32x4* __restrict__ gv = reinterpret_cast<const u32x4*>(g + head);
    const int64_t tile = (int64_t)64 * U;
    const int64_t stride = (int64_t)gridDim.x * tile;
    for (int64_t base = logical_block<XCD>() * tile + threadIdx.x; base < nvec; base += stride) {
        u32x4 q[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t i = base + (int64_t)u * 64;
            q[u] = i < nvec ? ld<NTL>(gv + i) : u32x4{0u, 0u, 0u, 0u};
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            a0 = acc_sq2(q[u].x, a0);
            a1 = acc_sq2(q[u].y, a1);
            a2 = acc_sq2(q[u].z, a2);
            a3 = acc_sq2(q[u].w, a3);
        }
    }
    if (blockIdx.x == 0) {
        const int64_t t = threadIdx.x;
        const int64_t tail0 = head + 8 * nvec;
        if (t < head)
            a0 += sq1(g[t]);
        if (t < 8 && tail0 + t < n)
            a1 += sq1(g[tail0 + t]);
    }
    const double s = wave_sum((a0 + a1) + (a2 + a3));
    const int b = (int)blockIdx.x, last = (int)gridDim.x - 1, group = b >> 6, groups = (last >> 6) + 1;
    const int count = group == groups - 1 ? (last & 63) + 1 : 64;
    double tot = s;
    if (!close_total(part + (b & ~63), count, b & 63, tot) ||
        !close_total(part + kMaxStatsBlocks, groups, group, tot))
        return;
    if (b != last)
        fin.before();
    if (threadIdx.x == 0)
        fin.total(tot);
}

// One double into device memory (the empty shard's local sum, enqueued in order).
[[maybe_unused]] static __global__ __launch_bounds__(64) void k_set_value(double* __restrict__ out, double value) {
    if (threadIdx.x == 0)
        *out = value;
}

// Zeroes n 64-bit words (counters cleared in stream order).
[[maybe_unused]] static __global__ __launch_bounds__(256) void k_zero_words(uint64_t* __restrict__ out, int64_t n) {
    for (int64_t i = threadIdx.x; i < n; i += 256)
        out[i] = 0;
}

// A caller's global sum of squares; +inf for what cannot be one.
__device__ __forceinline__ double sum_of_squares(double g) { return g >= 0.0 ? g : __builtin_inf(); }

// Result record from a global sum of squares in device memory (the
// asynchronous split phase); the skip flag also goes to `skipped` when given
// (device or host-mapped memory).
[[maybe_unused]] static __global__ __launch_bounds__(64) void k_set_result_dev(Result* __restrict__ res,
                                                                                const double* __restrict__ global,
                                                                                double loss_scale, double clip,
                                                                                int32_t* __restrict__ skipped,
                                                                                uint32_t seq) {
    if (threadIdx.x == 0) {
        const Result r = make_result(sum_of_squares(*global), loss_scale, clip, seq);
        *res = r;
        if (skipped)
            *skipped = r.skip;
    }
}

// The resident step's decision from the statistics total and the record `s`
// read before the step: the result record, and the record's new scaler fields
// written to *st (skipped = -1 and nothing else for a record out of range).
__device__ __forceinline__ Result resident_advance(zero_resident_state_t* __restrict__ st,
                                                   const zero_resident_state_t& s, double tot, uint32_t seq) {
    if (!resident_record_ok(s)) {
        Result r = make_result(0.0, 1.0, 0.0, seq);
        r.skip = 1;
        st->skipped = -1;
        return r;
    }
    const Result r = make_result(tot, s.loss_scale, s.clip, seq);
    st->steps = s.steps + 1;
    st->skipped = r.skip;
    if (r.skip) {
        const double h = s.loss_scale * 0.5;
        st->loss_scale = h > s.min_scale ? h : s.min_scale;
        st->good = 0;
    } else {
        st->t = s.t + 1;
        int64_t good = s.good + 1;
        if (s.window > 0 && good >= s.window) {
            st->loss_scale = s.loss_scale * 2.0;
            good = 0;
        }
        st->good = good;
    }
    return r;
}

// The resident step: the result record from the total and the state record's
// loss scale and clip, the fp32 constants from the record's hyperparameters and
// t (make_adam_const, the host's definition), and the loss-scale schedule on
// the record: after an overflow the scale halves (not below min_scale) and t
// stays; otherwise t and the good-step count advance and the scale doubles after
// `window` good steps.  The update kernel reads only the result record and the
// constants, so the schedule need not wait for it.  A record outside the
// accepted ranges (resident_record_ok) is left unchanged except for
// skipped = -1, and the step writes nothing.
struct FinishResident {
    zero_resident_state_t* st;
    Result* res;
    AdamConst* cout;
    uint32_t seq;
    zero_resident_state_t s;  // the record before the step
    __device__ __forceinline__ void before() {
        s = *st;
        const AdamConst c = make_adam_const(s.lr, s.beta1, s.beta2, s.eps, s.weight_decay, s.t);
        if (threadIdx.x == 0)
            *cout = c;
    }
    __device__ __forceinline__ void total(double tot) {
        *res = resident_advance(st, s, tot, seq);
    }
};

// Where an update takes its multiplier and constants from; false: the step is
// skipped and nothing may be written.
// A result record written by an earlier kernel of the stream.
struct FromResult {
    const Result* res;
    AdamConst consts;
    __device__ __forceinline__ bool get(float& mult, AdamConst& c) const {
        if (res->skip)
            return false;
        mult = res->mult;
        c = consts;
        return true;
    }
};

// The resident step: the constants, too, come from an earlier kernel.
struct FromResident {
    const Result* res;
    const AdamConst* consts;
    __device__ __forceinline__ bool get(float& mult, AdamConst& c) const {
        if (res->skip)
            return false;
        mult = res->mult;
        c = *consts;
        return true;
    }
};

// The split phase with a global sum that the host holds (it does not launch a
// skipped update).
struct FromHost {
    float multiplier;
    AdamConst consts;
    __device__ __forceinline__ bool get(float& mult, AdamConst& c) const {
        mult = multiplier;
        c = consts;
        return true;
    }
};

// The asynchronous split phase: a global sum in device memory, which every wave
// turns into the multiplier (a negative sum or NaN is not a sum of squares and
// skips like an overflow); the first workgroup stores the skip flag.
struct FromSum {
    const double* sum;
    double loss_scale, clip;
    int32_t* skipped;
    AdamConst consts;
    __device__ __forceinline__ bool get(float& mult, AdamConst& c) const {
        const Result r = make_result(sum_of_squares(*sum), loss_scale, clip, 0);
        if (skipped && blockIdx.x == 0 && threadIdx.x == 0)
            *skipped = r.skip;
        mult = r.mult;
        c = consts;
        return !r.skip;
    }
};

// ---------------------------------------------------------------------------
// The update direction u = (m / bc1) / (sqrt(v / bc2) + eps) from the new
// moments, every operation correctly rounded.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float direction(float m, float v, const AdamConst& c) {
#pragma clang fp contract(off)
    const float mhat = m / c.bc1;
    const float vhat = v / c.bc2;
    const float denom = __builtin_sqrtf(vhat) + c.eps;
    return mhat / denom;
}

// The same bits for moments in the usual range, in about half the instructions:
// the general division and square root spend most of theirs on scaling and on
// operands that do not occur here.  With 2^-80 <= |m| <= 2^40, 2^-100 <= v <=
// 2^60, bc1, bc2 >= 2^-24 and eps <= 2^40 no intermediate leaves the normal range.
//   x / bc: x times the double 1 / bc, rounded to fp32.  The product is within
//     2^-52 of the quotient; a quotient of two 24-bit significands is never a
//     midpoint between floats and lies at least 2^-49 from one, so the rounding
//     is the quotient's.
//   sqrt: v_rsq_f32 and one fused residual step (equal to the correctly rounded
//     root for every float in [2^-100, 2^84): the GPU tests go through them all).
//   mhat / denom: v_rcp_f32, one Newton step, and two residual corrections
//     (Markstein): the general division's own sequence without its scaling.
__device__ __forceinline__ float direction_quick(float m, float v, const AdamConst& c) {
#pragma clang fp contract(off)
    const float mhat = (float)((double)m * c.rbc1);
    const float vhat = (float)((double)v * c.rbc2);
    const float r = __builtin_amdgcn_rsqf(vhat);
    const float s0 = vhat * r;
    const float denom = __builtin_fmaf(__builtin_fmaf(-s0, s0, vhat), 0.5f * r, s0) + c.eps;
    float y = __builtin_amdgcn_rcpf(denom);
    y = __builtin_fmaf(__builtin_fmaf(-denom, y, 1.0f), y, y);
    float q = mhat * y;
    q = __builtin_fmaf(__builtin_fmaf(-denom, q, mhat), y, q);
    return __builtin_fmaf(__builtin_fmaf(-denom, q, mhat), y, q);
}

// Directions of four elements: the short sequences when all four of every
// active lane are in range (zero moments are not), the general ones otherwise.
// The vector ALU bounds neither the update nor the LAMB passes alone, but it
// shares their time: LAMB moments + apply (64-thread workgroups, 32 a CU) on
// 5.9M elements 49.4 us with them and 51.0 without, 61M 382 and 394, 140M 860
// and 875, 250M 1557 and 1560; the Adam step on 250M 1110 and 1113.
__device__ __forceinline__ void direction4(const float m[4], const float v[4], const AdamConst& c, float u[4]) {
    const float m0 = __builtin_fabsf(m[0]), m1 = __builtin_fabsf(m[1]), m2 = __builtin_fabsf(m[2]),
                m3 = __builtin_fabsf(m[3]);
    const float mlo = __builtin_fminf(__builtin_fminf(m0, m1), __builtin_fminf(m2, m3));
    const float mhi = __builtin_fmaxf(__builtin_fmaxf(m0, m1), __builtin_fmaxf(m2, m3));
    const float vlo = __builtin_fminf(__builtin_fminf(v[0], v[1]), __builtin_fminf(v[2], v[3]));
    const float vhi = __builtin_fmaxf(__builtin_fmaxf(v[0], v[1]), __builtin_fmaxf(v[2], v[3]));
    const bool usual = c.quick && mlo >= 0x1p-80f && mhi <= 0x1p40f && vlo >= 0x1p-100f && vhi <= 0x1p60f;
    if (__all(usual)) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            u[k] = direction_quick(m[k], v[k], c);
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            u[k] = direction(m[k], v[k], c);
    }
}

// ---------------------------------------------------------------------------
// The per-element update: one definition of each half for the vectors and for
// the single elements at the ends, so every element is computed identically.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void moments_elem(uint32_t g16, float mult, float& m, float& v, const AdamConst& c) {
#pragma clang fp contract(off)
    const float g = f16_to_f32(g16) * mult;
    m = c.b1 * m + c.omb1 * g;
    v = c.b2 * v + c.omb2 * (g * g);
}

__device__ __forceinline__ float decayed(float u, float th, const AdamConst& c) {
#pragma clang fp contract(off)
    return c.wd != 0.0f ? u + c.wd * th : u;
}

__device__ __forceinline__ uint32_t adam_elem(float u, float& th, const AdamConst& c) {
#pragma clang fp contract(off)
    th = th - c.lr * decayed(u, th, c);
    return f32_to_f16(th);
}

__device__ __forceinline__ void adam_one(const uint16_t* g, float* th, float* m, float* v, uint16_t* p, int64_t i,
                                         float mult, const AdamConst& c) {
    float t = th[i], mm = m[i], vv = v[i];
    moments_elem(g[i], mult, mm, vv, c);
    const uint32_t h = adam_elem(direction(mm, vv, c), t, c);
    th[i] = t;
    m[i] = mm;
    v[i] = vv;
    p[i] = (uint16_t)h;
}

// The elements outside the vectors, [0, head) and [head + 4*nvec, n), by the
// first kMaxHead + 4 threads of one workgroup.
__device__ __forceinline__ void adam_ends(const uint16_t* g, float* th, float* m, float* v, uint16_t* p, int64_t n,
                                          int64_t head, int64_t nvec, float mult, const AdamConst& c) {
    const int64_t t = threadIdx.x, tail = head + 4 * nvec + (t - kMaxHead);
    if (t < head)
        adam_one(g, th, m, v, p, t, mult, c);
    else if (t >= kMaxHead && tail < n)
        adam_one(g, th, m, v, p, tail, mult, c);
}

// Four consecutive elements of the vectors: the loaded gradient word pair
// and fp32 vectors in, the updated fp32 vectors and fp16 word pair out.
__device__ __forceinline__ void adam_vec4(u32x2 gq, f32x4 tq, f32x4 mq, f32x4 vq, float mult, const AdamConst& c,
                                          f32x4& to, f32x4& mo, f32x4& vo, u32x2& po) {
    float t[4] = {tq.x, tq.y, tq.z, tq.w};
    float mm[4] = {mq.x, mq.y, mq.z, mq.w};
    float vvv[4] = {vq.x, vq.y, vq.z, vq.w};
    const uint32_t gw[4] = {gq.x & 0xFFFFu, gq.x >> 16, gq.y & 0xFFFFu, gq.y >> 16};
    float u[4];
    uint32_t h[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        moments_elem(gw[k], mult, mm[k], vvv[k], c);
    direction4(mm, vvv, c, u);
#pragma unroll
    for (int k = 0; k < 4; ++k)
        h[k] = adam_elem(u[k], t[k], c);
    to = f32x4{t[0], t[1], t[2], t[3]};
    mo = f32x4{mm[0], mm[1], mm[2], mm[3]};
    vo = f32x4{vvv[0], vvv[1], vvv[2], vvv[3]};
    po = u32x2{h[0] | (h[1] << 16), h[2] | (h[3] << 16)};
}

// K2.  The shard in 4-element vectors after `head` (0..kMaxHead) single
// elements, which bring the fp32 master array to a cache line: one 16-byte
// access per fp32 array and one 8-byte access per fp16 array, consecutive
// lanes on consecutive vectors.  The other arrays may start at any element
// (the rank's slice of the flat fp16 buffers starts at rank * S, the fp32
// state at the start of an allocation): their accesses are then unaligned but
// still one instruction each.  HBM bandwidth bounds it.  Whole steps on 61M
// elements: 279 us aligned; 293 us with the fp16 arrays three elements off
// (two of the five lines of a wave's fp16 store are partial), 351 us by the
// element-by-element kernel that such arrays took before; 288 us with all five
// arrays three elements off, 363 us when their vectors began at the first
// 16-byte boundary and every fp32 store ended in partial lines.
// A tile is BLOCK*U vectors; each thread loads its U
// vectors of all four inputs before computing (with U = 1, the production
// shape, the loads, the update and the stores sit under one bounds test,
// which measured about 4 us faster per 250M-element launch than a separate
// test for the loads and for the rest).  Elements [head + 4*nvec, n) are the
// tail (0..3).  The last workgroup takes head and tail; the host gives them a
// workgroup without a tile, so that no workgroup has both latencies in a row.
// Any grid size is valid (tiles are strided by it).
template <int BLOCK, int U, bool NTL, bool NTS, bool XCD, bool REV, typename SRC>
__global__ __launch_bounds__(BLOCK) void k_adam_vec(const uint16_t* __restrict__ g, float* __restrict__ th,
                                                    float* __restrict__ m, float* __restrict__ v,
                                                    uint16_t* __restrict__ p, int64_t n, int64_t head, int64_t nvec,
                                                    SRC src) {
    float mult;
    AdamConst c;
    if (!src.get(mult, c))
        return;
    if (blockIdx.x == gridDim.x - 1)
        adam_ends(g, th, m, v, p, n, head, nvec, mult, c);
    const int64_t tile = (int64_t)BLOCK * U;
    const int64_t ntiles = (nvec + tile - 1) / tile;
    for (int64_t tb = logical_block<XCD>(); tb < ntiles; tb += gridDim.x) {
        const int64_t base = (REV ? ntiles - 1 - tb : tb) * tile + threadIdx.x;
        if constexpr (U == 1) {
            if (base < nvec) {
                const int64_t e = head + 4 * base;
                f32x4 to, mo, vo;
                u32x2 po;
                adam_vec4(ld4<NTL>(g + e), ld4<NTL>(th + e), ld4<NTL>(m + e), ld4<NTL>(v + e), mult, c, to, mo, vo,
                          po);
                st4<NTS>(to, th + e);
                st4<NTS>(mo, m + e);
                st4<NTS>(vo, v + e);
                st4<NTS>(po, p + e);
            }
        } else {
            u32x2 gq[U];
            f32x4 tq[U], mq[U], vq[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t i = base + (int64_t)u * BLOCK;
                if (i < nvec) {
                    const int64_t e = head + 4 * i;
                    gq[u] = ld4<NTL>(g + e);
                    tq[u] = ld4<NTL>(th + e);
                    mq[u] = ld4<NTL>(m + e);
                    vq[u] = ld4<NTL>(v + e);
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t i = base + (int64_t)u * BLOCK;
                if (i < nvec) {
                    f32x4 to, mo, vo;
                    u32x2 po;
                    adam_vec4(gq[u], tq[u], mq[u], vq[u], mult, c, to, mo, vo, po);
                    const int64_t e = head + 4 * i;
                    st4<NTS>(to, th + e);
                    st4<NTS>(mo, m + e);
                    st4<NTS>(vo, v + e);
                    st4<NTS>(po, p + e);
                }
            }
        }
    }
}

// Streaming copy of nvec 16-byte vectors: the achievable-bandwidth reference
// for the update kernel (same tiling knobs) and the calibration kernel for
// hardware byte counters.
template <int BLOCK, int U, bool NTL, bool NTS, bool XCD>
__global__ __launch_bounds__(BLOCK) void k_probe_copy(const u32x4* __restrict__ src, u32x4* __restrict__ dst,
                                                      int64_t nvec) {
    const int64_t tile = (int64_t)BLOCK * U;
    const int64_t stride = (int64_t)gridDim.x * tile;
    for (int64_t base = logical_block<XCD>() * tile + threadIdx.x; base < nvec; base += stride) {
        u32x4 q[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t i = base + (int64_t)u * BLOCK;
            if (i < nvec)
                q[u] = ld<NTL>(src + i);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t i = base + (int64_t)u * BLOCK;
            if (i < nvec)
                st<NTS>(q[u], dst + i);
        }
    }
}

}  // namespace zs
