// zero_lamb.hip -- host side of the LAMB shard step (declared in
// include/zero_shard.h): the layer-table plan and its work lists, argument
// checks, launches, split-phase entry points and sampled kernel timing.
//
// LAMB (You et al.) is listed in ZeRO's related work (Sec. 2.3) among the
// adaptive optimizers whose state ZeRO's partitioning (Sec. 5.1-5.2) makes
// affordable; the fp32 state per parameter is Adam's (Sec. 3.1, K = 12).
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <memory>
#include <mutex>
#include <vector>

#include "zero_shard.h"
#include "shard_kernels.hpp"
#include "lamb_kernels.hpp"
#include "lamb_small.hpp"
#include "host_common.hpp"

// ---------------------------------------------------------------------------
// Launch policy of the two LAMB streaming passes (template knobs in
// lamb_kernels.hpp): one tile of BLOCK*U 4-element vectors per workgroup, at
// most kLambPerCU resident workgroups per CU (an LDS reservation).  Fewer streams
// in flight suit the DRAM better, as for the Adam update (12 waves), but each
// wave here also waits for its tile's layer pieces and adds fp64 sums, so about
// 24 waves are needed to keep the streams busy.  MI355X, 250M elements, us of the
// moments and the apply pass by resident workgroups: 10: 855, 701; 11: 841, 707;
// 12: 835, 715; 13: 838, 718; 14: 842, 720; 16: 846, 720 (what the passes had
// before direction4 halved the arithmetic that more waves hid).  64-thread
// workgroups, 12: 1049, 933; 24: 832, 729; 256-thread ones, 6: 843, 706.  Tiles in
// the dispatcher's order, 128 x 12: 853, 733.  Whole steps, 16 against 12: 20M
// 150.5 -> 149.3, 94M 640 -> 634, 150M 1007 -> 987, 250M 1657 -> 1644.  (10 for the
// apply pass alone gains on 250M and costs 8 us on 94M.)
// ---------------------------------------------------------------------------
namespace {
constexpr int kLambBlock = 128, kLambUnroll = 1, kLambPerCU = 12;
constexpr bool kLambNTL = true, kLambNTS = true, kLambXCD = true;
constexpr int64_t kLambTile = 4 * (int64_t)kLambBlock * kLambUnroll;  // elements per tile
constexpr int64_t kLambMaxBlocks = 1 << 26;
// The event after a call orders streams of one device, for which a device-scope
// release is enough; up to this many elements leaving out the system-scope one
// pays (5.9M: 54.4 against 56.1 us a step), on larger shards it costs a little
// (20M: 150.2 against 147.9; 94M: 629 against 626).
constexpr int64_t kLambNoFenceNumel = 1 << 23;
constexpr int kHeads = zs::kMaxHead + 1;  // one work list per head (elements before the master array's first cache line)
}  // namespace

using namespace zsh;

constexpr int kLambSmallV[3] = {1, 2, 4};  // tiles per workgroup of the one-launch step
constexpr int64_t kLambSmallNumel =
    4 * (int64_t)zs::kLambSmallBlock * 4 * zs::kSmallSlots + zs::kMaxHead + 3;  // the most it can take

// The work lists of the one-launch step for one array alignment, on the device:
// the layer pieces of its workgroups (with the end sentinel), the first piece of
// every workgroup and of every layer (each list with its end sentinel).
struct LambSmall {
    zs::LambItem* items = nullptr;   // start of the one allocation behind the three lists
    int64_t* wg_first = nullptr;
    int64_t* layer_first = nullptr;
    int v = 0;                       // tiles per workgroup (0: the shard does not fit)
    unsigned grid = 0;
    bool built = false;
};

// The work lists of one array alignment, on the device: the items (tile pieces
// inside one layer, with the end sentinel), the first item of every tile, the
// chunks of the layer sums (item ranges inside one layer), each chunk's layer
// and the first chunk of every layer (the ranges with their end sentinels).
struct LambWork {
    unsigned char* base = nullptr;   // the one allocation behind the lists
    zs::LambItem* items = nullptr;
    int64_t* tile_first = nullptr;
    int64_t* chunk = nullptr;
    int32_t* chunk_layer = nullptr;
    int64_t* chunk_first = nullptr;
    int64_t n_items = 0, ntiles = 0, n_chunks = 0;
    bool built = false;
};

struct LambProfRec {
    hipEvent_t e[5];
};

// Per-device launch facts, computed once per device: the occupancy reservations
// of the moments and apply kernels and the workgroups of k_lamb_small<1, 2, 4>
// that a launch may take.
struct LambDev {
    size_t lds[2] = {0, 0};
    int64_t small_most[3] = {};
    bool ready = false;
};

struct zero_lamb_plan {
    std::mutex mu;
    int dev = 0;
    int64_t n = 0;
    int32_t n_seg = 0;
    std::vector<int64_t> seg_off;
    LambWork work[kHeads];
    LambSmall small[kHeads];
    Slots small_slots;               // exchange slots of the one-launch step (n at most kLambSmallNumel)
    unsigned char* ws = nullptr;     // the one allocation behind the next four
    zs::LayerSums* part = nullptr;   // one partial per item (sized for the longest list)
    uint64_t* slots = nullptr;       // two exchange slots per chunk
    bool slots_ready = false;        // the slots have been zeroed
    zs::LayerSums* sums = nullptr;   // per-layer sums of zero_lamb_step
    int64_t max_items = 0, max_chunks = 0;
    hipEvent_t done = nullptr;       // recorded after each call's kernels (ordering across streams)
    hipStream_t last_stream = nullptr;
    bool used = false;
    uint64_t prof_tick = 0;
    const LambDev* facts = nullptr;
};

namespace {

std::mutex g_lprof_mu;
std::vector<LambProfRec> g_lprof_pending;
std::vector<hipEvent_t> g_lprof_pool;
zero_lamb_profile_t g_lprof_acc = {0, 0.0, 0.0, 0.0, 0.0};

const void* moments_kernel() {
    return reinterpret_cast<const void*>(zs::k_lamb_moments<kLambBlock, kLambUnroll, kLambNTL, kLambNTS, kLambXCD, zs::FromResult>);
}
template <int PASS>
const void* probe_kernel() {
    return reinterpret_cast<const void*>(zs::k_probe_lamb<kLambBlock, kLambUnroll, kLambNTL, kLambNTS, kLambXCD, PASS>);
}
const void* apply_kernel() {
    return reinterpret_cast<const void*>(zs::k_lamb_apply<kLambBlock, kLambUnroll, kLambNTL, kLambNTS, kLambXCD, zs::FromResult>);
}

// Upper bound on the items of any alignment: one per tile the shard touches
// (at most n/T + 2, counting the partial tile below the first aligned vector)
// plus one per interior layer boundary.
int64_t max_items_for(int64_t n, int32_t n_seg) { return n / kLambTile + 2 + (int64_t)n_seg; }

// Chunks: each layer's items cut into runs of at most kChunkItems.
int64_t max_chunks_for(int64_t max_items, int32_t n_seg) { return max_items / zs::kChunkItems + 1 + (int64_t)n_seg; }

// Tiles (as the kernels' tile_range defines them): [0, head) when head > 0,
// then runs of kLambTile elements from head on.
int64_t tile_of(int64_t pos, int64_t head) {
    const int64_t hs = head > 0 ? 1 : 0;
    return pos < head ? 0 : hs + (pos - head) / kLambTile;
}

int64_t tile_count(int64_t n, int64_t head) {
    if (n == 0)
        return 0;
    const int64_t hs = head > 0 ? 1 : 0;
    return n > head ? hs + (n - head + kLambTile - 1) / kLambTile : 1;
}

// The part of a work list that has an entry per layer or chunk; k_lamb_items
// makes the part that has one per tile.
struct HostWork {
    int64_t ntiles = 0, n_items = 0;
    std::vector<int64_t> inner;       // n_seg: the layers 1..s that begin inside a tile
    std::vector<int64_t> chunk;       // n_chunks + 1 item indices
    std::vector<int32_t> chunk_layer; // n_chunks layers
    std::vector<int64_t> chunk_first; // n_seg + 1 chunk indices
};

// [0, n), n > 0, is cut at the tile boundaries and at the layer boundaries.  The
// items before a position are the tiles and the layers inside tiles that begin
// before it, which gives each layer's item range without a list of the items.
void build_work(const std::vector<int64_t>& off, int32_t n_seg, int64_t head, HostWork* w) {
    w->ntiles = tile_count(off[n_seg], head);
    w->inner.assign((size_t)n_seg, 0);
    std::vector<int64_t> first((size_t)n_seg + 1, 0);
    for (int32_t s = 1; s < n_seg; ++s) {
        const bool inside = off[s] < head || (off[s] - head) % kLambTile != 0;
        first[s] = tile_of(off[s], head) + (inside ? 1 : 0) + w->inner[s - 1];
        w->inner[s] = w->inner[s - 1] + (inside ? 1 : 0);
    }
    w->n_items = first[n_seg] = w->ntiles + w->inner[n_seg - 1];
    w->chunk.clear();
    w->chunk_layer.clear();
    w->chunk_first.assign((size_t)n_seg + 1, 0);
    for (int32_t s = 0; s < n_seg; ++s) {
        w->chunk_first[s] = (int64_t)w->chunk.size();
        for (int64_t k = first[s]; k < first[s + 1]; k += zs::kChunkItems) {
            w->chunk.push_back(k);
            w->chunk_layer.push_back(s);
        }
    }
    w->chunk_first[n_seg] = (int64_t)w->chunk.size();
    w->chunk.push_back(w->n_items);
}

// Host lists packed for one allocation and one copy to the device (each list on
// a 16-byte boundary).
struct Packer {
    std::vector<unsigned char> bytes;
    template <typename T>
    size_t add(const std::vector<T>& h) {
        const size_t at = (bytes.size() + 15) / 16 * 16;
        bytes.resize(at + h.size() * sizeof(T));
        if (!h.empty())
            std::memcpy(bytes.data() + at, h.data(), h.size() * sizeof(T));
        return at;
    }
    // Device memory for the packed lists and `more` bytes after them; the copy is queued on `stream`.
    int upload(unsigned char** d, size_t more, hipStream_t stream) const {
        if (hipMalloc(reinterpret_cast<void**>(d), bytes.size() + more) != hipSuccess) {
            *d = nullptr;
            (void)hipGetLastError();
            return fail(ZERO_ENOMEM, "zero_lamb: could not allocate work lists of %zu bytes", bytes.size() + more);
        }
        const hipError_t e = hipMemcpyAsync(*d, bytes.data(), bytes.size(), hipMemcpyHostToDevice, stream);
        if (e != hipSuccess) {
            (void)hipFree(*d);
            *d = nullptr;
            return fail(ZERO_EHIP, "zero_lamb: copying work lists: %s", hipGetErrorString(e));
        }
        return ZERO_OK;
    }
};

// The work list of `head`, made on first use: the short lists on the host, the
// items on the device.  Made on the host, the items of a 250M shard are 12 MB to
// fill, pack and upload: a plan's first step took 9.6 ms there (3.4 ms without the
// packing) and 3.6 ms (1.4) on 94M; now 1.8 and 0.75 ms, where a later step takes
// 1.66 and 0.63.  Split phase on 5.9M: 0.28 -> 0.12 ms.  There is a list for each
// of kHeads positions of the master array in its line, so a captured call may be
// the first at its position however many the plan has served: a list is made
// during a capture, too.  Caller holds plan->mu.
int get_work(zero_lamb_plan* plan, int head, hipStream_t stream, LambWork** out) {
    LambWork& w = plan->work[head];
    if (!w.built) {
        HostWork h;
        build_work(plan->seg_off, plan->n_seg, head, &h);
        const int64_t n_chunks = (int64_t)h.chunk.size() - 1;
        if (h.n_items > plan->max_items || n_chunks > plan->max_chunks)
            return fail(ZERO_EHIP, "zero_lamb: work lists (%lld items, %lld chunks) exceed their bounds",
                        (long long)h.n_items, (long long)n_chunks);
        Packer pk;
        const size_t at[5] = {pk.add(plan->seg_off), pk.add(h.inner), pk.add(h.chunk), pk.add(h.chunk_layer),
                              pk.add(h.chunk_first)};
        pk.bytes.resize((pk.bytes.size() + 15) / 16 * 16);
        const size_t items = pk.bytes.size(), tiles = items + (size_t)(h.n_items + 1) * sizeof(zs::LambItem);
        // on the null stream and waited for: any stream may use the lists next.  While `stream` is being
        // captured the null stream may not be used: a stream of their own then
        RelaxedCapture relaxed(stream);
        hipStream_t on = nullptr;
        if (relaxed.on)
            HIP_TRY(hipStreamCreateWithFlags(&on, hipStreamNonBlocking));
        unsigned char* d = nullptr;
        int rc = pk.upload(&d, tiles - items + (size_t)(h.ntiles + 1) * sizeof(int64_t), on);
        if (!rc) {
            const unsigned grid = (unsigned)((h.ntiles + zs::kItemsBlock) / zs::kItemsBlock);
            zs::k_lamb_items<<<grid, zs::kItemsBlock, 0, on>>>(
                reinterpret_cast<const int64_t*>(d + at[0]), reinterpret_cast<const int64_t*>(d + at[1]),
                plan->n_seg, (int64_t)head, h.ntiles, kLambTile, reinterpret_cast<zs::LambItem*>(d + items),
                reinterpret_cast<int64_t*>(d + tiles));
            hipError_t e = hipGetLastError();
            if (e == hipSuccess)
                e = hipStreamSynchronize(on);
            if (e != hipSuccess) {
                (void)hipFree(d);
                rc = fail(ZERO_EHIP, "zero_lamb: making work lists: %s", hipGetErrorString(e));
            }
        }
        if (on)
            (void)hipStreamDestroy(on);
        if (rc)
            return rc;
        w.base = d;
        w.items = reinterpret_cast<zs::LambItem*>(d + items);
        w.tile_first = reinterpret_cast<int64_t*>(d + tiles);
        w.chunk = reinterpret_cast<int64_t*>(d + at[2]);
        w.chunk_layer = reinterpret_cast<int32_t*>(d + at[3]);
        w.chunk_first = reinterpret_cast<int64_t*>(d + at[4]);
        w.n_items = h.n_items;
        w.ntiles = h.ntiles;
        w.n_chunks = n_chunks;
        w.built = true;
    }
    *out = &w;
    return ZERO_OK;
}

const void* small_kernel(int v) {
    switch (v) {
    case 1: return reinterpret_cast<const void*>(zs::k_lamb_small<1>);
    case 2: return reinterpret_cast<const void*>(zs::k_lamb_small<2>);
    default: return reinterpret_cast<const void*>(zs::k_lamb_small<4>);
    }
}

std::mutex g_lamb_dev_mu;
LambDev g_lamb_dev[kMaxDevices];

// The facts of device `dev`, filled on first use.
int lamb_dev(int dev, const LambDev** out) {
    const DevInfo* info = nullptr;
    const int rc = dev_info(dev, &info);  // checks dev
    if (rc)
        return rc;
    std::lock_guard<std::mutex> lk(g_lamb_dev_mu);
    LambDev& d = g_lamb_dev[dev];
    if (!d.ready) {
        hipDeviceProp_t prop;
        HIP_TRY(hipGetDeviceProperties(&prop, dev));
        int resident = 0;
        d.lds[0] = occupancy_lds(moments_kernel(), kLambBlock, kLambPerCU, prop, &resident);
        d.lds[1] = occupancy_lds(apply_kernel(), kLambBlock, kLambPerCU, prop, &resident);
        for (int k = 0; k < 3; ++k) {
            int per_cu = 0;
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, small_kernel(kLambSmallV[k]),
                                                             zs::kLambSmallBlock, 0) != hipSuccess) {
                (void)hipGetLastError();
                per_cu = 0;
            }
            d.small_most[k] = std::min<int64_t>(zs::kSmallSlots, (int64_t)per_cu * info->ncu / info->small_share);
        }
        d.ready = true;
    }
    *out = &d;
    return ZERO_OK;
}

// The one-launch step's shape and work lists for `head`, decided and uploaded
// on first use: the fewest tiles per workgroup whose grid fits the exchange slots
// and the plan's share of the device, if no workgroup meets more than kLambPieces
// layer pieces (v = 0 otherwise).  Caller holds plan->mu.
int get_small(zero_lamb_plan* plan, int head, LambSmall** out) {
    LambSmall& w = plan->small[head];
    *out = &w;
    if (w.built)
        return ZERO_OK;
    const int64_t n = plan->n, nvec = n > head ? (n - head) / 4 : 0;
    int v = 0;
    int64_t grid = 0;
    for (int k = 0; k < 3 && !v && plan->small_slots.words; ++k) {
        grid = (nvec + zs::kLambSmallBlock * kLambSmallV[k] - 1) / (zs::kLambSmallBlock * kLambSmallV[k]);
        grid = grid < 1 ? 1 : grid;
        if (grid <= plan->facts->small_most[k])
            v = kLambSmallV[k];
    }
    if (v) {
        const int64_t span = 4 * (int64_t)zs::kLambSmallBlock * v;
        std::vector<zs::LambItem> items;
        std::vector<int64_t> wg_first, layer_first((size_t)plan->n_seg + 1, 0);
        int32_t s = 0;       // the layer at pos
        int64_t pos = 0;
        for (int64_t b = 0; b < grid && v; ++b) {
            const int64_t end = b == grid - 1 ? n : head + span * (b + 1);
            wg_first.push_back((int64_t)items.size());
            while (pos < end) {
                if (pos == plan->seg_off[s])
                    layer_first[s] = (int64_t)items.size();
                items.push_back(zs::LambItem{pos, s, 0});
                pos = plan->seg_off[s + 1] < end ? plan->seg_off[s + 1] : end;
                if (pos == plan->seg_off[s + 1])
                    ++s;
            }
            if ((int64_t)items.size() - wg_first.back() > zs::kLambPieces ||
                (int64_t)items.size() > zs::kLambSmallItems)
                v = 0;
        }
        if (v) {
            wg_first.push_back((int64_t)items.size());
            layer_first[plan->n_seg] = (int64_t)items.size();
            items.push_back(zs::LambItem{n, -1, 0});
            Packer pk;
            const size_t at[3] = {pk.add(items), pk.add(wg_first), pk.add(layer_first)};
            unsigned char* d = nullptr;
            const int rc = pk.upload(&d, 0, nullptr);
            if (rc)
                return rc;
            if (hipStreamSynchronize(nullptr) != hipSuccess) {
                (void)hipFree(d);
                return fail(ZERO_EHIP, "zero_lamb: copying work lists failed");
            }
            w.items = reinterpret_cast<zs::LambItem*>(d + at[0]);
            w.wg_first = reinterpret_cast<int64_t*>(d + at[1]);
            w.layer_first = reinterpret_cast<int64_t*>(d + at[2]);
        }
    }
    w.v = v;
    w.grid = (unsigned)grid;
    w.built = true;
    return ZERO_OK;
}

int check_plan(const char* fn, const zero_lamb_plan_t* plan) {
    if (!plan)
        return fail(ZERO_EINVAL, "%s: NULL plan", fn);
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev != plan->dev)
        return fail(ZERO_EINVAL, "%s: plan was created on device %d, current device is %d", fn, plan->dev, dev);
    return ZERO_OK;
}

int check_phi(const char* fn, double phi_lo, double phi_hi) {
    if (std::isnan(phi_lo) || std::isnan(phi_hi) || !(phi_lo >= 0.0) || !(phi_hi >= phi_lo) || std::isinf(phi_lo))
        return fail(ZERO_EINVAL, "%s: need 0 <= phi_lo <= phi_hi (phi_hi may be +inf)", fn);
    return ZERO_OK;
}

// Alignment, NULL, overlap and allocation checks of the arrays a call touches
// (NULL entries of ptrs are arrays the call does not take).
int check_lamb_arrays(const char* fn, const void* const ptrs[5], int64_t n) {
    static const size_t esz[5] = {2, 4, 4, 4, 2};
    size_t bytes[5];
    const void* live[5];
    size_t live_bytes[5];
    int k = 0;
    for (int i = 0; i < 5; ++i) {
        bytes[i] = esz[i] * (size_t)n;
        if (!ptrs[i])
            continue;
        if (reinterpret_cast<uintptr_t>(ptrs[i]) % esz[i])
            return fail(ZERO_EINVAL, "%s: array %d is not %zu-byte aligned", fn, i, esz[i]);
        live[k] = ptrs[i];
        live_bytes[k] = bytes[i];
        ++k;
    }
    if (n == 0)
        return ZERO_OK;
    for (int i = 0; i < 5; ++i)
        for (int j = i + 1; j < 5; ++j)
            if (ptrs[i] && ptrs[j] &&
                overlaps(reinterpret_cast<uintptr_t>(ptrs[i]), bytes[i], reinterpret_cast<uintptr_t>(ptrs[j]),
                         bytes[j]))
                return fail(ZERO_EINVAL, "%s: arrays %d and %d overlap", fn, i, j);
    return check_ranges(fn, live, live_bytes, k);
}

int check_layer_sums(const char* fn, const zero_lamb_plan_t* plan, const void* layer_sumsq,
                     const void* const arrays[5]) {
    if (!layer_sumsq || reinterpret_cast<uintptr_t>(layer_sumsq) % 16)
        return fail(ZERO_EINVAL, "%s: layer_sumsq must be a 16-byte aligned device array", fn);
    const size_t bytes = 16 * (size_t)plan->n_seg;
    for (int i = 0; i < 5; ++i)
        if (arrays[i] && overlaps(reinterpret_cast<uintptr_t>(arrays[i]), (i == 0 || i == 4 ? 2 : 4) * (size_t)plan->n,
                                  reinterpret_cast<uintptr_t>(layer_sumsq), bytes))
            return fail(ZERO_EINVAL, "%s: layer_sumsq overlaps array %d", fn, i);
    return check_ranges(fn, &layer_sumsq, &bytes, 1);
}

// Work queued on the plan's previous stream must finish before another
// stream reuses the plan's partials and sums: the new stream waits (on the
// device) for the event recorded after the plan's last call.  The event stays
// valid after that stream is destroyed, and no other stream or the host waits.
int switch_stream(zero_lamb_plan* plan, hipStream_t stream) {
    if (plan->used && plan->last_stream != stream)
        HIP_TRY(hipStreamWaitEvent(stream, plan->done, 0));
    plan->used = true;
    plan->last_stream = stream;
    return ZERO_OK;
}

// The launch of a call's last kernel, whose completion is the event `done` (see
// switch_stream).  The kernel's own completion signal serves as the event: a
// record after it puts a marker into the stream (1M elements: 23.4 us a step
// against 25.9; the split phase, two calls a step, on 5.9M: 64.3 against 69.9).
// A stream that is being captured takes the record (a captured launch carries
// no event).
template <typename F, typename... A>
int launch_last(zero_lamb_plan* plan, F* kernel, unsigned grid, int block, size_t lds, hipStream_t stream, A... args) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    HIP_TRY(hipStreamIsCapturing(stream, &cap));
    if (cap == hipStreamCaptureStatusNone) {
        hipExtLaunchKernelGGL(kernel, dim3(grid), dim3((unsigned)block), (uint32_t)lds, stream, nullptr, plan->done, 0,
                              args...);
        HIP_TRY(hipGetLastError());
    } else {
        kernel<<<grid, block, lds, stream>>>(args...);
        HIP_TRY(hipGetLastError());
        HIP_TRY(hipEventRecord(plan->done, stream));
    }
    return ZERO_OK;
}

// Grid of the tile passes: a multiple of 8 (the XCD count) so that the XCD
// remapping of workgroups is a bijection; the extra workgroups find no tile.
unsigned tile_grid(int64_t ntiles) {
    int64_t b = ntiles < 1 ? 1 : ntiles;
    b = b > kLambMaxBlocks ? kLambMaxBlocks : b;
    return (unsigned)((b + 7) / 8 * 8);
}

template <typename SRC>
int launch_moments(zero_lamb_plan* plan, const LambWork& w, int head, const uint16_t* g, const float* th, float* m,
                   float* v, const SRC& src, hipStream_t stream) {
    zs::k_lamb_moments<kLambBlock, kLambUnroll, kLambNTL, kLambNTS, kLambXCD, SRC>
        <<<tile_grid(w.ntiles), kLambBlock, plan->facts->lds[0], stream>>>(g, th, m, v, w.items, w.tile_first, w.ntiles,
                                                                    plan->n, head, src, plan->part);
    HIP_TRY(hipGetLastError());
    return ZERO_OK;
}

// The layer sums into `sums`; `res`: the record whose skip flag applies, or NULL.
int launch_sums(zero_lamb_plan* plan, const LambWork& w, zs::LayerSums* sums, const zs::Result* res, bool last,
                hipStream_t stream) {
    const int rc = ready_slots(plan->slots, 2 * plan->max_chunks, &plan->slots_ready, stream);
    if (rc)
        return rc;
    const unsigned grid = (unsigned)w.n_chunks;
    if (last)
        return launch_last(plan, zs::k_lamb_sums, grid, zs::kChunkBlock, 0, stream, (const zs::LayerSums*)plan->part,
                           (const int64_t*)w.chunk, (const int32_t*)w.chunk_layer, (const int64_t*)w.chunk_first,
                           plan->slots, sums, res);
    zs::k_lamb_sums<<<grid, zs::kChunkBlock, 0, stream>>>(plan->part, w.chunk, w.chunk_layer, w.chunk_first,
                                                          plan->slots, sums, res);
    HIP_TRY(hipGetLastError());
    return ZERO_OK;
}

template <typename SRC>
int launch_apply(zero_lamb_plan* plan, const LambWork& w, int head, float* th, const float* m, const float* v,
                 uint16_t* p, const zs::LayerSums* sums, const SRC& src, double lr, double phi_lo, double phi_hi,
                 hipStream_t stream) {
    return launch_last(plan, zs::k_lamb_apply<kLambBlock, kLambUnroll, kLambNTL, kLambNTS, kLambXCD, SRC>,
                       tile_grid(w.ntiles), kLambBlock, plan->facts->lds[1], stream, th, m, v, p,
                       (const zs::LambItem*)w.items, (const int64_t*)w.tile_first, w.ntiles, plan->n, (int64_t)head,
                       sums, src, lr, phi_lo, phi_hi);
}

// The one-launch step.
int launch_small(zero_lamb_plan* plan, const LambSmall& w, int head, const uint16_t* g, float* th, float* m, float* v,
                 uint16_t* p, uint64_t* host_dev, double loss_scale, double clip, uint32_t seq, const zs::AdamConst& c,
                 double lr, double phi_lo, double phi_hi, hipStream_t stream) {
    Slots& sl = plan->small_slots;
    int rc = ready_slots(sl.words, 2 * zs::kLambSmallWords, &sl.ready, stream);
    if (rc)
        return rc;
    uint64_t* const set = sl.words + sl.set * zs::kLambSmallWords;
    uint64_t* const other = sl.words + (1 - sl.set) * zs::kLambSmallWords;
    const int n = (int)plan->n, h = head < n ? head : n, nvec = (n - h) / 4;
    const auto launch = [&](auto kernel) {
        return launch_last(plan, kernel, w.grid, zs::kLambSmallBlock, 0, stream, g, th, m, v, p, n, h, nvec,
                           (const zs::LambItem*)w.items, (const int64_t*)w.wg_first, (const int64_t*)w.layer_first,
                           set, other, host_dev, loss_scale, clip, seq, c, lr, phi_lo, phi_hi);
    };
    rc = w.v == 1   ? launch(zs::k_lamb_small<1>)
         : w.v == 2 ? launch(zs::k_lamb_small<2>)
                    : launch(zs::k_lamb_small<4>);
    if (!rc)
        sl.set = 1 - sl.set;
    return rc;
}

hipEvent_t lprof_event() {
    if (!g_lprof_pool.empty()) {
        hipEvent_t e = g_lprof_pool.back();
        g_lprof_pool.pop_back();
        return e;
    }
    hipEvent_t e = nullptr;
    return hipEventCreate(&e) == hipSuccess ? e : nullptr;
}

// Events of one sampled step, or false when this step is not sampled (or an
// event could not be created).  Caller holds plan->mu.
bool lprof_begin(zero_lamb_plan* plan, LambProfRec* rec) {
    const int every = prof_every();
    if (every <= 0 || plan->prof_tick++ % (uint64_t)every != 0)
        return false;
    std::lock_guard<std::mutex> lk(g_lprof_mu);
    bool ok = true;
    for (int i = 0; i < 5; ++i) {
        rec->e[i] = lprof_event();
        ok = ok && rec->e[i];
    }
    if (!ok) {
        for (int i = 0; i < 5; ++i)
            if (rec->e[i])
                g_lprof_pool.push_back(rec->e[i]);
        return false;
    }
    return true;
}

void lprof_drain_locked() {
    for (LambProfRec& r : g_lprof_pending) {
        hipError_t e = hipEventSynchronize(r.e[4]);
        float t[4] = {0.f, 0.f, 0.f, 0.f};
        for (int i = 0; i < 4 && e == hipSuccess; ++i)
            e = hipEventElapsedTime(&t[i], r.e[i], r.e[i + 1]);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            prof_defer_error(1, "reading LAMB step events", e);
            continue;
        }
        g_lprof_acc.steps += 1;
        g_lprof_acc.stats_ms += t[0];
        g_lprof_acc.moments_ms += t[1];
        g_lprof_acc.layer_ms += t[2];
        g_lprof_acc.apply_ms += t[3];
    }
    for (LambProfRec& r : g_lprof_pending)
        for (int i = 0; i < 5; ++i)
            g_lprof_pool.push_back(r.e[i]);
    g_lprof_pending.clear();
}

// Records event i of a sampled step; a failure drops the sample (deferred error).
void lprof_record(LambProfRec* rec, bool* ok, int i, hipStream_t stream) {
    if (!*ok)
        return;
    const hipError_t e = hipEventRecord(rec->e[i], stream);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        *ok = false;
        prof_defer_error(1, "hipEventRecord", e);
    }
}

// Queues a sampled step's record for the next read, or returns its events to
// the pool when a record failed.
void lprof_end(const LambProfRec& rec, bool ok) {
    std::lock_guard<std::mutex> lk(g_lprof_mu);
    if (!ok) {
        for (int i = 0; i < 5; ++i)
            g_lprof_pool.push_back(rec.e[i]);
        return;
    }
    g_lprof_pending.push_back(rec);
    if (g_lprof_pending.size() >= 4096)
        lprof_drain_locked();
}

void set_last_stats(const zs::Result& r, int64_t n, int32_t path) {
    t_stats.sumsq = r.sumsq;
    t_stats.norm = r.norm;
    t_stats.coef = r.coef;
    t_stats.mult = r.mult;
    t_stats.overflow = r.overflow;
    t_stats.skipped = r.skip;
    t_stats.path = path;
    t_stats.n = n;
    t_have_stats = true;
}

void free_plan(zero_lamb_plan* p) {
    for (LambWork& w : p->work)
        if (w.base) (void)hipFree(w.base);
    for (LambSmall& w : p->small)
        if (w.items) (void)hipFree(w.items);
    if (p->ws) (void)hipFree(p->ws);
    if (p->done) (void)hipEventDestroy(p->done);
}

}  // namespace

extern "C" {

int zero_lamb_plan_create(const int64_t* seg_off, int32_t n_seg, int64_t n, zero_lamb_plan_t** out) {
    if (!out)
        return fail(ZERO_EINVAL, "zero_lamb_plan_create: NULL out");
    *out = nullptr;
    if (n < 0 || n > kMaxNumel)
        return fail(ZERO_EINVAL, "zero_lamb_plan_create: n=%lld outside [0, 2^40]", (long long)n);
    if (n_seg < 0 || (n == 0) != (n_seg == 0))
        return fail(ZERO_EINVAL, "zero_lamb_plan_create: need n_seg > 0 for n > 0 and n_seg = 0 for n = 0");
    if (n_seg > 0) {
        if (!seg_off)
            return fail(ZERO_EINVAL, "zero_lamb_plan_create: NULL seg_off");
        if (seg_off[0] != 0 || seg_off[n_seg] != n)
            return fail(ZERO_EINVAL, "zero_lamb_plan_create: seg_off must start at 0 and end at n");
        for (int32_t s = 0; s < n_seg; ++s)
            if (seg_off[s + 1] <= seg_off[s])
                return fail(ZERO_EINVAL, "zero_lamb_plan_create: seg_off must rise strictly (layer %d)", s);
    }
    std::unique_ptr<zero_lamb_plan> p(new zero_lamb_plan);
    HIP_TRY(hipGetDevice(&p->dev));
    p->n = n;
    p->n_seg = n_seg;
    if (n_seg > 0)
        p->seg_off.assign(seg_off, seg_off + n_seg + 1);
    else
        p->seg_off.assign(1, 0);
    p->max_items = max_items_for(n, n_seg);
    p->max_chunks = max_chunks_for(p->max_items, n_seg);
    const unsigned fence = n <= kLambNoFenceNumel ? hipEventDisableSystemFence : 0;
    if (hipEventCreateWithFlags(&p->done, hipEventDisableTiming | fence) != hipSuccess) {
        p->done = nullptr;
        (void)hipGetLastError();
        return fail(ZERO_EHIP, "zero_lamb_plan_create: could not create the plan's event");
    }
    if (n > 0) {
        int rc = lamb_dev(p->dev, &p->facts);
        const bool small = n <= kLambSmallNumel;
        const size_t part = 0, sums = part + (size_t)p->max_items * sizeof(zs::LayerSums),
                     slots = sums + (size_t)n_seg * sizeof(zs::LayerSums),
                     small_slots = slots + (size_t)p->max_chunks * 2 * sizeof(uint64_t),
                     bytes = small_slots + (small ? 2 * zs::kLambSmallWords * sizeof(uint64_t) : 0);
        if (!rc && hipMalloc(reinterpret_cast<void**>(&p->ws), bytes) != hipSuccess) {
            p->ws = nullptr;
            (void)hipGetLastError();
            rc = fail(ZERO_ENOMEM, "zero_lamb_plan_create: could not allocate the plan workspace");
        }
        if (rc) {
            free_plan(p.get());
            return rc;
        }
        p->part = reinterpret_cast<zs::LayerSums*>(p->ws + part);
        p->sums = reinterpret_cast<zs::LayerSums*>(p->ws + sums);
        p->slots = reinterpret_cast<uint64_t*>(p->ws + slots);
        p->small_slots.words = small ? reinterpret_cast<uint64_t*>(p->ws + small_slots) : nullptr;
    }
    *out = p.release();
    return ZERO_OK;
}

int zero_lamb_plan_destroy(zero_lamb_plan_t* plan) {
    if (!plan)
        return ZERO_OK;
    int rc = ZERO_OK;
    {
        std::lock_guard<std::mutex> lk(plan->mu);
        int cur = 0;
        if (hipGetDevice(&cur) == hipSuccess && cur != plan->dev)
            (void)hipSetDevice(plan->dev);
        // the plan's last call recorded `done` after its kernels, and every call waited
        // for the previous one's, so this waits for all of the plan's work
        if (plan->used && hipEventSynchronize(plan->done) != hipSuccess) {
            (void)hipGetLastError();
            rc = fail(ZERO_EHIP, "zero_lamb_plan_destroy: waiting for the plan's work failed");
        }
        free_plan(plan);
        if (cur != plan->dev)
            (void)hipSetDevice(cur);
    }
    delete plan;
    return rc;
}

int zero_lamb_step(const zero_lamb_plan_t* plan_, const uint16_t* grad16, float* master32, float* m32, float* v32,
                   uint16_t* param16_out, double lr, double beta1, double beta2, double eps, double weight_decay,
                   int64_t step, double loss_scale, double clip, double phi_lo, double phi_hi, void* stream_) {
    const char* fn = "zero_lamb_step";
    zero_lamb_plan* plan = const_cast<zero_lamb_plan*>(plan_);
    int rc = check_plan(fn, plan);
    if (rc || (rc = check_hyper(fn, lr, beta1, beta2, eps, weight_decay, step, loss_scale, clip)) ||
        (rc = check_phi(fn, phi_lo, phi_hi)))
        return rc;
    const int64_t n = plan->n;
    if (n > 0 && (!grad16 || !master32 || !m32 || !v32 || !param16_out))
        return fail(ZERO_EINVAL, "%s: NULL array with n > 0", fn);
    const void* arrays[5] = {grad16, master32, m32, v32, param16_out};
    if ((rc = check_lamb_arrays(fn, arrays, n)))
        return rc;
    if (n == 0) {
        t_stats = zero_step_stats_t{0.0, 0.0, 1.0, (float)(1.0 / loss_scale), 0, 0, 0, 0};
        t_have_stats = true;
        return ZERO_OK;
    }
    hipStream_t stream = reinterpret_cast<hipStream_t>(stream_);
    std::lock_guard<std::mutex> plk(plan->mu);
    CtxLock ctx;
    if ((rc = lock_ctx(stream, &ctx)))
        return rc;
    const int head = (int)line_head(master32, sizeof(float));
    LambSmall* sm = nullptr;
    LambWork* w = nullptr;
    if ((rc = get_small(plan, head, &sm)) || (!sm->v && (rc = get_work(plan, head, stream, &w))) ||
        (rc = switch_stream(plan, stream)))
        return rc;
    const zs::AdamConst c = adam_const(lr, beta1, beta2, eps, weight_decay, step);
    const zs::FromResult src{ctx->res, c};
    zs::Result r;
    bool given_up = false;
    const auto attempt = [&](bool small) -> int {
        const uint32_t seq = next_seq(ctx.get());
        LambProfRec pr;
        bool prof = lprof_begin(plan, &pr);
        const bool sampled = prof;
        int e = ZERO_OK;
        lprof_record(&pr, &prof, 0, stream);
        if (!small)
            e = launch_stats_planned(ctx.get(), grad16, n, loss_scale, clip, seq, stream);
        lprof_record(&pr, &prof, 1, stream);
        if (!e && !small)
            e = launch_moments(plan, *w, head, grad16, master32, m32, v32, src, stream);
        lprof_record(&pr, &prof, 2, stream);
        if (!e && !small)
            e = launch_sums(plan, *w, plan->sums, ctx->res, false, stream);
        lprof_record(&pr, &prof, 3, stream);
        if (!e && small)
            e = launch_small(plan, *sm, head, grad16, master32, m32, v32, param16_out, ctx->host_dev, loss_scale, clip,
                             seq, c, lr, phi_lo, phi_hi, stream);
        else if (!e)
            e = launch_apply(plan, *w, head, master32, m32, v32, param16_out, plan->sums, src, lr, phi_lo, phi_hi,
                             stream);
        lprof_record(&pr, &prof, 4, stream);
        if (sampled)
            lprof_end(pr, prof && !e);
        if (e) {
            (void)hipEventRecord(plan->done, stream);  // what was queued before the failure
            return e;
        }
        return wait_result(ctx.get(), seq, stream, loss_scale, clip, &r, &given_up);
    };
    bool small = sm->v != 0;
    rc = attempt(small);
    if (rc && given_up && small) {
        // the device did not run the one-launch grid together: its slots are emptied before the next
        // launch, and the kernel sequence, which needs no such thing, takes the step
        plan->small_slots.ready = small = false;
        if (!(rc = get_work(plan, head, stream, &w)))
            rc = attempt(false);
    }
    if (rc)
        return rc;
    set_last_stats(r, n, small ? 1 : 0);
    return r.skip ? ZERO_SKIPPED : ZERO_OK;
}

int zero_lamb_moments(const zero_lamb_plan_t* plan_, const uint16_t* grad16, const float* master32, float* m32,
                      float* v32, double global_sumsq, double beta1, double beta2, double eps, double weight_decay,
                      int64_t step, double loss_scale, double clip, double* layer_sumsq, void* stream_) {
    const char* fn = "zero_lamb_moments";
    zero_lamb_plan* plan = const_cast<zero_lamb_plan*>(plan_);
    int rc = check_plan(fn, plan);
    if (rc || (rc = check_hyper(fn, 0.0, beta1, beta2, eps, weight_decay, step, loss_scale, clip)))
        return rc;
    if (std::isnan(global_sumsq) || global_sumsq < 0.0)
        return fail(ZERO_EINVAL, "%s: global_sumsq must be >= 0 (+inf for an overflow)", fn);
    const int64_t n = plan->n;
    if (n > 0 && (!grad16 || !master32 || !m32 || !v32))
        return fail(ZERO_EINVAL, "%s: NULL array with n > 0", fn);
    const void* arrays[5] = {grad16, master32, m32, v32, nullptr};
    if ((rc = check_lamb_arrays(fn, arrays, n)))
        return rc;
    if (n > 0 && (rc = check_layer_sums(fn, plan, layer_sumsq, arrays)))
        return rc;
    if (!std::isfinite(global_sumsq))
        return ZERO_SKIPPED;
    if (n == 0)
        return ZERO_OK;
    hipStream_t stream = reinterpret_cast<hipStream_t>(stream_);
    std::lock_guard<std::mutex> plk(plan->mu);
    CtxLock ctx;
    if ((rc = lock_ctx(stream, &ctx)))
        return rc;
    const int head = (int)line_head(master32, sizeof(float));
    LambWork* w = nullptr;
    if ((rc = get_work(plan, head, stream, &w)) || (rc = switch_stream(plan, stream)))
        return rc;
    const zs::AdamConst c = adam_const(0.0, beta1, beta2, eps, weight_decay, step);
    const float mult = zs::make_result(global_sumsq, loss_scale, clip, 0).mult;
    rc = launch_moments(plan, *w, head, grad16, master32, m32, v32, zs::FromHost{mult, c}, stream);
    if (!rc)
        rc = launch_sums(plan, *w, reinterpret_cast<zs::LayerSums*>(layer_sumsq), nullptr, true, stream);
    if (rc)
        (void)hipEventRecord(plan->done, stream);  // what was queued before the failure
    return rc;
}

int zero_lamb_apply(const zero_lamb_plan_t* plan_, float* master32, const float* m32, const float* v32,
                    uint16_t* param16_out, double global_sumsq, const double* layer_sumsq, double lr, double beta1,
                    double beta2, double eps, double weight_decay, int64_t step, double phi_lo, double phi_hi,
                    void* stream_) {
    const char* fn = "zero_lamb_apply";
    zero_lamb_plan* plan = const_cast<zero_lamb_plan*>(plan_);
    int rc = check_plan(fn, plan);
    if (rc || (rc = check_hyper(fn, lr, beta1, beta2, eps, weight_decay, step, 1.0, 0.0)) ||
        (rc = check_phi(fn, phi_lo, phi_hi)))
        return rc;
    if (std::isnan(global_sumsq) || global_sumsq < 0.0)
        return fail(ZERO_EINVAL, "%s: global_sumsq must be >= 0 (+inf for an overflow)", fn);
    const int64_t n = plan->n;
    if (n > 0 && (!master32 || !m32 || !v32 || !param16_out))
        return fail(ZERO_EINVAL, "%s: NULL array with n > 0", fn);
    const void* arrays[5] = {nullptr, master32, m32, v32, param16_out};
    if ((rc = check_lamb_arrays(fn, arrays, n)))
        return rc;
    if (n > 0 && (rc = check_layer_sums(fn, plan, layer_sumsq, arrays)))
        return rc;
    if (!std::isfinite(global_sumsq))
        return ZERO_SKIPPED;
    if (n == 0)
        return ZERO_OK;
    hipStream_t stream = reinterpret_cast<hipStream_t>(stream_);
    std::lock_guard<std::mutex> plk(plan->mu);
    CtxLock ctx;
    if ((rc = lock_ctx(stream, &ctx)))
        return rc;
    const int head = (int)line_head(master32, sizeof(float));
    LambWork* w = nullptr;
    if ((rc = get_work(plan, head, stream, &w)) || (rc = switch_stream(plan, stream)))
        return rc;
    const zs::AdamConst c = adam_const(lr, beta1, beta2, eps, weight_decay, step);
    return launch_apply(plan, *w, head, master32, m32, v32, param16_out,
                        reinterpret_cast<const zs::LayerSums*>(layer_sumsq), zs::FromHost{0.0f, c}, lr, phi_lo, phi_hi,
                        stream);
}

int zero_probe_lamb_pass(int32_t pass, const uint16_t* grad16, float* master32, float* m32, float* v32,
                         uint16_t* param16_out, int64_t n, void* stream_) {
    const char* fn = "zero_probe_lamb_pass";
    if (pass != 0 && pass != 1)
        return fail(ZERO_EINVAL, "%s: pass must be 0 (moments) or 1 (apply)", fn);
    if (n < 0 || n > kMaxNumel)
        return fail(ZERO_EINVAL, "%s: n=%lld outside [0, 2^40]", fn, (long long)n);
    if (n == 0)
        return ZERO_OK;
    const void* arrays[5] = {pass == 0 ? grad16 : nullptr, master32, m32, v32, pass == 1 ? param16_out : nullptr};
    static const size_t align[5] = {8, 16, 16, 16, 8};
    for (int i = 0; i < 5; ++i)
        if (arrays[i] == nullptr && ((pass == 0 && i != 4) || (pass == 1 && i != 0)))
            return fail(ZERO_EINVAL, "%s: NULL array %d", fn, i);
        else if (arrays[i] && reinterpret_cast<uintptr_t>(arrays[i]) % align[i])
            return fail(ZERO_EINVAL, "%s: array %d must be %zu-byte aligned", fn, i, align[i]);
    int rc = check_lamb_arrays(fn, arrays, n);
    if (rc)
        return rc;
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    hipDeviceProp_t prop;
    HIP_TRY(hipGetDeviceProperties(&prop, dev));
    const void* kern = pass == 0 ? probe_kernel<0>() : probe_kernel<1>();
    int resident = 0;
    const size_t lds = occupancy_lds(kern, kLambBlock, kLambPerCU, prop, &resident);
    const int64_t ntiles = (n + kLambTile - 1) / kLambTile;
    const unsigned grid = tile_grid(ntiles);
    hipStream_t stream = reinterpret_cast<hipStream_t>(stream_);
    if (pass == 0)
        zs::k_probe_lamb<kLambBlock, kLambUnroll, kLambNTL, kLambNTS, kLambXCD, 0>
            <<<grid, kLambBlock, lds, stream>>>(grad16, master32, m32, v32, param16_out, ntiles, n);
    else
        zs::k_probe_lamb<kLambBlock, kLambUnroll, kLambNTL, kLambNTS, kLambXCD, 1>
            <<<grid, kLambBlock, lds, stream>>>(grad16, master32, m32, v32, param16_out, ntiles, n);
    HIP_TRY(hipGetLastError());
    return ZERO_OK;
}

int zero_lamb_profile_read(zero_lamb_profile_t* out) {
    if (!out)
        return fail(ZERO_EINVAL, "zero_lamb_profile_read: NULL out");
    std::lock_guard<std::mutex> lk(g_lprof_mu);
    lprof_drain_locked();
    const int rc = prof_take_error(1);
    *out = g_lprof_acc;
    g_lprof_acc = zero_lamb_profile_t{0, 0.0, 0.0, 0.0, 0.0};
    return rc;
}

}  // extern "C"
