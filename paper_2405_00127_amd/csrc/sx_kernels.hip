// HIP kernels of the stroke-expansion hot path for gfx950 (wave64).
//
//  scan_tags_kernel       tag-monoid prefix scan (Section 8.2): single pass,
//                         wave64 shuffle scan + LDS block scan + decoupled
//                         look-back over dynamically numbered tiles.
//  bisect_kernel          Algorithm 2 in FP64 over the bisection trees' open
//                         nodes (a wave owns a range of tags and tries 64
//                         nodes at a time): slots per tag (pieces + 1 tail)
//                         and the codes of the pieces found; those of a tag
//                         with more than are kept, in order, by a second run.
//  list_kernel            every piece {tag, code} at its canonical position
//  list_small_kernel      in the piece list (small scenes: with the scan of
//                         the slot counts).
//  scan_counts_kernel     exclusive scan of u32 counts into u64 offsets (slot
//  scan_slots_kernel      bases; record offsets, with the count read on the
//  scan_counts_dev_kernel
//                         device).  Replaces the paper's atomic bump
//                         allocation: the output order is canonical.
//  slot_kernel            per piece, the Euler spiral, parallel curves,
//                         cusp split, evolutes and counts (Sections 4-6),
//                         over tiles of 256 pieces.  Writes emission items
//                         into per-tile workspace regions and the slot's
//                         record count.
//  tail_kernel            per tag, its tail slot: the join or cap
//                         (Algorithm 1), items into the same regions.
//  record_kernel          per item chunk, the FP32 per-point work: records
//                         at roff[slot] + the chunk's position in its slot,
//                         staged per tile in LDS and written coalesced.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "sx_device.h"
#include "sx_kernels.h"

namespace sx {

// ------------------------------------------------------ look-back scan
// A tile publishes its aggregate, then its inclusive prefix, as four 32-bit
// parts each (the pair (a, b) split in halves), every part in its own 64-bit
// word next to the launch's epoch: (epoch << 32) | part.  A word is read and
// written with single relaxed device-scope atomics, so a reader sees a part
// only together with its epoch and no fences are needed (on this GPU a
// release or acquire at device scope writes back or invalidates the whole L2
// of the XCD).  A part is ready once its word carries the current epoch; the
// epoch (kept in device memory, advanced by the last tile of every launch,
// never 0) makes stale words of earlier launches read as "not ready", so
// nothing is cleared between launches and the kernels can be replayed inside
// a HIP graph.  Aggregate and inclusive words are separate, so a reader that
// takes a tile's aggregate never mixes in its inclusive prefix.
struct TileStatus {
    unsigned long long agg[4];
    unsigned long long inc[4];
};
static_assert(sizeof(TileStatus) == 64, "tile status layout");

struct Pair {
    uint64_t a, b;
};

struct ScanCtl {
    uint32_t ticket, done, epoch, err;
};
__device__ __forceinline__ Pair operator+(Pair x, Pair y) { return Pair{x.a + y.a, x.b + y.b}; }

__device__ __forceinline__ uint64_t shfl_up_u64(uint64_t v, int d) {
    uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
    lo = __shfl_up(lo, d, 64);
    hi = __shfl_up(hi, d, 64);
    return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ uint64_t shfl_u64(uint64_t v, int src) {
    uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
    lo = __shfl(lo, src, 64);
    hi = __shfl(hi, src, 64);
    return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ uint64_t shfl_xor_u64(uint64_t v, int m) {
    uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
    lo = __shfl_xor(lo, m, 64);
    hi = __shfl_xor(hi, m, 64);
    return ((uint64_t)hi << 32) | lo;
}

// inclusive wave64 scan
__device__ __forceinline__ Pair wave_scan(Pair v, int lane) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        uint64_t ua = shfl_up_u64(v.a, d), ub = shfl_up_u64(v.b, d);
        if (lane >= d) { v.a += ua; v.b += ub; }
    }
    return v;
}
__device__ __forceinline__ Pair wave_sum(Pair v) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
        v.a += shfl_xor_u64(v.a, m);
        v.b += shfl_xor_u64(v.b, m);
    }
    return v;
}

__device__ __forceinline__ uint32_t pair_part(Pair v, int k) {
    const uint64_t w = (k < 2) ? v.a : v.b;
    return (k & 1) ? (uint32_t)(w >> 32) : (uint32_t)w;
}

// Lanes 0..3 of the calling wave publish the four parts of v.
__device__ __forceinline__ void publish(TileStatus* st, uint32_t tile, uint32_t epoch, bool inclusive, Pair v,
                                       int lane) {
    if (lane < 4) {
        const unsigned long long w = ((unsigned long long)epoch << 32) | pair_part(v, lane);
        unsigned long long* p = inclusive ? &st[tile].inc[lane] : &st[tile].agg[lane];
        __hip_atomic_store(p, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

__device__ __forceinline__ unsigned long long rd(const unsigned long long* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The four words of a status record as a pair, if all carry `epoch`.
__device__ __forceinline__ bool read4(const unsigned long long* w, uint32_t epoch, Pair& v) {
    const unsigned long long w0 = rd(w), w1 = rd(w + 1), w2 = rd(w + 2), w3 = rd(w + 3);
    const bool ok = (uint32_t)(w0 >> 32) == epoch && (uint32_t)(w1 >> 32) == epoch && (uint32_t)(w2 >> 32) == epoch &&
                    (uint32_t)(w3 >> 32) == epoch;
    v.a = (uint64_t)(uint32_t)w0 | ((uint64_t)(uint32_t)w1 << 32);
    v.b = (uint64_t)(uint32_t)w2 | ((uint64_t)(uint32_t)w3 << 32);
    return ok;
}

// Wave 0 of tile `tile` computes the exclusive prefix of all earlier tiles.
// The wait for a predecessor is bounded: after kSpinLimit polls the tile
// gives up, records the failure in *err and carries on (wrong sums, but every
// wave exits).  Predecessors always hold earlier tickets, so they are resident
// and the limit is never reached in a correct run.
constexpr uint32_t kSpinLimit = 1u << 22;

__device__ Pair look_back(TileStatus* st, uint32_t tile, uint32_t epoch, int lane, uint32_t* err) {
    Pair excl{0, 0};
    int64_t pos = (int64_t)tile - 1;
    while (pos >= 0) {
        const int64_t idx = pos - lane;
        uint32_t state;  // 0 not ready, 1 aggregate, 2 inclusive, 3 before tile 0 (inclusive zero)
        Pair v{0, 0};
        for (uint32_t spins = 0;; spins++) {
            state = 3;
            v = Pair{0, 0};
            if (idx >= 0) {
                // both records in one round trip, the inclusive one preferred
                Pair vi, va;
                const bool ri = read4(st[idx].inc, epoch, vi);
                const bool ra = read4(st[idx].agg, epoch, va);
                state = ri ? 2u : (ra ? 1u : 0u);
                v = ri ? vi : va;
            }
            if (__ballot(state == 0u) == 0ull) break;
            if (spins >= kSpinLimit) {
                if (lane == 0) atomicOr(err, 1u);
                state = 3;
                v = Pair{0, 0};
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
        const uint64_t incl_mask = __ballot(state >= 2u);
        if (incl_mask) {
            const int first = __builtin_ctzll(incl_mask);  // nearest tile with a full prefix
            if (lane > first) v = Pair{0, 0};
            excl = excl + wave_sum(v);
            break;
        }
        excl = excl + wave_sum(v);
        pos -= 64;
    }
    return excl;
}

// --------------------------------------------------------- tag monoid
constexpr int kScanBlock = 256;
// Items per thread of a scan, by the number of items.  A tile's loads and
// stores follow one another (a thread's items are consecutive), so a small
// scene takes short tiles; a large one long tiles, for its look-back chain.
constexpr int kTagItems = 16;    // tags per thread of the tag-monoid scan
constexpr int kTagItemsSmall = 4;
constexpr uint32_t kTagSmall = 1u << 16;
constexpr int kCountItems = 32;  // counts per thread of the count scans
constexpr int kCountItemsSmall = 8;
constexpr uint32_t kCountSmall = 1u << 18;
constexpr int kRecCountItems = 64;  // counts per thread of the record-count scan (one round of tiles)
constexpr int kRecCountMid = 16, kRecCountSmall = 8;  // the same for fewer slots
constexpr uint32_t kRecMidSlots = 1u << 20, kRecSmallSlots = 1u << 17;
constexpr uint32_t kCountLine = 0x80000000u;  // bit of a slot-count word: a line segment

__device__ __forceinline__ Pair tag_inc(uint32_t t) {
    uint64_t pts = (t & kTagCount) + ((t & kTagEnd) ? 1u : 0u);
    uint64_t pth = (t & kTagPath) ? 1u : 0u;
    uint64_t sty = (t & kTagStyle) ? 1u : 0u;
    uint64_t xf = (t & kTagXform) ? 1u : 0u;
    return Pair{pts | (pth << 32), sty | (xf << 32)};
}

// The last block of a launch resets the ticket and done counters and
// records the epoch it used, so the next launch starts clean without any
// memset.
// (The next launch reads these words after the kernel boundary, which
// makes them visible; no fence is needed here.)
__device__ __forceinline__ void finish_scan(ScanCtl* ctl, uint32_t epoch_used, uint32_t blocks) {
    if (atomicAdd(&ctl->done, 1u) == blocks - 1) {
        ctl->ticket = 0;
        ctl->done = 0;
        ctl->epoch = epoch_used;
    }
}

// blocks: those of the grid that come here.
template <int Items, class Load, class Store>
__device__ void scan_tile(Load load, Store store, uint32_t n, ScanCtl* ctl, TileStatus* st,
                          uint32_t blocks = gridDim.x) {
    constexpr uint32_t kTile = kScanBlock * Items;
    __shared__ uint32_t s_tile, s_epoch;
    __shared__ Pair s_wave[kScanBlock / 64];
    __shared__ Pair s_excl;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    if (tid == 0) {
        s_tile = atomicAdd(&ctl->ticket, 1u);
        // this launch's epoch: one past the last launch's, never 0 (zeroed words)
        const uint32_t e = ctl->epoch + 1u;
        s_epoch = e ? e : 1u;
    }
    __syncthreads();
    const uint32_t tile = s_tile, epoch = s_epoch;
    const uint32_t ntiles = (n + kTile - 1) / kTile;
    if (tile >= ntiles) {
        // a grid sized for a capacity larger than this launch's n: nothing to scan
        if (tid == 0) finish_scan(ctl, s_epoch, blocks);
        return;
    }
    const uint64_t base = (uint64_t)tile * kTile + (uint64_t)tid * Items;
    Pair item[Items];
    load(base, item);
    Pair run{0, 0};
#pragma unroll
    for (int j = 0; j < Items; j++) {
        run = run + item[j];
        item[j] = run;  // thread-local inclusive
    }
    Pair wincl = wave_scan(run, lane);
    if (lane == 63) s_wave[wv] = wincl;
    __syncthreads();
    Pair wpre{0, 0}, agg{0, 0};
#pragma unroll
    for (int k = 0; k < kScanBlock / 64; k++) {
        if (k < wv) wpre = wpre + s_wave[k];
        agg = agg + s_wave[k];
    }
    Pair texcl = wpre + wincl;
    texcl.a -= run.a;
    texcl.b -= run.b;
    if (wv == 0) {
        Pair excl{0, 0};
        if (tile == 0) {
            publish(st, tile, epoch, true, agg, lane);
        } else {
            publish(st, tile, epoch, false, agg, lane);
            excl = look_back(st, tile, epoch, lane, &ctl->err);
            publish(st, tile, epoch, true, excl + agg, lane);
        }
        if (lane == 0) s_excl = excl;
    }
    __syncthreads();
    Pair pre = s_excl + texcl;
    store(base, item, pre);
    __syncthreads();
    if (tid == 0) finish_scan(ctl, s_epoch, blocks);
}

template <int Items>
__global__ __launch_bounds__(kScanBlock) void scan_tags_kernel(const uint8_t* __restrict__ tags, uint32_t n,
                                                               uint32_t* __restrict__ mon, ScanCtl* ctl,
                                                               TileStatus* st, WsCtl* ws_reset) {
    // the workspace counters of the piece kernel that follows start at zero
    if (ws_reset && blockIdx.x == 0 && threadIdx.x == 0) {
        ws_reset->ovf_n = 0;
        ws_reset->items_total = 0;
        ws_reset->ordered_n = 0;
        ws_reset->rich_n = 0;
    }
    auto load = [&](uint64_t base, Pair* item) {
        if (base + Items <= n) {
            uint32_t w[Items / 4];
            if constexpr (Items == 16) {
                const uint4 raw = *reinterpret_cast<const uint4*>(tags + base);
                w[0] = raw.x, w[1] = raw.y, w[2] = raw.z, w[3] = raw.w;
            } else {
                w[0] = *reinterpret_cast<const uint32_t*>(tags + base);
            }
#pragma unroll
            for (int j = 0; j < Items; j++) item[j] = tag_inc((w[j >> 2] >> (8 * (j & 3))) & 0xffu);
        } else {
#pragma unroll
            for (int j = 0; j < Items; j++) item[j] = (base + j < n) ? tag_inc(tags[base + j]) : Pair{0, 0};
        }
    };
    auto store = [&](uint64_t base, const Pair* incl, Pair pre) {
        // item j: exclusive = pre + incl[j-1]; style/xform stored inclusive - 1
        uint32_t o_off[Items], o_pth[Items], o_sty[Items], o_xf[Items];
#pragma unroll
        for (int j = 0; j < Items; j++) {
            Pair ex = pre;
            if (j > 0) ex = ex + incl[j - 1];
            Pair in = pre + incl[j];
            o_off[j] = (uint32_t)ex.a;
            o_pth[j] = (uint32_t)(ex.a >> 32);
            o_sty[j] = (uint32_t)in.b - 1u;
            o_xf[j] = (uint32_t)(in.b >> 32) - 1u;
        }
        // rows of mon_stride_of(n) words: 16-byte aligned, so a full run of
        // tags (base a multiple of Items) stores as uint4
        const size_t stride = mon_stride_of(n);
        uint32_t* m0 = mon;
        uint32_t* m1 = mon + stride;
        uint32_t* m2 = mon + 2 * stride;
        uint32_t* m3 = mon + 3 * stride;
        if (base + Items <= n) {
#pragma unroll
            for (int j = 0; j < Items; j += 4) {
                *reinterpret_cast<uint4*>(m0 + base + j) = make_uint4(o_off[j], o_off[j + 1], o_off[j + 2], o_off[j + 3]);
                *reinterpret_cast<uint4*>(m1 + base + j) = make_uint4(o_pth[j], o_pth[j + 1], o_pth[j + 2], o_pth[j + 3]);
                *reinterpret_cast<uint4*>(m2 + base + j) = make_uint4(o_sty[j], o_sty[j + 1], o_sty[j + 2], o_sty[j + 3]);
                *reinterpret_cast<uint4*>(m3 + base + j) = make_uint4(o_xf[j], o_xf[j + 1], o_xf[j + 2], o_xf[j + 3]);
            }
        } else {
#pragma unroll
            for (int j = 0; j < Items; j++) {
                if (base + j < n) {
                    m0[base + j] = o_off[j];
                    m1[base + j] = o_pth[j];
                    m2[base + j] = o_sty[j];
                    m3[base + j] = o_xf[j];
                }
            }
        }
    };
    scan_tile<Items>(load, store, n, ctl, st);
}

// exclusive scan of u32 counts into u64 offsets; out[n] = total
// (Mask: the bits of an input word that count)
template <int Items, uint32_t Mask = ~0u>
__device__ __forceinline__ void scan_u32_body(const uint32_t* __restrict__ in, uint32_t n, uint64_t* __restrict__ out,
                                              ScanCtl* ctl, TileStatus* st, uint32_t blocks = gridDim.x);
__global__ __launch_bounds__(kScanBlock) void scan_counts_kernel(const uint32_t* __restrict__ in, uint32_t n,
                                                                 uint64_t* __restrict__ out, ScanCtl* ctl,
                                                                 TileStatus* st) {
    scan_u32_body<kCountItems>(in, n, out, ctl, st);
}
// the same with n read from device memory (clamped to the buffers' capacity);
// the grid covers the capacity
template <int Items>
__global__ __launch_bounds__(kScanBlock) void scan_counts_dev_kernel(const uint32_t* __restrict__ in,
                                                                     const uint64_t* __restrict__ n_dev, uint32_t cap,
                                                                     uint64_t* __restrict__ out, ScanCtl* ctl,
                                                                     TileStatus* st) {
    const uint64_t nd = *n_dev;
    if (nd == 0 && blockIdx.x == 0 && threadIdx.x == 0) out[0] = 0;
    scan_u32_body<Items>(in, nd < cap ? (uint32_t)nd : cap, out, ctl, st);
}
template <int Items, uint32_t Mask>
__device__ __forceinline__ void scan_u32_body(const uint32_t* __restrict__ in, uint32_t n, uint64_t* __restrict__ out,
                                              ScanCtl* ctl, TileStatus* st, uint32_t blocks) {
    auto load = [&](uint64_t base, Pair* item) {
        if (base + Items <= n) {
#pragma unroll
            for (int j = 0; j < Items; j += 4) {
                uint4 v = *reinterpret_cast<const uint4*>(in + base + j);
                item[j] = Pair{v.x & Mask, 0};
                item[j + 1] = Pair{v.y & Mask, 0};
                item[j + 2] = Pair{v.z & Mask, 0};
                item[j + 3] = Pair{v.w & Mask, 0};
            }
        } else {
#pragma unroll
            for (int j = 0; j < Items; j++) item[j] = Pair{(base + j < n) ? (uint64_t)(in[base + j] & Mask) : 0ull, 0};
        }
    };
    auto store = [&](uint64_t base, const Pair* incl, Pair pre) {
#pragma unroll
        for (int j = 0; j < Items; j++) {
            const uint64_t ex = pre.a + (j > 0 ? incl[j - 1].a : 0ull);
            if (base + j < n) out[base + j] = ex;
            if (base + j == (uint64_t)n - 1u) out[n] = pre.a + incl[j].a;
        }
    };
    scan_tile<Items>(load, store, n, ctl, st, blocks);
}

// --------------------------------------------------------- bisection
// Algorithm 2 as a tree: a node is an interval [t0, t0 + 2^-depth] of one
// curve, tried on its own (node_accepted); an accepted one is a piece, any
// other is replaced by its two halves.  One wave per workgroup owns `range`
// consecutive tags and keeps the open nodes of up to 64 of their curves on a
// stack in LDS (the curves' control polygons beside it); every turn its lanes
// try the 64 deepest open nodes, and idle lanes take the range's next curves
// once there are kRefillLanes of them.  A curve's trials run side by side, so
// the wave's time follows its number of trials and the depth of its trees,
// not its longest curve's trials in sequence.  With one curve per lane and its
// trials in order (and the library's divisions, square roots and arctangents
// in the trial): 24 random cubics 293 us (one lane's 180 trials), 1,000 of them
// 371 us, 10,007 stress cubics 680 us, 1M map segments 257 us (23 of 64 lanes
// active).  Side by side: 28, 41, 129 and 178 us; with a trial on unit vectors
// and reciprocals, roots and arctangents of its own (node_accepted) 20.5, 28, 68
// and 92 us (with shorter ranges too).  Bound by the FP64 latency of a trial on
// small scenes and by FP64 issue on large ones.
// Pieces are found in no particular order: the q-th one found of tag i is
// kept at codes[i * keep + q] (the first `keep` of each tag), and the write
// pass orders them by their start.
constexpr int kBisectBlock = 64;
constexpr uint32_t kRefillLanes = 16;       // idle lanes that trigger a refill
constexpr uint32_t kNodeSegs = 64;          // curves with open nodes (a refilling wave holds fewer than 64 nodes)
// Open nodes of a wave.  The stack is ordered by depth (deepest on top) and a
// turn takes the top 64: nodes of one depth are pushed at most 128 at a time
// and at most 64 of them stay behind when deeper ones are pushed over them,
// for each depth up to kMaxDepth.
constexpr uint32_t kNodeStack = 64u * (uint32_t)(kMaxDepth + 1);
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A tag with more pieces than codes kept (a rich one) runs its bisection once
// more, by a whole wave, and its codes go to `ordered` in parameter order.
// Their starts are marked in a bitmap of the 2^kMaxDepth parameters, so that
// their order is that of the bits and a piece's depth follows from the next
// one's start.  The first round tries every node above depth 6, of which the
// ones below an accepted node are then dropped.  Who does it: blocks of the slot
// scan that have no tile, from a list (rich tags come in clusters, and one
// wave's range of them would be the launch's length); in a small scene, which
// has no such scan, and ranges of one or two tags, the wave that has bisected
// the tag.  300 stress cubics beside 1M map segments, 32 codes kept: the pass is
// 1.72 ms with one lane per tag in the list launch, 3.28 with the tags of each
// wave's range at its end, 1.09 this way.  400,000 stress cubics, 80 kept: 24.5 ms
// with one lane per tag, 2.9 either other way.  (The list kernel needs 25 VGPRs
// without that code, 93 with it.)
constexpr uint32_t kMarkWords = 1u << (kMaxDepth - 5);
struct BisectLds {
    double seg[13][kNodeSegs];      // NodeSeg
    uint32_t tag[kNodeSegs];        // tag of a segment
    uint32_t open[kNodeSegs];       // its open nodes
    uint32_t found[kNodeSegs];      // its pieces so far
    uint32_t free_[kNodeSegs];      // unused segments
    uint32_t curve[128];            // ring of curves not yet taken
    uint32_t node[kNodeStack];      // segment << 21 | depth << 16 | t0
    uint32_t rich[kBisectMaxRange / 32];  // tags with more pieces than codes kept
    uint32_t n_rich;                      // and their pieces
};
static_assert(offsetof(BisectLds, node) >= kMarkWords * 4, "the bitmap ends before the node stack");
static_assert(kMarkWords == 32u * kBisectBlock, "32 words per lane");

__device__ __forceinline__ bool try_node(const SceneView& sv, const Cfg& cfg, const NodeSeg& e, uint32_t tag,
                                         uint32_t t0u, uint32_t depth) {
    bool tie, ok = node_accepted(e, cfg, t0u, depth, tie);
    if (__builtin_expect(tie, 0)) {
        TagInfo ti;
        Seg s;
        fetch_tag(sv, tag, ti, s);
        ok = hodo_turns(s, t0u, depth);
    }
    return ok;
}

// The pieces of tag i in order (a wave), room for `room` of them; returns
// their number.
__device__ __forceinline__ uint32_t order_codes(const SceneView& sv, const Cfg& cfg, uint32_t i, uint32_t* mark,
                                                uint32_t* node, uint32_t* __restrict__ out, uint64_t room) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    constexpr uint32_t D = (uint32_t)kMaxDepth;
    NodeSeg e;
    {
        TagInfo ti;
        Seg s;
        fetch_tag(sv, i, ti, s);
        e = node_seg(s);
    }
    // (word w of the bitmap at [w % 32][w / 32]: lane l owns words 32 l to 32 l + 31)
    for (uint32_t w = 0; w < 32u; w++) mark[w * 64u + lane] = 0u;
    uint32_t n_node = 0;
    for (bool first = true;; first = false) {
        const uint32_t n_pop = min(n_node, 64u);
        if (!first && n_pop == 0u) break;
        uint32_t depth = 31u - (uint32_t)__builtin_clz(lane + 1u), t0u = lane + 1u - (1u << depth);
        bool act = lane < (first ? 63u : n_pop);
        if (!first && act) {
            const uint32_t w = node[n_node - 1u - lane];
            depth = w >> 16;
            t0u = w & 0xffffu;
        }
        n_node -= n_pop;
        wave_lds_sync();
        const bool ok = act && try_node(sv, cfg, e, i, t0u, depth);
        if (first) {
            const uint64_t m = __ballot(ok);
            for (uint32_t p = (lane + 1u) >> 1; p != 0u; p >>= 1) act = act && ((m >> (p - 1u)) & 1ull) == 0ull;
        }
        const bool split = act && !ok && depth < D && (!first || depth == 5u);
        if (act && (ok || depth == D)) {
            const uint32_t at = t0u << (D - depth);
            atomicOr(&mark[((at >> 5) & 31u) * 64u + (at >> 10)], 1u << (at & 31u));
        }
        const uint64_t m_split = __ballot(split);
        const uint32_t n_split = (uint32_t)__popcll(m_split);
        if (split) {
            const uint32_t to = n_node + 2u * (n_split - 1u - (uint32_t)__popcll(m_split & below));
            const uint32_t w = ((depth + 1u) << 16) | (2u * t0u);
            if (to + 1u < kNodeStack) {
                node[to] = w;
                node[to + 1u] = w + 1u;
            }
        }
        n_node += 2u * n_split;
        wave_lds_sync();
    }
    // this lane's pieces: their number, its first start, the next lane's
    uint32_t cnt = 0, head = 1u << D;
    for (uint32_t w = 0; w < 32u; w++) {
        const uint32_t bits = mark[w * 64u + lane];
        if (cnt == 0u && bits) head = lane * 1024u + w * 32u + (uint32_t)__builtin_ctz(bits);
        cnt += (uint32_t)__popc(bits);
    }
    uint32_t q = cnt;
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t u = __shfl_up(q, d, 64);
        if ((int)lane >= d) q += u;
    }
    const uint32_t total = __shfl(q, 63, 64);
    q -= cnt;
    const uint64_t later = __ballot(cnt != 0u) & ~(below | (1ull << lane));
    const uint32_t after = __shfl(head, later ? (int)__builtin_ctzll(later) : (int)lane, 64);
    const uint32_t tail = later ? after : 1u << D;
    auto put = [&](uint32_t n, uint32_t start, uint32_t depth) {
        const bool pivot = depth == D && !try_node(sv, cfg, e, i, start, D);
        if (n < room) out[n] = slot_code(start >> (D - depth), depth, pivot);
    };
    uint32_t at = head;  // the piece to write: it ends where the next one starts
    for (uint32_t w = 0; w < 32u && cnt; w++) {
        uint32_t bits = mark[w * 64u + lane];
        while (bits) {
            const uint32_t next = lane * 1024u + w * 32u + (uint32_t)__builtin_ctz(bits);
            bits &= bits - 1u;
            if (next == at) continue;  // (its own start)
            const uint32_t depth = D - (uint32_t)__builtin_ctz(next - at);
            put(q++, at, depth);
            at = next;
        }
    }
    if (cnt) {
        const uint32_t depth = D - (uint32_t)__builtin_ctz(tail - at);
        put(q, at, depth);
    }
    wave_lds_sync();
    return total;
}

// Where a rich tag's pieces are: from wave_base[tag / range] + its row's first
// word (its place among its wave's) on in `ordered`; past its end when full (the
// scene then has more slots than the buffers hold).
__device__ __forceinline__ uint64_t ordered_at(const OrderedCodes& oc, uint32_t keep, const uint32_t* codes, uint32_t i) {
    const uint32_t w = oc.wave_base[i / oc.range];
    return w == ~0u ? ~0ull >> 1 : (uint64_t)w + codes[(size_t)i * keep];
}

// Small: the wave orders its rich tags itself.
template <bool Stats, bool Small, int MinWaves>
__global__ __launch_bounds__(kBisectBlock, MinWaves) void bisect_kernel(SceneView sv, Cfg cfg, uint32_t keep,
                                                                        uint32_t* __restrict__ nslots,
                                                                        uint32_t* __restrict__ codes, OrderedCodes oc,
                                                                        unsigned long long* __restrict__ stats) {
    __shared__ BisectLds lds;
    auto& s_seg = lds.seg;
    auto& s_node = lds.node;
    auto& s_tag = lds.tag;
    auto& s_open = lds.open;
    auto& s_found = lds.found;
    auto& s_free = lds.free_;
    auto& s_curve = lds.curve;
    const uint32_t lane = threadIdx.x, range = oc.range;
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const uint32_t a = blockIdx.x * range;
    const uint32_t b = min(sv.n_tags, a + range);
    uint32_t n_trials = 0, n_lines = 0;
    uint32_t at = a;                       // next tag to look at
    uint32_t c_lo = 0, c_hi = 0;           // the ring's entries
    uint32_t n_free = kNodeSegs, n_node = 0;
    s_free[lane] = lane;
    if (lane < kBisectMaxRange / 32u) lds.rich[lane] = 0u;
    if (lane == 0u) lds.n_rich = 0u;
    wave_lds_sync();
    for (;;) {
        // this turn's nodes: the top of the stack on the first lanes
        const uint32_t n_pop = min(n_node, 64u);
        uint32_t take = 0;
        if (64u - n_pop >= kRefillLanes || n_pop == 0u) {
            // the next curves of the range.  Lines (one straight piece each,
            // reading G32), markers and invalid tags need no bisection and
            // are settled here, 64 consecutive tags at a time.
            while (c_hi - c_lo < 64u - n_pop && at < b) {
                const uint32_t i = at + lane;
                bool curve = false;
                if (i < b) {
                    bool line;
                    const int kind = tag_kind(sv, i, line);
                    curve = kind == kTagSegment && !line;
                    if (kind == kTagSegment && line) {
                        nslots[i] = 2u | kCountLine;
                        if (Stats) n_lines++;
                    } else if (!curve) {
                        nslots[i] = 1u;  // only the tail slot
                    }
                }
                const uint64_t m = __ballot(curve);
                if (curve) s_curve[(c_hi + (uint32_t)__popcll(m & below)) & 127u] = i;
                c_hi += (uint32_t)__popcll(m);
                at += 64u;
            }
            take = min(min(64u - n_pop, c_hi - c_lo), n_free);
            wave_lds_sync();
        }
        const uint32_t n_now = n_pop + take;
        if (n_now == 0u) break;
        const bool act = lane < n_now;
        uint32_t sg = 0, depth = 0, t0u = 0;
        if (lane < n_pop) {
            const uint32_t w = s_node[n_node - 1u - lane];
            sg = w >> 21;
            depth = (w >> 16) & 31u;
            t0u = w & 0xffffu;
        } else if (act) {
            const uint32_t i = s_curve[(c_lo + (lane - n_pop)) & 127u];
            sg = s_free[n_free - 1u - (lane - n_pop)];
            TagInfo ti;
            Seg s;
            fetch_tag(sv, i, ti, s);
            const NodeSeg e = node_seg(s);
            s_seg[0][sg] = e.D1.x;
            s_seg[1][sg] = e.D1.y;
            s_seg[2][sg] = e.A2.x;
            s_seg[3][sg] = e.A2.y;
            s_seg[4][sg] = e.C3.x;
            s_seg[5][sg] = e.C3.y;
            s_seg[6][sg] = e.us.x;
            s_seg[7][sg] = e.us.y;
            s_seg[8][sg] = e.ue.x;
            s_seg[9][sg] = e.ue.y;
            s_seg[10][sg] = e.m1;
            s_seg[11][sg] = e.w;
            s_seg[12][sg] = e.eps;
            s_tag[sg] = i;
            s_open[sg] = 1u;
            s_found[sg] = 0u;
        }
        n_node -= n_pop;
        c_lo += take;
        n_free -= take;
        wave_lds_sync();
        bool split = false, done = false;
        if (act) {
            const NodeSeg e{d2(s_seg[0][sg], s_seg[1][sg]), d2(s_seg[2][sg], s_seg[3][sg]),
                            d2(s_seg[4][sg], s_seg[5][sg]), d2(s_seg[6][sg], s_seg[7][sg]),
                            d2(s_seg[8][sg], s_seg[9][sg]), s_seg[10][sg], s_seg[11][sg], s_seg[12][sg]};
            const bool ok = try_node(sv, cfg, e, s_tag[sg], t0u, depth);
            if (Stats) n_trials++;
            split = !ok && depth < (uint32_t)kMaxDepth;
            if (!split) {
                const uint32_t q = atomicAdd(&s_found[sg], 1u);
                if (q < keep) codes[(size_t)s_tag[sg] * keep + q] = slot_code(t0u, depth, !ok);
            }
            // the lane that closes a segment's last open node finishes its tag
            done = atomicAdd(&s_open[sg], split ? 1u : ~0u) == 1u && !split;
            if (done) {
                const uint32_t np = s_found[sg], k = s_tag[sg] - a;
                nslots[a + k] = np + 1u;
                if (np > keep) {
                    codes[(size_t)(a + k) * keep] = atomicAdd(&lds.n_rich, np);
                    atomicOr(&lds.rich[k >> 5], 1u << (k & 31u));
                }
            }
        }
        // the halves of this turn's nodes, the deepest (lane 0's) on top
        const uint64_t m_split = __ballot(split), m_done = __ballot(done);
        const uint32_t n_split = (uint32_t)__popcll(m_split);
        if (split) {
            const uint32_t to = n_node + 2u * (n_split - 1u - (uint32_t)__popcll(m_split & below));
            const uint32_t w = (sg << 21) | ((depth + 1u) << 16) | (2u * t0u);
            if (to + 1u < kNodeStack) {
                s_node[to] = w;
                s_node[to + 1u] = w + 1u;
            }
        }
        n_node += 2u * n_split;
        if (done) s_free[n_free + (uint32_t)__popcll(m_done & below)] = sg;
        n_free += (uint32_t)__popcll(m_done);
        wave_lds_sync();
    }
    const uint32_t more = lds.n_rich;
    if (more) {
        const uint32_t bits = lane < kBisectMaxRange / 32u ? lds.rich[lane] : 0u, cnt = (uint32_t)__popc(bits);
        uint32_t pre = cnt;
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t u = __shfl_up(pre, d, 64);
            if ((int)lane >= d) pre += u;
        }
        unsigned long long at = 0;
        if (lane == 0u) at = atomicAdd(&oc.ctl->ordered_n, (unsigned long long)more);
        if (!Small && lane == 63u) at = atomicAdd(&oc.ctl->rich_n, (unsigned long long)pre);
        const unsigned long long first = __shfl(at, 0, 64);
        const bool fits = first + more <= oc.cap;
        if (lane == 0u) oc.wave_base[blockIdx.x] = fits ? (uint32_t)first : ~0u;
        if (Small && fits) {
            uint32_t off = 0;
            for (uint32_t w = 0; w < (b - a + 31u) / 32u; w++) {
                uint32_t m = __shfl(bits, (int)w, 64);
                while (m) {
                    const uint32_t i = a + w * 32u + (uint32_t)__builtin_ctz(m);
                    m &= m - 1u;
                    if (lane == 0u) codes[(size_t)i * keep] = off;
                    off += order_codes(sv, cfg, i, reinterpret_cast<uint32_t*>(&lds), s_node,
                                       oc.codes + first + off, oc.cap - first - off);
                }
            }
        } else if (!Small) {
            uint32_t m = bits;
            for (unsigned long long k = __shfl(at, 63, 64) + pre - cnt; m; m &= m - 1u)
                oc.rich[k++] = a + lane * 32u + (uint32_t)__builtin_ctz(m);
        }
    }
    if (Stats) {
        atomicAdd(&stats[kStTrials], (unsigned long long)n_trials);
        atomicAdd(&stats[kStLines], (unsigned long long)n_lines);
    }
}

// Slot bases: the scan of the slot counts, by the first blocks; the others put
// the rich tags' codes in order, a wave at a time (without a ticket: 768 more of
// them, all on one word, were 45 us).
template <int Items>
__global__ __launch_bounds__(kScanBlock, 3) void scan_slots_kernel(const uint32_t* __restrict__ nslots,
                                                                uint64_t* __restrict__ base, ScanCtl* ctl,
                                                                TileStatus* st, SceneView sv, Cfg cfg, uint32_t keep,
                                                                const uint32_t* __restrict__ codes, OrderedCodes oc) {
    __shared__ uint32_t s_order[kScanBlock / 64][kMarkWords + kNodeStack];
    const uint32_t n = sv.n_tags, n_tiles = (n + kScanBlock * Items - 1u) / (kScanBlock * Items);
    if (blockIdx.x < n_tiles) {
        scan_u32_body<Items, ~kCountLine>(nslots, n, base, ctl, st, n_tiles);
        return;
    }
    const uint32_t wv = threadIdx.x >> 6, n_rich = (uint32_t)oc.ctl->rich_n;
    for (uint32_t k = (blockIdx.x - n_tiles) * (kScanBlock / 64u) + wv; k < n_rich;
         k += (gridDim.x - n_tiles) * (kScanBlock / 64u)) {
        const uint32_t i = oc.rich[k];
        const uint64_t at = ordered_at(oc, keep, codes, i);
        if (at < oc.cap)
            order_codes(sv, cfg, i, s_order[wv], s_order[wv] + kMarkWords, oc.codes + at, oc.cap - at);
    }
}

// The piece list: every piece {tag, code} at its canonical position (pieces
// in t order; the piece of ordinal p of tag i has slot p + i, since every tag
// before it owns one tail slot besides its pieces).  One thread per piece: a
// tag's piece count says nothing of its neighbours' (a stress cubic has
// hundreds, a line one), so blocks of tags would wait for their richest tag.
// The thread finds its tag from the slot bases and takes its place among the
// tag's kept codes by counting the ones that start before it (the lanes of a
// tag read its row together).  A tag with more pieces than codes kept has
// them in order elsewhere.
constexpr int kListBlock = 256;
// pieces of a block's turn (list_kernel), by the slots it is launched for: a
// thread's pieces follow one another (20,011 segments: 256 a turn 7.7 us, 512
// 9.4, 1,024 13), a large scene's turns share their searches (1M segments:
// 38, 36 and 39 us)
constexpr uint32_t kListPieces = 512, kListPiecesSmall = 256;
constexpr uint32_t kListSmallSlots = 1u << 20;
constexpr uint32_t kListSpan = 1024;        // tags of a turn whose bases are staged in LDS
constexpr uint32_t kSmallTags = 4096;       // scenes whose blocks scan all counts themselves
constexpr uint32_t kSmallBlocks = 768;      // their grid cap

__device__ __forceinline__ uint32_t code_start(uint32_t code) {
    return code_t0u(code) << ((uint32_t)kMaxDepth - code_depth(code));
}
// Piece q of the np pieces of tag i, whose first piece has ordinal `first`.
// Ahead: turns of the row loop unrolled (long rows: four loads in flight; 10,007
// stress cubics: 25.9 -> 24.4 us; 1M map segments, of five pieces a curve, 36 us
// without, 42 with).
template <int Ahead>
__device__ __forceinline__ void list_piece(uint32_t keep, const uint32_t* __restrict__ codes, const OrderedCodes& oc,
                                           bool line,
                                           uint32_t i, uint32_t q, uint32_t np, uint64_t first,
                                           Slot* __restrict__ pcs, uint64_t slot_cap) {
    if (np > keep) {
        const uint64_t at = ordered_at(oc, keep, codes, i) + q;
        if (first + q < slot_cap) pcs[first + q] = Slot{i, at < oc.cap ? oc.codes[at] : slot_code(0u, 0u, false)};
        return;
    }
    uint32_t code = slot_code(0u, 0u, false) | kCodeLine, rank = 0;
    if (!line) {
        const uint32_t* row = codes + (size_t)i * keep;
        code = row[q];
        const uint32_t start = code_start(code);
#pragma unroll Ahead
        for (uint32_t r = 0; r < np; r += 4u) {
            const uint4 v = *reinterpret_cast<const uint4*>(row + r);
            rank += (code_start(v.x) < start ? 1u : 0u) + (r + 1u < np && code_start(v.y) < start ? 1u : 0u) +
                    (r + 2u < np && code_start(v.z) < start ? 1u : 0u) +
                    (r + 3u < np && code_start(v.w) < start ? 1u : 0u);
        }
    }
    if (first + rank < slot_cap) pcs[first + rank] = Slot{i, code};
}

// From the scanned slot bases; a block takes `turn` pieces at a time.
template <int Ahead>
__global__ __launch_bounds__(kListBlock) void list_kernel(uint32_t n, uint32_t keep,
                                                          const uint32_t* __restrict__ nslots,
                                                          const uint32_t* __restrict__ codes, OrderedCodes oc,
                                                          const uint64_t* __restrict__ base, Slot* __restrict__ pcs,
                                                          uint64_t slot_cap, uint32_t turn) {
    __shared__ uint32_t s_tag[2];
    __shared__ uint32_t s_off[kListSpan];  // pieces of the turn before each of its tags
    const uint32_t t = threadIdx.x, lane = t & 63u, wv = t >> 6;
    const uint64_t n_pieces = base[n] - n;
    // (piece ordinal of tag i: base[i] - i)
    for (uint64_t p0 = (uint64_t)blockIdx.x * turn; p0 < n_pieces; p0 += (uint64_t)gridDim.x * turn) {
        const uint64_t p1 = min(p0 + turn, n_pieces);
        // the tags of the turn's first and last piece: the last tag whose
        // pieces start at or before it, 64 probes at a time
        if (wv < 2u) {
            const uint64_t p = wv == 0u ? p0 : p1 - 1u;
            uint32_t lo = 0, cnt = n;  // the answer is in [lo, lo + cnt)
            while (cnt > 1u) {
                const uint32_t step = (cnt + 63u) / 64u;
                const uint32_t off = lane * step;
                const bool le = off < cnt && base[lo + off] - (lo + off) <= p;
                const uint32_t last = 63u - (uint32_t)__builtin_clzll(__ballot(le));  // (lane 0 always is)
                lo += last * step;
                cnt = min(step, cnt - last * step);
            }
            if (lane == 0u) s_tag[wv] = lo;
        }
        __syncthreads();
        const uint32_t tag0 = s_tag[0], tag1 = s_tag[1];
        const uint64_t f0 = base[tag0] - tag0;
        const bool staged = tag1 - tag0 < kListSpan;
        if (staged)
            for (uint32_t k = t; k <= tag1 - tag0; k += kListBlock)
                s_off[k] = (uint32_t)(base[tag0 + k] - (tag0 + k) - f0);
        __syncthreads();
        for (uint64_t p = p0 + t; p < p1; p += kListBlock) {
            uint32_t lo = 0, cnt = tag1 - tag0 + 1u;
            while (cnt > 1u) {
                const uint32_t half = cnt / 2u;
                const uint64_t off = staged ? s_off[lo + half] : base[tag0 + lo + half] - (tag0 + lo + half) - f0;
                const bool le = off <= p - f0;
                lo = le ? lo + half : lo;
                cnt = le ? cnt - half : half;
            }
            const uint32_t i = tag0 + lo, w = nslots[i];
            const uint64_t first = staged ? f0 + s_off[lo] : base[i] - i;
            list_piece<Ahead>(keep, codes, oc, (w & kCountLine) != 0u, i, (uint32_t)(p - first),
                              (w & ~kCountLine) - 1u, first, pcs, slot_cap);
        }
        __syncthreads();  // s_tag and s_off are reused
    }
}

// Small scenes: every block scans all slot counts into LDS (n_tags words), so
// bases and list take one launch without a wait between blocks (1,000 cubics:
// 7.3 us, 11.9 with a scan launch; at 11,000 tags the scan launch and list
// take 30 us, this 35).
__global__ __launch_bounds__(kListBlock) void list_small_kernel(uint32_t n, uint32_t keep,
                                                                const uint32_t* __restrict__ nslots,
                                                                const uint32_t* __restrict__ codes, OrderedCodes oc,
                                                                uint64_t* __restrict__ base, Slot* __restrict__ pcs,
                                                                uint64_t slot_cap) {
    extern __shared__ uint32_t s_end[];  // pieces of tags 0..i; bit 31: a line
    __shared__ uint32_t s_wave[kListBlock / 64];
    const uint32_t t = threadIdx.x, lane = t & 63u, wv = t >> 6;
    // each thread's consecutive tags (a multiple of 4 of them), 16 bytes at a time
    const uint32_t per = ((n + kListBlock - 1u) / kListBlock + 3u) & ~3u;
    const uint32_t i0 = min(t * per, n), i1 = min(i0 + per, n);
    uint32_t mine = 0;
    for (uint32_t i = i0; i < i1; i += 4u) {
        const uint4 v = *reinterpret_cast<const uint4*>(nslots + i);
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (uint32_t j = 0; j < 4u; j++)
            if (i + j < i1) {
                mine += (w[j] & ~kCountLine) - 1u;
                s_end[i + j] = mine | (w[j] & kCountLine);
            }
    }
    uint32_t v = mine;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t u = __shfl_up(v, d, 64);
        if ((int)lane >= d) v += u;
    }
    if (lane == 63u) s_wave[wv] = v;
    __syncthreads();
    uint32_t before = v - mine, run = 0;
#pragma unroll
    for (uint32_t k = 0; k < kListBlock / 64; k++) {
        if (k < wv) before += s_wave[k];
        run += s_wave[k];
    }
    for (uint32_t i = i0; i < i1; i++) s_end[i] += before;
    __syncthreads();
    for (uint32_t i = blockIdx.x * kListBlock + t; i < n; i += gridDim.x * kListBlock) {
        base[i] = (uint64_t)(i ? s_end[i - 1u] & ~kCountLine : 0u) + i;
        if (i == n - 1u) base[n] = (uint64_t)run + n;
    }
    for (uint32_t p = blockIdx.x * kListBlock + t; p < run; p += gridDim.x * kListBlock) {
        uint32_t i = 0, cnt = n;  // the first tag whose pieces end after p
        while (cnt > 1u) {
            const uint32_t half = cnt / 2u;
            const bool le = (s_end[i + half - 1u] & ~kCountLine) <= p;
            i = le ? i + half : i;
            cnt = le ? cnt - half : half;
        }
        const uint32_t first = i ? s_end[i - 1u] & ~kCountLine : 0u, e = s_end[i];
        list_piece<4>(keep, codes, oc, (e & kCountLine) != 0u, i, p - first,
                      (e & ~kCountLine) - first, first, pcs, slot_cap);
    }
}

// ------------------------------------------------------------- slots
constexpr int kSlotBlock = 256;   // pieces per workgroup and per workspace tile
constexpr int kSlotGrid = 8192;   // persistent grid of the slot kernel (tiles stride by it)
constexpr int kTailBlock = 256;   // tags per tail-kernel workgroup
constexpr int kTailGrid = 8192;   // grid cap of the tail kernel (tags stride by it)
constexpr int kTailWin = 64;      // slot tiles a tail-kernel block counts in LDS
constexpr int kRecBlock = 256;
constexpr uint32_t kRecGrid = 8192;  // grid cap of the record kernel (tiles stride by it)
constexpr uint32_t kStageWords = 6400;  // LDS words staging a tile's records (25 KB)
constexpr uint32_t kRecSplit = 8;     // most blocks of a tile (scenes of few tiles)
constexpr uint32_t kRecSplitGrid = 1024;  // record-kernel blocks that a small scene spreads over
// Slots from which the items, about 100 bytes a slot, are more than the 256 MB
// cache holds until they are read: they are then loaded past the caches (1M
// map segments, 3.7M slots: records 223 -> 210 us; 0.9M slots of stress cubics
// the other way, 56 -> 62 us).  Stored past them, the piece launch's lines,
// which fill up bit by bit, took 415 us instead of 243; the tails' nothing.
constexpr uint64_t kStreamSlots = 1u << 21;
constexpr uint32_t kOvfBlocks = 512;  // most record-kernel blocks striding over the overflow units

// Unit allocation of the piece launch.  A piece's items are first counted
// by a dry run of its puts (CountSink: nothing is written); the lane then
// reserves them with one LDS atomic on its tile's counter (the address
// differs between lanes, so this is a plain per-lane atomic, not a scalar
// loop over the lanes) and hands its reservation out in order (UnitSink).
// A reservation that does not fit in the tile's region moves as a whole to
// the shared overflow area (the part inside the region is left empty), in
// chunks of K_ovf records: a small scene's short chunks take up to four times
// the units, and what its regions do not hold has to fit where longer ones did.
struct CountSink {
    static constexpr bool kStats = false;
    uint32_t K, units;
    template <class P>
    __device__ void put(uint32_t, uint32_t nrec, uint32_t, const P&) {
        units += item_units<P>(nrec, K);
    }
};
template <bool Stats>
struct UnitSink {
    static constexpr bool kStats = Stats;
    UnitAt at;            // the next unit of the reservation (null: dropped)
    uint32_t K;           // records per chunk
    uint32_t path, slot;  // output path id, slot index
    uint32_t n;           // records of the slot so far
    uint32_t st[Stats ? kStN : 1];
    template <class P>
    __device__ void put(uint32_t hdr, uint32_t nrec, uint32_t, const P& p) {
        if constexpr (Stats) st[(hdr & 15u) == kItemOffset ? kStRanges : kStEvolutes]++;
        if (at.p) {
            write_item_q(at, hdr, path, slot, n, nrec, K, p);
            at.p += item_units<P>(nrec, K);
        }
        n += nrec;
    }
};
// Units `at` to `at` + `need` of a tile's region, when they fit there.
__device__ __forceinline__ bool units_fit(const ItemWs& ws, uint32_t at, uint32_t need) {
    return at + need <= ws.region_cap;
}
__device__ __forceinline__ UnitAt region_units(const ItemWs& ws, uint64_t tile, uint32_t at) {
    return UnitAt{ws.units + tile * ws.region_cap * 4u + at, ws.region_cap};
}
// `need` units of the overflow area (null: full); the region's units from `at`
// on, reserved and not used, are left empty.
__device__ __forceinline__ UnitAt overflow_units(const ItemWs& ws, uint64_t tile, uint32_t at, uint32_t need) {
    uint4* region = ws.units + tile * ws.region_cap * 4u;
    for (uint32_t u = at; u < ws.region_cap; u++) region[u].x = 0u;
    const unsigned long long o = atomicAdd(&ws.ctl->ovf_n, (unsigned long long)need);
    return UnitAt{o + need <= ws.ovf_cap ? ws.units + ws.ovf_base * 4u + o : nullptr, ws.ovf_cap};
}
constexpr uint32_t kPieceGroup = 4;     // piece tiles a piece-launch workgroup orders together
constexpr uint32_t kSingleTiles = 1024;  // the last piece tiles, taken one per workgroup
constexpr uint32_t kGroupTiles = 4096;   // tiles from which groups are taken at all
// Piece tiles: tile T holds the pieces of ordinals [T, T + 1) x kSlotBlock
// and owns the slots from the first of them up to the first slot of tile
// T + 1 (so also the tails of the tags whose last piece it holds; tile 0
// starts at slot 0, and there is always at least one tile).  Its item
// region and its contiguous range of output records follow from that.
__device__ __forceinline__ uint32_t piece_tile_count(uint64_t n_pieces) {
    return n_pieces ? (uint32_t)((n_pieces + kSlotBlock - 1) / kSlotBlock) : 1u;
}
__device__ __forceinline__ uint64_t tile_first_slot(const Slot* pcs, uint32_t tile, uint32_t n_tiles,
                                                    uint64_t n_slots) {
    if (tile == 0u) return 0u;
    if (tile >= n_tiles) return n_slots;
    const uint64_t p = (uint64_t)tile * kSlotBlock;
    return p + pcs[p].tag;
}
// The tile of tag i's tail slot: the tile of the last piece of tags 0..i.
__device__ __forceinline__ uint64_t tail_tile(const uint64_t* base, uint32_t i) {
    const uint64_t p = base[i + 1] - (uint64_t)(i + 1);  // pieces of tags 0..i
    return p ? (p - 1u) / kSlotBlock : 0u;
}

// One thread per piece: its Euler spiral and parallel curves as emission
// items (records relative to the slot) and the slot's record count.  A
// workgroup takes kPieceGroup consecutive piece tiles at a time and orders
// their pieces by work class (curve pieces, then line pieces), so a wave runs
// pieces of one kind and only one wave of the group mixes the two; it then
// runs the order in passes of kSlotBlock pieces, each piece's items going to
// its own tile's region.  The tails are done by tail_kernel.  Every side has
// one range, a few have a second one past a
// parallel-curve cusp: the counts of the first ranges run on the piece's own
// thread, the second ranges of each wave are packed onto its first lanes
// (the piece's k0, k1, L, width and cusp go through the wave's part of LDS,
// so no block barrier is needed), and then each thread writes its piece's
// items in canonical order.
// Bound by instruction issue (107M wave instructions, mostly FP64, are 175 us of
// the map scene's 245, 1M segments, with 45% of the lanes active) and by the
// items written after it.  With the library's divisions, square roots and
// arctangents, separate multiplies and adds in the polynomials, and all six
// branch breaks walked per range: 362 us; with whole items of one or two
// units: 279 us; 248 us with the tangents, chord and end angles of a piece in
// the oracle's operations.
template <int MinWaves, bool Stats, bool Newton>
__global__ __launch_bounds__(kSlotBlock, MinWaves) void slot_kernel(SceneView sv, Cfg cfg, ItemWs ws,
                                                                    const Slot* __restrict__ pcs,
                                                                    const uint64_t* __restrict__ n_slots_dev,
                                                                    uint64_t slot_cap, uint32_t* __restrict__ rc,
                                                                    unsigned long long* __restrict__ stats) {
    __shared__ uint32_t s_n[kPieceGroup];  // units taken in each tile of the group
    __shared__ uint32_t s_order[kPieceGroup * kSlotBlock];  // group ordinal at each position of the class order
    __shared__ uint32_t s_hist[kPieceGroup][kSlotBlock / 64][2];
    __shared__ uint32_t s_task[2 * kSlotBlock];     // owner thread << 2 | side << 1 | reversed
    __shared__ double s_own[kSlotBlock][4];        // k0, k1, L, w of the owner's piece
    __shared__ XTab s_xtab;
    __shared__ double s_tc[kSlotBlock][2];         // cusp u of each side
    __shared__ RangeRes s_res[2 * kSlotBlock];
    __shared__ RangeRes s_first[2][kSlotBlock];    // each side's first range
    const uint64_t n_slots = *n_slots_dev;
    if (n_slots > slot_cap) return;  // reported by the record kernel
    const uint64_t n_pieces = n_slots - sv.n_tags;
    const uint32_t n_tiles = piece_tile_count(n_pieces);
    // groups of kPieceGroup tiles, then the last kSingleTiles tiles one at a
    // time, so that the launch's last round is short; a scene of fewer than
    // kGroupTiles takes single tiles alone (100,003 segments, 1,055 tiles:
    // seven groups of four were the launch's length, 69 us, 53 without)
    const uint32_t n_multi = n_tiles > kGroupTiles ? (n_tiles - kSingleTiles) / kPieceGroup : 0u;
    const uint32_t n_groups = n_multi + (n_tiles - n_multi * kPieceGroup);
    const uint32_t t = threadIdx.x, lane = t & 63u, wv = t >> 6;
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    uint32_t st[kStN] = {0, 0, 0, 0, 0, 0};
    if (t == 0u) set_xtab(s_xtab, cfg.xinc);  // (read after the first barrier)
    for (uint32_t grp = blockIdx.x; grp < n_groups; grp += gridDim.x) {
        const uint32_t tile0 = grp < n_multi ? grp * kPieceGroup : n_multi * kPieceGroup + (grp - n_multi);
        const uint32_t n_gt = grp < n_multi ? kPieceGroup : 1u;  // tiles of this group
        const uint64_t gfirst = (uint64_t)tile0 * kSlotBlock;
        if (t < kPieceGroup) s_n[t] = 0u;
        // the group's work-class order (curve pieces, then line pieces): each
        // thread ranks its piece of every tile among its wave's pieces of that
        // class, and the waves' class counts go to s_hist
        uint32_t cls[kPieceGroup], rank[kPieceGroup];
#pragma unroll
        for (uint32_t g = 0; g < kPieceGroup; g++) {
            const uint64_t p = gfirst + g * kSlotBlock + t;
            cls[g] = (g < n_gt && p < n_pieces) ? (code_line(pcs[p].code) ? 1u : 0u) : 2u;
            rank[g] = 0u;
#pragma unroll
            for (uint32_t c = 0; c < 2; c++) {
                const uint64_t m = __ballot(cls[g] == c);
                if (cls[g] == c) rank[g] = (uint32_t)__popcll(m & below);
                if (lane == 0) s_hist[g][wv][c] = (uint32_t)__popcll(m);
            }
        }
        __syncthreads();
        uint32_t n_curve = 0, n_valid = 0;
        for (uint32_t g = 0; g < kPieceGroup; g++)
            for (uint32_t w = 0; w < kSlotBlock / 64; w++) {
                n_curve += s_hist[g][w][0];
                n_valid += s_hist[g][w][0] + s_hist[g][w][1];
            }
#pragma unroll
        for (uint32_t g = 0; g < kPieceGroup; g++) {
            if (cls[g] < 2u) {
                uint32_t pos = rank[g] + (cls[g] ? n_curve : 0u);
                for (uint32_t g2 = 0; g2 < kPieceGroup; g2++)
                    for (uint32_t w = 0; w < kSlotBlock / 64; w++)
                        if (g2 < g || (g2 == g && w < wv)) pos += s_hist[g2][w][cls[g]];
                s_order[pos] = g * kSlotBlock + t;
            }
        }
        __syncthreads();
        for (uint32_t pass = 0; pass < kPieceGroup && pass * kSlotBlock < n_valid; pass++) {
            const uint32_t qo = pass * kSlotBlock + t;  // this thread's position in the class order
            // phase 1: the piece's spiral, its sides and the first range of each
            const bool act = qo < n_valid;
            uint64_t j = 0;  // the piece's slot
            uint32_t kt = 0;  // its tile within the group
            Slot sl{0u, kSlotTail};
            if (act) {
                const uint32_t o = s_order[qo];
                kt = o / kSlotBlock;
                sl = pcs[gfirst + o];
                j = gfirst + o + sl.tag;
            }
            UnitSink<Stats> k;
            k.at = UnitAt{nullptr, 0u};
            k.K = cfg.K;
            k.path = 0xffffffffu;
            k.slot = (uint32_t)j;
            k.n = 0;
            if (Stats)
                for (int q = 0; q < kStN; q++) k.st[q] = 0;
            bool have = false;
            ES es;
            SideGeo g0, g1;
            uint32_t qa = 0, qb = 0;
            bool side1 = false;  // a stroke's second side (a fill has one)
            if (act && sl.tag < sv.n_tags) {
                k.path = path_of(sv, sl.tag);
                TagInfo ti;
                Seg sg;
                fetch_tag(sv, sl.tag, ti, sg);
                if (ti.kind == kTagSegment) {
                    have = true;
                    piece_es(sg, ti.line, code_t0u(sl.code), code_depth(sl.code), code_pivot(sl.code), es);
                    if constexpr (Stats) k.st[kStPieces]++;
                    const V2 er = es.pivot ? es.fd : es.frot;
                    ws.es_lo[j] = make_uint4(f_bits(es.fp0.x), f_bits(es.fp0.y), f_bits(er.x), f_bits(er.y));
                    ws.es_hi[j] = make_uint4(f_bits(es.fk0), f_bits(es.fk1), f_bits(es.fL), f_bits(es.fbase));
                    side1 = !sg.fill;
                    g0 = side_geo(es, sg.w, 0);
                    g1 = side_geo(es, sg.w, 1);
                    g1.split = g1.split && side1;
                    const PieceK pk = piece_k(cfg, es.k0, es.k1, es.L, sg.w);
                    s_first[0][t] = range_count<Newton>(cfg, s_xtab, pk, 0, 0.0, g0.tc, g0.rev1);
                    if (side1) s_first[1][t] = range_count<Newton>(cfg, s_xtab, pk, 1, 0.0, g1.tc, g1.rev1);
                    if (g0.split || g1.split) {
                        s_own[t][0] = pk.k0;
                        s_own[t][1] = pk.k1;
                        s_own[t][2] = pk.L;
                        s_own[t][3] = pk.w;
                        s_tc[t][0] = g0.tc;
                        s_tc[t][1] = g1.tc;
                    }
                }
            }
            // phase 2: the second ranges of the wave, packed onto its first lanes
            // (wave-private LDS: no block barrier)
            const bool sp0 = have && g0.split, sp1 = have && g1.split;
            const uint64_t m0 = __ballot(sp0), m1 = __ballot(sp1);
            const uint32_t n0 = (uint32_t)__popcll(m0), n_task = n0 + (uint32_t)__popcll(m1);
            uint32_t* w_task = s_task + wv * 128u;
            RangeRes* w_res = s_res + wv * 128u;
            if (sp0) {
                qa = (uint32_t)__popcll(m0 & below);
                w_task[qa] = (t << 2) | (g0.rev2 ? 1u : 0u);
            }
            if (sp1) {
                qb = n0 + (uint32_t)__popcll(m1 & below);
                w_task[qb] = (t << 2) | 2u | (g1.rev2 ? 1u : 0u);
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            for (uint32_t q = lane; q < n_task; q += 64u) {
                const uint32_t task = w_task[q], own = task >> 2, side = (task >> 1) & 1u;
                const PieceK pk = piece_k(cfg, s_own[own][0], s_own[own][1], s_own[own][2], s_own[own][3]);
                w_res[q] = range_count<Newton>(cfg, s_xtab, pk, (int)side, s_tc[own][side], 1.0, (task & 1u) != 0u);
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            // phase 3: the items of each piece in canonical order, into units
            // reserved for the whole wave at once
            auto put_all = [&](auto& sink) {
                range_put(sink, cfg, es, g0.h, 0.0, g0.tc, g0.rev1, true, !g0.split, g0.P0, g0.Pc, s_first[0][t]);
                if (g0.split) range_put(sink, cfg, es, g0.h, g0.tc, 1.0, g0.rev2, false, true, g0.Pc, g0.P1, w_res[qa]);
                if (side1) {
                    range_put(sink, cfg, es, g1.h, 0.0, g1.tc, g1.rev1, true, !g1.split, g1.P0, g1.Pc, s_first[1][t]);
                    if (g1.split)
                        range_put(sink, cfg, es, g1.h, g1.tc, 1.0, g1.rev2, false, true, g1.Pc, g1.P1, w_res[qb]);
                }
            };
            if (have) {
                // one LDS atomic per lane on its tile's counter (lanes of a wave
                // can belong to different tiles of the group)
                uint32_t at = 0;
                for (bool spill = false;; spill = true) {
                    CountSink dry{k.K, 0u};
                    put_all(dry);
                    if (spill) {
                        k.at = overflow_units(ws, tile0 + kt, at, dry.units);
                        break;
                    }
                    at = atomicAdd(&s_n[kt], dry.units);
                    if (units_fit(ws, at, dry.units)) {
                        k.at = region_units(ws, tile0 + kt, at);
                        break;
                    }
                    k.K = cfg.K_ovf;
                }
            }
            if (have) put_all(k);
            if (act) {
                rc[j] = k.n;
                if (Stats)
                    for (int q = 0; q < kStN; q++) st[q] += k.st[q];
            }
        }
        __syncthreads();
        if (t < n_gt) ws.tile_n[tile0 + t] = s_n[t];
    }
    if (Stats) {
        for (int q = kStPieces; q <= kStEvolutes; q++)
            if (st[q]) atomicAdd(&stats[q], (unsigned long long)st[q]);
    }
}

// Sink of a tail: a join or cap is one item (or none), held in registers
// until the block has placed it.
template <bool Stats>
struct TailSink {
    static constexpr bool kStats = Stats;
    uint32_t hdr, nrec, n;
    JoinP p;
    uint32_t st[Stats ? kStN : 1];
    __device__ void put(uint32_t h, uint32_t nr, uint32_t, const JoinP& q) {
        if constexpr (Stats) st[kStJoins]++;
        hdr = h;
        nrec = nr;
        p = q;
        n += nr;
    }
};

// One thread per tag: its tail slot (the last of its slots, at
// base[tag + 1] - 1) holds the join with the next segment or the cap
// (Algorithm 1).  The items continue the regions of the tails' piece tiles
// after the piece launch's items: a block's consecutive tags have increasing
// tail tiles spanning a few tiles, so it counts its units per tile in LDS and
// takes them from each tile's counter with one global atomic (per lane only
// when the block spans more than kTailWin tiles).  Bound by a block's chain of
// dependent loads, its tiles' atomics and the write: 43 us for 1M tags with
// blocks of 128 or 256, 50 us with 1,024, whose few blocks also leave a small
// scene on few CUs (1,000 cubics: 6.9, 7.7, 12 and 18 us with 128 to 1,024);
// 45 us with a join's unit vectors and turn correctly rounded.
template <bool Stats>
__global__ __launch_bounds__(kTailBlock, 3) void tail_kernel(SceneView sv, Cfg cfg, ItemWs ws,
                                                            const uint64_t* __restrict__ base, uint64_t slot_cap,
                                                            uint32_t* __restrict__ rc,
                                                            unsigned long long* __restrict__ stats) {
    __shared__ uint32_t s_cnt[kTailWin];
    __shared__ uint32_t s_at[kTailWin];
    const uint32_t n = sv.n_tags;
    if (base[n] > slot_cap) return;  // reported by the record kernel
    const uint32_t t = threadIdx.x;
    uint32_t joins = 0;
    for (uint32_t i0 = blockIdx.x * kTailBlock; i0 < n; i0 += gridDim.x * kTailBlock) {
        const uint32_t i = i0 + t;
        const uint32_t ilast = min(n, i0 + kTailBlock) - 1u;
        const uint64_t tile_lo = tail_tile(base, i0);
        const uint64_t span = tail_tile(base, ilast) - tile_lo + 1u;
        const bool win = span <= (uint64_t)kTailWin;
        if (t < kTailWin) s_cnt[t] = 0u;
        __syncthreads();
        TailSink<Stats> k;
        k.nrec = 0;
        k.n = 0;
        if (Stats) k.st[kStJoins] = 0;
        uint64_t slot = 0, tile = 0;
        uint32_t need = 0, local = 0;
        if (i < n) {
            slot = base[i + 1] - 1u;
            tile = tail_tile(base, i);
            TagInfo ti;
            Seg sg;
            fetch_tag(sv, i, ti, sg);
            emit_tail(k, cfg, sv, i, ti, sg);
            need = item_units<JoinP>(k.nrec, cfg.K);
            if (win && need) local = atomicAdd(&s_cnt[tile - tile_lo], need);
        }
        __syncthreads();
        if (win && t < span && s_cnt[t]) s_at[t] = atomicAdd(&ws.tile_n[tile_lo + t], s_cnt[t]);
        __syncthreads();
        if (i < n) {
            if (need) {
                const uint32_t at = win ? s_at[tile - tile_lo] + local : atomicAdd(&ws.tile_n[tile], need);
                const bool fit = units_fit(ws, at, need);
                const uint32_t K = fit ? cfg.K : cfg.K_ovf;
                const UnitAt u = fit ? region_units(ws, tile, at)
                                     : overflow_units(ws, tile, at, item_units<JoinP>(k.nrec, K));
                if (u.p) write_item_q(u, k.hdr, path_of(sv, i), (uint32_t)slot, 0u, k.nrec, K, k.p);
            }
            rc[slot] = k.n;
            if (Stats) joins += k.st[kStJoins];
        }
        __syncthreads();  // s_cnt and s_at are reused
    }
    if (Stats && joins) atomicAdd(&stats[kStJoins], (unsigned long long)joins);
}

// Stream: an item is read once, past the caches (kStreamSlots).
template <bool Stream>
__device__ __forceinline__ uint4 load_quarter(const uint4* p) {
    typedef uint32_t V __attribute__((ext_vector_type(4)));
    if (!Stream) return *p;
    const V v = __builtin_nontemporal_load(reinterpret_cast<const V*>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
}

// One item chunk starting at a unit: reads it and writes its records.
template <bool Newton, bool Stream>
__device__ __forceinline__ void record_item(const SceneView& sv, const ItemWs& ws, const UnitAt& u,
                                            const uint64_t* roff, uint64_t n_slots, float* out, uint64_t cap,
                                            int arcs, const XIncF& xi, float* stage = nullptr, uint64_t lo = 0,
                                            uint64_t hi = 0) {
    uint32_t w[2 * kUnitWords] = {};
    auto quarter = [p0 = u.p, stride = u.stride](uint32_t v, uint32_t j) {
        const uint4* p = p0 + v * stride + j;
        return j ? *p : load_quarter<Stream>(p);
    };
    if (!read_item(quarter, w)) return;
    const uint32_t path = w[1], slot = w[2];
    if (slot >= n_slots) return;
    const uint64_t end = roff[slot + 1] < cap ? roff[slot + 1] : cap;
    RecOut o{out, roff[slot] + w[3], end, path, arcs, stage, lo, hi};
    __align__(16) float es[8];
    if (needs_spiral(w[0], arcs != 0)) {
        *reinterpret_cast<uint4*>(es) = ws.es_lo[slot];
        *reinterpret_cast<uint4*>(es + 4) = ws.es_hi[slot];
    }
    emit_item<Newton>(w, es, xi, o);
}
// Per item chunk, the FP32 per-point work: records at
// roff[slot] + the chunk's position within its slot.  A tile is one block's
// turn; a scene of few tiles gives each to several blocks (every split-th
// round of 256 units), since a block's rounds of records follow one another
// and a chunk's records too: 24 cubics (10 tiles of about 750 units) took 27
// us with a block per tile and chunks of 16, 24 us with chunks of 4, and 15 us
// with 4 or 8 blocks a tile besides (1,000 cubics: 32 and 17 us).  The first
// block also publishes dst[0] = records and dst[1] = 0 when everything fit, else
// 1 (slots or items were dropped: the workspace must grow; the counters stay in
// ws.ctl), for which a launch of its own took 4.6 us.  Bound by its bytes and by
// waiting for them, not by the points: 1M map segments, 198 us; of 243 us before
// the items shrank, 237 were left with every point's computation taken out, 222
// without the copy out.
template <bool Newton>
__global__ __launch_bounds__(kRecBlock, Newton ? 3 : 6) void record_kernel(SceneView sv, ItemWs ws, int arcs,
                                                           const uint64_t* __restrict__ roff,
                                                           const Slot* __restrict__ pcs,
                                                           const uint64_t* __restrict__ n_slots_dev, uint64_t slot_cap,
                                                           float* __restrict__ out, uint64_t cap_records, XIncF xi,
                                                           uint32_t ovf_blocks, uint64_t* __restrict__ dst) {
    const uint64_t n_slots = *n_slots_dev;
    const bool fit = n_slots <= slot_cap && ws.ctl->ovf_n <= ws.ovf_cap;
    if (dst && blockIdx.x == 0u && threadIdx.x == 0u) {
        dst[0] = n_slots <= slot_cap ? roff[n_slots] : 0ull;
        dst[1] = fit ? 0ull : 1ull;
        ws.ctl->slots_total = n_slots;
    }
    if (!fit && n_slots <= slot_cap && blockIdx.x == 0u) {
        // the units to make room for (counting them as they were taken, one
        // atomic per block on one address, 13 ns each, set the tail launch's
        // length: 69 us of the 1M-segment map scene, 43 without)
        unsigned long long asked = 0;
        for (uint32_t i = threadIdx.x; i < piece_tile_count(n_slots - sv.n_tags); i += kRecBlock) asked += ws.tile_n[i];
        if (asked) atomicAdd(&ws.ctl->items_total, asked);
    }
    // nothing is written when the records exceed the capacity, or slots or items were dropped
    if (!fit || roff[n_slots] > cap_records) return;
    const uint32_t n_tiles = piece_tile_count(n_slots - sv.n_tags);
    const uint32_t b = blockIdx.x, n_main = gridDim.x - ovf_blocks;
    if (b < n_main) {
        // a tile's units, one per thread (units in any order: every record's
        // position comes from the scans)
        // the tile's slots own one contiguous output range: records in its
        // first kStageWords words are staged in LDS and copied out with
        // coalesced stores once the tile is done
        __shared__ float s_stage[kStageWords];
        const uint32_t words = arcs ? 6u : 5u;
        // blocks per tile (a split tile's blocks write their records directly)
        const uint32_t split = max(1u, min(kRecSplit, min(n_main, kRecSplitGrid) / n_tiles));
        for (uint32_t turn = b; turn < n_tiles * split; turn += n_main) {
            const uint32_t tile = turn / split, part = turn % split;
            const uint32_t cnt = ws.tile_n[tile] < ws.region_cap ? ws.tile_n[tile] : ws.region_cap;
            uint4* base = ws.units + (uint64_t)tile * ws.region_cap * 4u;
            const uint64_t s_lo = tile_first_slot(pcs, tile, n_tiles, n_slots);
            const uint64_t s_hi = tile_first_slot(pcs, tile + 1u, n_tiles, n_slots);
            const uint64_t lo = roff[s_lo];
            const uint64_t n_rec = roff[s_hi] - lo;
            // (a tile whose items spilled into the overflow area is not
            // staged: those records are written by the overflow blocks)
            const uint64_t n_st = ws.tile_n[tile] > ws.region_cap || split > 1u ? 0u
                                  : (n_rec < kStageWords / words ? n_rec : kStageWords / words);
            auto items = [&](auto st) {
                for (uint32_t s2 = part * kRecBlock + threadIdx.x; s2 < cnt; s2 += split * kRecBlock)
                    record_item<Newton, decltype(st)::value>(sv, ws, UnitAt{base + s2, ws.region_cap}, roff, n_slots,
                                                             out, cap_records, arcs, xi, s_stage, lo, lo + n_st);
            };
            if (n_slots > kStreamSlots) items(std::true_type{});
            else items(std::false_type{});
            if (split > 1u) continue;
            __syncthreads();
            uint32_t* dst32 = reinterpret_cast<uint32_t*>(out) + lo * words;
            const uint32_t* src = reinterpret_cast<const uint32_t*>(s_stage);
            // (written once: past the caches)
            for (uint32_t d = threadIdx.x; d < (uint32_t)n_st * words; d += kRecBlock)
                __builtin_nontemporal_store(src[d], dst32 + d);
            __syncthreads();
        }
    } else {
        const uint64_t cnt = ws.ctl->ovf_n;
        uint4* base = ws.units + ws.ovf_base * 4u;
        for (uint64_t s = (uint64_t)(b - n_main) * kRecBlock + threadIdx.x; s < cnt;
             s += (uint64_t)ovf_blocks * kRecBlock)
            record_item<Newton, false>(sv, ws, UnitAt{base + s, ws.ovf_cap}, roff, n_slots, out, cap_records, arcs, xi);
    }
}

// ----------------------------------------------------- single pass
// The paper's own organisation (Section 8.1), kept as an ablation of the
// count / scan / write pipeline: one thread per tag runs its bisection, its
// pieces' sides and its join or cap in sequence, and every item's records
// are reserved with one atomic add on a global counter and written at once
// (a line soup: records of a range stay together, ranges land in any order).
struct SoupSink {
    static constexpr bool kStats = false;
    float* out;
    uint64_t cap;
    unsigned long long* counter;
    float* es_tab;  // the current piece's FP32 spiral (8 floats, slot 0)
    XIncF xi;
    uint32_t path, slot, n, arcs, newton;
    uint32_t st[1];
    template <class P>
    __device__ void put(uint32_t hdr, uint32_t nrec, uint32_t K, const P& p) {
        n += nrec;
        if (nrec == 0u) return;
        const uint64_t base = atomicAdd(counter, (unsigned long long)nrec);
        if (base + nrec > cap) return;  // counted only: the caller sees the total
        uint32_t w[2 * kUnitWords];
        *reinterpret_cast<P*>(w + kHdrWords) = p;
        const uint32_t nc = chunks(nrec, K);
        for (uint32_t c = 0; c < nc; c++) {
            const uint32_t nchunk = (c + 1 < nc) ? K : nrec - c * K;
            w[0] = hdr | (nchunk << 24);
            w[1] = path;
            w[2] = 0u;
            w[3] = c * K;
            w[4] = c * K;
            w[5] = nrec;
            RecOut o{out, base + (uint64_t)c * K, base + nrec, path, (int)arcs, nullptr, 0, 0};
            if (newton) emit_item<true>(w, es_tab, xi, o);
            else emit_item<false>(w, es_tab, xi, o);
        }
    }
};

__global__ __launch_bounds__(256) void soup_kernel(SceneView sv, Cfg cfg, XIncF xi, float* __restrict__ out,
                                                   uint64_t cap, unsigned long long* __restrict__ counter) {
    const uint32_t stride = gridDim.x * blockDim.x;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < sv.n_tags; i += stride) {
        float es_loc[8];
        SoupSink k{out, cap, counter, es_loc, xi, path_of(sv, i), 0u, 0u, (uint32_t)cfg.arcs,
                   (uint32_t)(cfg.newton && !cfg.arcs), {0u}};
        soup_tag(k, cfg, sv, i);
    }
}

hipError_t launch_soup(const SceneView& sv, const Cfg& cfg, void* out, uint64_t cap_records,
                       unsigned long long* counter, hipStream_t s) {
    if (sv.n_tags == 0) return hipSuccess;
    XIncF xi;
    for (int k = 0; k < 5; k++) xi.v[k] = (float)cfg.xinc[k];
    const uint32_t blocks = (sv.n_tags + 255u) / 256u;
    soup_kernel<<<blocks < 16384u ? blocks : 16384u, 256, 0, s>>>(sv, cfg, xi, (float*)out, cap_records, counter);
    return hipGetLastError();
}

// Per-tag record counts and offsets (verification exports):
// offs[t] = roff[base[t]], counts[t] = offs[t + 1] - offs[t].
__global__ void tag_records_kernel(const uint64_t* __restrict__ base, const uint64_t* __restrict__ roff,
                                   uint64_t slot_cap, uint32_t n_tags, uint32_t* __restrict__ counts,
                                   uint64_t* __restrict__ offs) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i > n_tags) return;
    const bool fit = base[n_tags] <= slot_cap;  // else the slots were dropped: report zeros
    const uint64_t o = fit ? roff[base[i]] : 0ull;
    if (offs) offs[i] = o;
    if (counts && i < n_tags) counts[i] = fit ? (uint32_t)(roff[base[i + 1]] - o) : 0u;
}

// ------------------------------------------------------------- batches
// Concatenate scenes into one arena: block (x, s) copies a strided share of
// scene s's streams.  Concatenation needs no index fix-ups: every scene
// starts a path, a style and a transform, so the tag-monoid scan of the
// arena gives global stream indices, and the path map keeps each scene's own
// input path numbers.
constexpr int kGatherBlock = 256;
constexpr int kGatherBlocksPerScene = 32;

__global__ __launch_bounds__(kGatherBlock) void gather_kernel(const GatherDesc* __restrict__ descs,
                                                              uint8_t* __restrict__ tags, float2* __restrict__ pts,
                                                              StyleD* __restrict__ styles, float* __restrict__ xforms,
                                                              uint32_t* __restrict__ path_map) {
    const GatherDesc d = descs[blockIdx.y];
    const uint32_t stride = kGatherBlock * kGatherBlocksPerScene;
    const uint32_t t0 = blockIdx.x * kGatherBlock + threadIdx.x;
    for (uint32_t i = t0; i < d.n_tags; i += stride) tags[d.tag_base + i] = d.tags[i];
    for (uint32_t i = t0; i < d.n_pts; i += stride) pts[d.pt_base + i] = d.pts[i];
    for (uint32_t i = t0; i < d.n_styles; i += stride) styles[d.style_base + i] = d.styles[i];
    for (uint32_t i = t0; i < 6 * d.n_xforms; i += stride) xforms[6 * (size_t)d.xform_base + i] = d.xforms[i];
    for (uint32_t i = t0; i < d.n_paths; i += stride) path_map[d.path_base + i] = d.path_map[i];
}

// scene_offsets[s] = first record of scene s; scene_offsets[n] = total
// (slot base of the scene's first tag, then that slot's record offset)
__global__ void scene_offsets_kernel(const uint64_t* __restrict__ base, const uint64_t* __restrict__ roff,
                                     uint64_t slot_cap, const GatherDesc* __restrict__ descs, uint32_t n_scenes,
                                     uint32_t n_tags, uint64_t* __restrict__ out) {
    const uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
    // zeros when empty or when the slots were dropped (the status word says so)
    const bool fit = n_tags && base[n_tags] <= slot_cap;
    if (s < n_scenes) out[s] = fit ? roff[base[descs[s].tag_base]] : 0ull;
    if (s == n_scenes) out[s] = fit ? roff[base[n_tags]] : 0ull;
}

// ------------------------------------------------------------- launches
int scan_tiles(uint32_t n) { return (int)((n + kScanBlock * kTagItems - 1) / (kScanBlock * kTagItems)); }
static int count_scan_tiles(uint32_t n, int items = kCountItems) {
    return (int)((n + (uint32_t)(kScanBlock * items) - 1) / (uint32_t)(kScanBlock * items));
}

uint32_t piece_tiles(uint32_t n, uint32_t tile) { return (n + tile - 1) / tile; }
uint32_t slot_tiles(uint64_t n_slots) { return (uint32_t)((n_slots + kSlotBlock - 1) / kSlotBlock); }
uint32_t slot_block() { return kSlotBlock; }

hipError_t launch_scan_tags(const uint8_t* tags, uint32_t n, uint32_t* mon, void* ctl, void* st, WsCtl* ws_reset,
                            hipStream_t s) {
    if (n == 0) return hipSuccess;
    if (n <= kTagSmall)
        scan_tags_kernel<kTagItemsSmall><<<count_scan_tiles(n, kTagItemsSmall), kScanBlock, 0, s>>>(
            tags, n, mon, (ScanCtl*)ctl, (TileStatus*)st, ws_reset);
    else
        scan_tags_kernel<kTagItems><<<scan_tiles(n), kScanBlock, 0, s>>>(tags, n, mon, (ScanCtl*)ctl, (TileStatus*)st,
                                                                         ws_reset);
    return hipGetLastError();
}
hipError_t launch_scan_counts(const uint32_t* in, uint32_t n, uint64_t* out, void* ctl, void* st, hipStream_t s) {
    if (n == 0) return hipSuccess;
    scan_counts_kernel<<<count_scan_tiles(n), kScanBlock, 0, s>>>(in, n, out, (ScanCtl*)ctl, (TileStatus*)st);
    return hipGetLastError();
}
__global__ void zero_u64_kernel(uint64_t* out) {
    if (threadIdx.x == 0) out[0] = 0ull;
}
hipError_t launch_zero_u64(uint64_t* out, hipStream_t s) {
    zero_u64_kernel<<<1, 64, 0, s>>>(out);
    return hipGetLastError();
}
hipError_t launch_scan_counts_dev(const uint32_t* in, const uint64_t* n_dev, uint32_t cap, uint64_t* out, void* ctl,
                                  void* st, hipStream_t s) {
    // a small scene's tiles are short: its one or two tiles' loads and stores
    // would follow one another (24 cubics: 64 counts per thread 8.7 us, 16
    // 4.1 us); a large one's are long, one round of tiles
    if (cap <= kRecSmallSlots)
        scan_counts_dev_kernel<kRecCountSmall><<<count_scan_tiles(cap > 0 ? cap : 1, kRecCountSmall), kScanBlock, 0, s>>>(
            in, n_dev, cap, out, (ScanCtl*)ctl, (TileStatus*)st);
    else if (cap <= kRecMidSlots)
        scan_counts_dev_kernel<kRecCountMid><<<count_scan_tiles(cap, kRecCountMid), kScanBlock, 0, s>>>(
            in, n_dev, cap, out, (ScanCtl*)ctl, (TileStatus*)st);
    else
        scan_counts_dev_kernel<kRecCountItems><<<count_scan_tiles(cap, kRecCountItems), kScanBlock, 0, s>>>(
            in, n_dev, cap, out, (ScanCtl*)ctl, (TileStatus*)st);
    return hipGetLastError();
}

template <bool Stats>
static void bisect_launch(uint32_t g, hipStream_t s, int waves, const SceneView& sv, const Cfg& cfg, uint32_t keep,
                          uint32_t* nslots, uint32_t* codes, const OrderedCodes& oc, unsigned long long* stats) {
    auto* k = list_is_small(sv.n_tags) ? bisect_kernel<Stats, true, 2>
              : waves <= 2             ? bisect_kernel<Stats, false, 2>
              : waves == 3             ? bisect_kernel<Stats, false, 3>
                                       : bisect_kernel<Stats, false, 4>;
    k<<<g, kBisectBlock, 0, s>>>(sv, cfg, keep, nslots, codes, oc, stats);
}
hipError_t launch_bisect(const SceneView& sv, const Cfg& cfg, uint32_t keep, int waves, uint32_t* nslots,
                         uint32_t* codes, const OrderedCodes& oc, unsigned long long* stats, hipStream_t s) {
    if (sv.n_tags == 0) return hipSuccess;
    if (oc.range == 0 || oc.range > kBisectMaxRange || keep < (uint32_t)kKeepCodes || keep % 16u)
        return hipErrorInvalidValue;
    const uint32_t g = (uint32_t)(((uint64_t)sv.n_tags + oc.range - 1) / oc.range);
    if (stats)
        bisect_launch<true>(g, s, waves, sv, cfg, keep, nslots, codes, oc, stats);
    else
        bisect_launch<false>(g, s, waves, sv, cfg, keep, nslots, codes, oc, stats);
    return hipGetLastError();
}
hipError_t launch_scan_slots(const SceneView& sv, const Cfg& cfg, uint32_t keep, const uint32_t* nslots,
                             const uint32_t* codes, const OrderedCodes& oc, uint64_t* base, void* ctl, void* st,
                             hipStream_t s) {
    const uint32_t n = sv.n_tags;
    if (n == 0) return hipSuccess;
    // blocks for rich tags: a wave for 64 tags, up to what the chip holds (they
    // leave at once when there are none)
    const uint32_t more = std::min(768u, n / 256u);
    if (n <= kCountSmall)
        scan_slots_kernel<kCountItemsSmall><<<count_scan_tiles(n, kCountItemsSmall) + more, kScanBlock, 0, s>>>(
            nslots, base, (ScanCtl*)ctl, (TileStatus*)st, sv, cfg, keep, codes, oc);
    else
        scan_slots_kernel<kCountItems><<<count_scan_tiles(n) + more, kScanBlock, 0, s>>>(
            nslots, base, (ScanCtl*)ctl, (TileStatus*)st, sv, cfg, keep, codes, oc);
    return hipGetLastError();
}
bool list_is_small(uint32_t n_tags) { return n_tags <= kSmallTags; }
hipError_t launch_list(uint32_t n_tags, uint32_t keep, const uint32_t* nslots, const uint32_t* codes,
                       const OrderedCodes& oc, uint64_t* base, Slot* pcs, uint64_t slot_cap, hipStream_t s) {
    if (n_tags == 0) return hipSuccess;
    if (list_is_small(n_tags)) {
        const uint32_t g = (uint32_t)std::min<uint64_t>(kSmallBlocks, (slot_cap + kListBlock - 1) / kListBlock);
        list_small_kernel<<<g, kListBlock, n_tags * sizeof(uint32_t), s>>>(n_tags, keep, nslots, codes, oc, base, pcs,
                                                                          slot_cap);
    } else {
        const uint32_t turn = slot_cap <= kListSmallSlots ? kListPiecesSmall : kListPieces;
        const uint32_t g = (uint32_t)std::min<uint64_t>(8192, (slot_cap + turn - 1) / turn);
        // (many pieces per tag: long rows)
        auto* k = slot_cap > 8ull * n_tags ? list_kernel<4> : list_kernel<1>;
        k<<<g, kListBlock, 0, s>>>(n_tags, keep, nslots, codes, oc, base, pcs, slot_cap, turn);
    }
    return hipGetLastError();
}
template <bool Newton>
static void slot_launch(uint32_t g, hipStream_t s, int waves, const SceneView& sv, const Cfg& cfg, const ItemWs& ws,
                        const Slot* pcs, const uint64_t* n_slots_dev, uint64_t slot_cap, uint32_t* rc,
                        unsigned long long* stats) {
    if (stats)
        slot_kernel<1, true, Newton><<<g, kSlotBlock, 0, s>>>(sv, cfg, ws, pcs, n_slots_dev, slot_cap, rc, stats);
    else if (waves <= 1)
        slot_kernel<1, false, Newton><<<g, kSlotBlock, 0, s>>>(sv, cfg, ws, pcs, n_slots_dev, slot_cap, rc, stats);
    else if (waves == 2)
        slot_kernel<2, false, Newton><<<g, kSlotBlock, 0, s>>>(sv, cfg, ws, pcs, n_slots_dev, slot_cap, rc, stats);
    else
        slot_kernel<3, false, Newton><<<g, kSlotBlock, 0, s>>>(sv, cfg, ws, pcs, n_slots_dev, slot_cap, rc, stats);
}
hipError_t launch_slots(const SceneView& sv, const Cfg& cfg, const ItemWs& ws, const Slot* pcs,
                        const uint64_t* n_slots_dev, uint64_t slot_cap, uint32_t* rc, int waves,
                        unsigned long long* stats, hipStream_t s) {
    if (sv.n_tags == 0) return hipSuccess;
    const uint32_t g = std::min<uint32_t>(kSlotGrid, std::max<uint32_t>(1u, slot_tiles(slot_cap)));
    // the exact-integral counts apply to line output only
    if (cfg.newton && !cfg.arcs)
        slot_launch<true>(g, s, waves, sv, cfg, ws, pcs, n_slots_dev, slot_cap, rc, stats);
    else
        slot_launch<false>(g, s, waves, sv, cfg, ws, pcs, n_slots_dev, slot_cap, rc, stats);
    return hipGetLastError();
}
hipError_t launch_tails(const SceneView& sv, const Cfg& cfg, const ItemWs& ws, const uint64_t* base,
                        uint64_t slot_cap, uint32_t* rc, unsigned long long* stats, hipStream_t s) {
    if (sv.n_tags == 0) return hipSuccess;
    const uint32_t g = std::min<uint32_t>(kTailGrid, (sv.n_tags + kTailBlock - 1) / kTailBlock);
    if (stats) tail_kernel<true><<<g, kTailBlock, 0, s>>>(sv, cfg, ws, base, slot_cap, rc, stats);
    else tail_kernel<false><<<g, kTailBlock, 0, s>>>(sv, cfg, ws, base, slot_cap, rc, stats);
    return hipGetLastError();
}
hipError_t launch_records(const SceneView& sv, const ItemWs& ws, const Cfg& cfg, const uint64_t* roff, const Slot* pcs,
                          const uint64_t* n_slots_dev, uint64_t slot_cap, void* out, uint64_t cap, uint64_t* dst,
                          hipStream_t s) {
    if (sv.n_tags == 0) return hipSuccess;
    XIncF xi;
    for (int k = 0; k < 5; k++) xi.v[k] = (float)cfg.xinc[k];
    // a block per tile that the slot buffers can hold; small scenes: several
    // per tile, up to kRecSplitGrid in all (the kernel takes what there is);
    // half as many for the overflow area: with a sixteenth, 200,000 lines with
    // round joins of 18 records, half of whose items overflow, took 107 us here
    // (71 with half), and without overflow the idle blocks cost under 1 us
    const uint32_t tiles = std::min<uint32_t>(kRecGrid, std::max<uint32_t>(1u, slot_tiles(slot_cap)));
    const uint32_t g = std::max<uint32_t>(tiles, std::min<uint32_t>(tiles * kRecSplit, kRecSplitGrid));
    const uint32_t go = std::min<uint32_t>(kOvfBlocks, g / 2u + 1u);
    // exact-density items exist only with line output in the Newton mode
    if (cfg.newton && !cfg.arcs)
        record_kernel<true><<<g + go, kRecBlock, 0, s>>>(sv, ws, cfg.arcs, roff, pcs, n_slots_dev, slot_cap,
                                                         (float*)out, cap, xi, go, dst);
    else
        record_kernel<false><<<g + go, kRecBlock, 0, s>>>(sv, ws, cfg.arcs, roff, pcs, n_slots_dev, slot_cap,
                                                          (float*)out, cap, xi, go, dst);
    return hipGetLastError();
}
hipError_t launch_gather(const GatherDesc* descs, uint32_t n_scenes, uint8_t* tags, float2* pts, StyleD* styles,
                         float* xforms, uint32_t* path_map, hipStream_t s) {
    if (n_scenes == 0) return hipSuccess;
    gather_kernel<<<dim3(kGatherBlocksPerScene, n_scenes), kGatherBlock, 0, s>>>(descs, tags, pts, styles, xforms,
                                                                                 path_map);
    return hipGetLastError();
}
hipError_t launch_scene_offsets(const uint64_t* base, const uint64_t* roff, uint64_t slot_cap, const GatherDesc* descs,
                                uint32_t n_scenes, uint32_t n_tags, uint64_t* scene_offsets, hipStream_t s) {
    scene_offsets_kernel<<<(n_scenes + 1 + 255) / 256, 256, 0, s>>>(base, roff, slot_cap, descs, n_scenes, n_tags,
                                                                    scene_offsets);
    return hipGetLastError();
}
__global__ __launch_bounds__(256) void zero_kernel(ZeroList l) {
    for (int k = 0; k < kZeroParts; k++) {
        uint32_t* p = static_cast<uint32_t*>(l.part[k].p);
        for (size_t i = blockIdx.x * 256u + threadIdx.x; i < l.part[k].bytes / 4u; i += gridDim.x * 256u) p[i] = 0u;
    }
}
hipError_t launch_zero(const ZeroList& list, hipStream_t s) {
    if (!list.ok()) return hipErrorInvalidValue;
    size_t most = 0;
    for (const ZeroPart& x : list.part) most = std::max(most, x.bytes);
    if (most == 0) return hipSuccess;
    zero_kernel<<<(uint32_t)std::min<size_t>(1024, most / 4 / 256 + 1), 256, 0, s>>>(list);
    return hipGetLastError();
}
__global__ void zero2_u64_kernel(uint64_t* out) {
    if (threadIdx.x < 2) out[threadIdx.x] = 0ull;
}
hipError_t launch_no_records(uint64_t* dst, hipStream_t s) {
    zero2_u64_kernel<<<1, 64, 0, s>>>(dst);
    return hipGetLastError();
}
hipError_t launch_tag_records(const uint64_t* base, const uint64_t* roff, uint64_t slot_cap, uint32_t n_tags,
                              uint32_t* counts, uint64_t* offs, hipStream_t s) {
    tag_records_kernel<<<(n_tags + 1 + 255) / 256, 256, 0, s>>>(base, roff, slot_cap, n_tags, counts, offs);
    return hipGetLastError();
}
// (enough for every scan of at most n items: short tiles for few of them)
size_t scan_status_bytes(uint32_t n) {
    const uint32_t few = std::min(std::max(n, 1u), kTagSmall), some = std::min(std::max(n, 1u), kCountSmall);
    return sizeof(TileStatus) * (size_t)std::max({scan_tiles(std::max(n, 1u)), count_scan_tiles(few, kTagItemsSmall),
                                                  count_scan_tiles(some, kCountItemsSmall)});
}
size_t scan_ctl_bytes() { return sizeof(ScanCtl); }


// ------------------------------------------------------------- dashing
// The dashed encoding of a scene (dash patterns of Sections 1 and 9.3), in
// five passes over the source tags: the grid length of every dashed segment;
// an exclusive scan of (length, subpath ends) giving each tag its position
// along the scene and its subpath; each subpath's start position; per tag
// the tags and points it contributes to the dashed encoding; a scan of
// those counts; and the write pass.  Every path of the result opens with an
// empty closed subpath carrying its style and transform bits and ends with
// one carrying its path end bit; each dash is an open subpath ([start point]
// [parts of segments][stroke cap marker]); solid strokes and fills are
// copied.
__global__ __launch_bounds__(256) void dash_measure_kernel(SceneView sv, const DashDesc* __restrict__ desc,
                                                           uint64_t* __restrict__ len, double* __restrict__ panels) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= sv.n_tags) return;
    const uint32_t tag = sv.tags[i];
    uint64_t q = 0;
    if (!(tag & kTagEnd)) {
        const uint32_t sty = sv.mon[2 * (size_t)sv.mon_stride + i];
        if (sty < sv.n_styles && desc[sty].n) {
            const int c = (int)(tag & kTagCount);
            const float2* D = sv.pts + sv.mon[i];
            D2 P[4];
            for (int j = 0; j <= c; j++) P[j] = d2((double)D[j].x, (double)D[j].y);
            double panel[kDashPanels];
            q = (uint64_t)dash_fix(dash_len_d(P, c, panel));
            // kept for the count and write passes (panel k of every tag together)
            for (int k = 0; k < kDashPanels; k++) panels[(size_t)k * sv.n_tags + i] = panel[k];
        }
    }
    len[i] = q;
}

// exclusive scan of (len, subpath end) over the tags; cum[n], subix[n] = totals
__global__ __launch_bounds__(kScanBlock) void dash_scan_kernel(const uint8_t* __restrict__ tags,
                                                               const uint64_t* __restrict__ len, uint32_t n,
                                                               uint64_t* __restrict__ cum,
                                                               uint32_t* __restrict__ subix, ScanCtl* ctl,
                                                               TileStatus* st) {
    auto load = [&](uint64_t base, Pair* item) {
#pragma unroll
        for (int j = 0; j < kTagItems; j++)
            item[j] = (base + j < n) ? Pair{len[base + j], (tags[base + j] & kTagEnd) ? 1ull : 0ull} : Pair{0, 0};
    };
    auto store = [&](uint64_t base, const Pair* incl, Pair pre) {
#pragma unroll
        for (int j = 0; j < kTagItems; j++) {
            const Pair ex = j > 0 ? pre + incl[j - 1] : pre;
            if (base + j < n) {
                cum[base + j] = ex.a;
                subix[base + j] = (uint32_t)ex.b;
            }
            if (base + j == (uint64_t)n - 1u) {
                cum[n] = pre.a + incl[j].a;
                subix[n] = (uint32_t)(pre.b + incl[j].b);
            }
        }
    };
    scan_tile<kTagItems>(load, store, n, ctl, st);
}

__global__ __launch_bounds__(256) void dash_sub_start_kernel(const uint8_t* __restrict__ tags,
                                                             const uint64_t* __restrict__ cum,
                                                             const uint32_t* __restrict__ subix, uint32_t n,
                                                             uint64_t* __restrict__ sub_start) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    if (i == 0) sub_start[0] = 0;
    if (tags[i] & kTagEnd) sub_start[subix[i] + 1u] = cum[i];
}

// chunks of each tag (at most kDashMaxChunks; more sets the flag)
__global__ __launch_bounds__(256) void dash_nch_kernel(DashIn in, uint32_t* __restrict__ nch,
                                                       uint32_t* __restrict__ flag) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= in.sv.n_tags) return;
    uint32_t q = dash_chunks(in, i);
    if (q > kDashMaxChunks) {
        atomicOr(flag, 1u);
        q = 1u;
    }
    nch[i] = q;
}

// the owner tag of every chunk
__global__ __launch_bounds__(256) void dash_chunk_tag_kernel(const uint32_t* __restrict__ nch,
                                                             const uint64_t* __restrict__ chb, uint32_t n,
                                                             uint32_t* __restrict__ ch_tag) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint64_t at = chb[i];
    for (uint32_t q = 0; q < nch[i]; q++) ch_tag[at + q] = i;
}

// The chunk a thread of a 256-thread block takes: the block's chunks
// ordered by kind (dashed lines, quadratics, cubics, the rest), so that a
// wave mostly runs one degree's code (the per-degree dash code would
// otherwise run three times over in a mixed wave).  ~0u: none.
__device__ uint32_t dash_chunk_of_thread(const DashIn& in, const uint32_t* __restrict__ ch_tag, uint32_t n_ch,
                                         uint32_t* s_ord, uint32_t (*s_hist)[4]) {
    const uint32_t t = threadIdx.x, lane = t & 63u, wv = t >> 6;
    const uint32_t k = blockIdx.x * 256u + t;
    uint32_t cls = 4u;
    if (k < n_ch) {
        const uint32_t i = ch_tag[k];
        const uint32_t tag = in.sv.tags[i];
        cls = (!(tag & kTagEnd) && dash_desc_of(in, i).n) ? (tag & kTagCount) - 1u : 3u;
    }
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    uint32_t rank = 0;
#pragma unroll
    for (uint32_t c = 0; c < 4; c++) {
        const uint64_t m = __ballot(cls == c);
        if (cls == c) rank = (uint32_t)__popcll(m & below);
        if (lane == 0) s_hist[wv][c] = (uint32_t)__popcll(m);
    }
    __syncthreads();
    uint32_t pos = rank, n_valid = 0;
    for (uint32_t c = 0; c < 4; c++)
        for (uint32_t w = 0; w < 4; w++) {
            if (c < cls || (c == cls && w < wv)) pos += s_hist[w][c];
            n_valid += s_hist[w][c];
        }
    if (cls < 4u) s_ord[pos] = t;
    __syncthreads();
    return t < n_valid ? blockIdx.x * 256u + s_ord[t] : ~0u;
}

__global__ __launch_bounds__(256) void dash_count_kernel(DashIn in, const uint32_t* __restrict__ ch_tag,
                                                         const uint64_t* __restrict__ chb, uint32_t n_ch,
                                                         uint2* __restrict__ cnt) {
    __shared__ uint32_t s_ord[256];
    __shared__ uint32_t s_hist[4][4];
    const uint32_t k = dash_chunk_of_thread(in, ch_tag, n_ch, s_ord, s_hist);
    if (k == ~0u) return;
    const uint32_t i = ch_tag[k];
    uint32_t nt = 0, np = 0;
    dash_tag<false>(in, i, (uint32_t)(k - chb[i]), nullptr, nullptr, 0, 0, nt, np);
    cnt[k] = make_uint2(nt, np);
}

// exclusive scan of (tags, points) counts; otag[n], opt[n] = totals
__global__ __launch_bounds__(kScanBlock) void dash_off_scan_kernel(const uint2* __restrict__ cnt, uint32_t n,
                                                                   uint64_t* __restrict__ otag,
                                                                   uint64_t* __restrict__ opt, ScanCtl* ctl,
                                                                   TileStatus* st) {
    auto load = [&](uint64_t base, Pair* item) {
#pragma unroll
        for (int j = 0; j < kTagItems; j++) {
            const uint2 v = (base + j < n) ? cnt[base + j] : make_uint2(0u, 0u);
            item[j] = Pair{v.x, v.y};
        }
    };
    auto store = [&](uint64_t base, const Pair* incl, Pair pre) {
#pragma unroll
        for (int j = 0; j < kTagItems; j++) {
            const Pair ex = j > 0 ? pre + incl[j - 1] : pre;
            if (base + j < n) {
                otag[base + j] = ex.a;
                opt[base + j] = ex.b;
            }
            if (base + j == (uint64_t)n - 1u) {
                otag[n] = pre.a + incl[j].a;
                opt[n] = pre.b + incl[j].b;
            }
        }
    };
    scan_tile<kTagItems>(load, store, n, ctl, st);
}

__global__ __launch_bounds__(256) void dash_write_kernel(DashIn in, const uint32_t* __restrict__ ch_tag,
                                                         const uint64_t* __restrict__ chb, uint32_t n_ch,
                                                         const uint64_t* __restrict__ otag,
                                                         const uint64_t* __restrict__ opt,
                                                         uint8_t* __restrict__ tags_out, float2* __restrict__ pts_out) {
    __shared__ uint32_t s_ord[256];
    __shared__ uint32_t s_hist[4][4];
    const uint32_t k = dash_chunk_of_thread(in, ch_tag, n_ch, s_ord, s_hist);
    if (k == ~0u) return;
    const uint32_t i = ch_tag[k];
    uint32_t nt = 0, np = 0;
    dash_tag<true>(in, i, (uint32_t)(k - chb[i]), tags_out, pts_out, otag[k], opt[k], nt, np);
}

hipError_t launch_dash(const SceneView& sv, const DashBufs& b, int phase, uint8_t* tags_out, float2* pts_out,
                       hipStream_t s) {
    const uint32_t n = sv.n_tags;
    if (n == 0) return hipSuccess;
    const uint32_t g = (n + 255u) / 256u;
    DashIn in{sv, b.desc, b.pat, b.panels, b.len, b.cum, b.subix, b.sub_start};
    if (phase == 0) {
        dash_measure_kernel<<<g, 256, 0, s>>>(sv, b.desc, b.len, b.panels);
        dash_scan_kernel<<<scan_tiles(n), kScanBlock, 0, s>>>(sv.tags, b.len, n, b.cum, b.subix, (ScanCtl*)b.ctl0,
                                                               (TileStatus*)b.st0);
        dash_sub_start_kernel<<<g, 256, 0, s>>>(sv.tags, b.cum, b.subix, n, b.sub_start);
        dash_nch_kernel<<<g, 256, 0, s>>>(in, b.nch, b.flag);
        return launch_scan_counts(b.nch, n, b.chb, b.ctl1, b.st1, s);
    }
    if (b.n_ch == 0) return hipSuccess;
    const uint32_t gc = (b.n_ch + 255u) / 256u;
    if (phase == 1) {
        dash_chunk_tag_kernel<<<g, 256, 0, s>>>(b.nch, b.chb, n, b.ch_tag);
        dash_count_kernel<<<gc, 256, 0, s>>>(in, b.ch_tag, b.chb, b.n_ch, b.cnt);
        dash_off_scan_kernel<<<scan_tiles(b.n_ch), kScanBlock, 0, s>>>(b.cnt, b.n_ch, b.otag, b.opt,
                                                                        (ScanCtl*)b.ctl2, (TileStatus*)b.st2);
    } else {
        dash_write_kernel<<<gc, 256, 0, s>>>(in, b.ch_tag, b.chb, b.n_ch, b.otag, b.opt, tags_out, pts_out);
    }
    return hipGetLastError();
}

}  // namespace sx
