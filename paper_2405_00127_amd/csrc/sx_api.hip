// C ABI of the strokex library (declared in include/strokex.h).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstddef>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <string>
#include <unordered_map>
#include <vector>

#include "strokex.h"
#include "sx_device.h"
#include "sx_encode.h"
#include "sx_kernels.h"

// Device memory of a context's scenes.  Large blocks that a scene gives back
// are kept for the next one, up to kPoolBytes in kPoolBlocks blocks: a
// document opened, drawn and closed maps and frees 200 MB otherwise (closing
// took 0.84 ms at 50,000 segments).  Blocks below kPoolMin cost the runtime
// almost nothing and are not kept.  A block is given back with the device
// idle, as hipFree would wait for it, so it has no user on any stream.
// Shared by the context and its scenes (a scene may be released after its
// context; nothing is kept then).
// A device allocation that fails makes every context of the process give its
// kept blocks back.
class DevPool {
   public:
    explicit DevPool(int device) : device_(device) {
        std::lock_guard<std::mutex> lk(all_mu());
        all().push_back(this);
    }
    DevPool(const DevPool&) = delete;
    DevPool& operator=(const DevPool&) = delete;
    ~DevPool() {
        {
            std::lock_guard<std::mutex> lk(all_mu());
            all().erase(std::find(all().begin(), all().end(), this));
        }
        close();
    }
    // Waits for the device; false when that failed.  By freeing a small block:
    // hipFree waits for every stream, and a stream captured in the relaxed mode
    // goes on, where hipDeviceSynchronize would end its capture.
    bool idle() {
        int cur = device_;
        (void)hipGetDevice(&cur);
        if (cur != device_ && hipSetDevice(device_) != hipSuccess) return false;
        void* p = nullptr;
        const bool ok = hipMalloc(&p, 16) == hipSuccess && hipFree(p) == hipSuccess;
        if (!ok) (void)hipGetLastError();
        if (cur != device_) (void)hipSetDevice(cur);
        return ok;
    }
    hipError_t take(void** p, size_t bytes) {
        *p = nullptr;
        bytes = (std::max<size_t>(bytes, 16) + 255) & ~(size_t)255;
        if (bytes >= kPoolMin) {
            std::lock_guard<std::mutex> lk(mu_);
            // the smallest block that holds it, at most twice its size
            size_t best = held_.size();
            for (size_t i = 0; i < held_.size(); i++)
                if (held_[i].bytes >= bytes && held_[i].bytes / 2 <= bytes &&
                    (best == held_.size() || held_[i].bytes < held_[best].bytes))
                    best = i;
            if (best < held_.size()) {
                const Blk b = held_[best];
                held_.erase(held_.begin() + (ptrdiff_t)best);
                total_ -= b.bytes;
                note(b.p, b.bytes);
                *p = b.p;
                return hipSuccess;
            }
        }
        hipError_t e = hipMalloc(p, bytes);
        if (e == hipErrorOutOfMemory && trim_all()) {
            (void)hipGetLastError();
            e = hipMalloc(p, bytes);
        }
        if (e == hipSuccess && bytes >= kPoolMin) {
            std::lock_guard<std::mutex> lk(mu_);
            note(*p, bytes);
        }
        return e;
    }
    // Gives a block back; is_idle: idle() was called and held.
    void give(void* p, bool is_idle) {
        if (!p) return;
        std::lock_guard<std::mutex> lk(mu_);
        const auto it = out_.find(p);
        const size_t bytes = it == out_.end() ? 0 : it->second;
        if (bytes) out_.erase(it);
        if (bytes && bytes <= kPoolBytes && is_idle && !closed_) {
            try {
                held_.push_back(Blk{p, bytes});
                total_ += bytes;
                trim(kPoolBytes);
                return;
            } catch (const std::bad_alloc&) {
                // (freed, not kept)
            }
        }
        (void)hipFree(p);
    }
    void close() {
        std::lock_guard<std::mutex> lk(mu_);
        closed_ = true;
        trim(0);
    }

   private:
    static constexpr size_t kPoolMin = (size_t)256 << 10, kPoolBytes = (size_t)384 << 20, kPoolBlocks = 48;
    struct Blk {
        void* p;
        size_t bytes;
    };
    // (never destroyed: a context may outlive the library's static objects)
    static std::mutex& all_mu() {
        static std::mutex* m = new std::mutex;
        return *m;
    }
    static std::vector<DevPool*>& all() {
        static std::vector<DevPool*>* v = new std::vector<DevPool*>;
        return *v;
    }
    // frees what every pool holds; false when that was nothing
    static bool trim_all() {
        std::lock_guard<std::mutex> lk(all_mu());
        bool any = false;
        for (DevPool* q : all()) {
            std::lock_guard<std::mutex> lq(q->mu_);
            any = any || !q->held_.empty();
            q->trim(0);
        }
        return any;
    }
    // the size of a block in use (one that is not noted is freed, not kept)
    void note(void* p, size_t bytes) {
        try {
            out_[p] = bytes;
        } catch (const std::bad_alloc&) {
        }
    }
    // frees the oldest blocks until at most `most` bytes are held
    void trim(size_t most) {
        while (!held_.empty() && (total_ > most || held_.size() > kPoolBlocks)) {
            (void)hipFree(held_.front().p);
            total_ -= held_.front().bytes;
            held_.erase(held_.begin());
        }
    }
    const int device_;
    std::mutex mu_;
    std::vector<Blk> held_;                  // oldest first
    std::unordered_map<void*, size_t> out_;  // large blocks in use
    size_t total_ = 0;
    bool closed_ = false;
};

static void* pinned_get(size_t bytes) {
    void* p = nullptr;
    if (hipHostMalloc(&p, bytes, hipHostMallocDefault) == hipSuccess) return p;
    (void)hipGetLastError();
    return nullptr;
}
static void pinned_put(void* p) { (void)hipHostFree(p); }
// Scenes of up to this many verbs and paths are encoded into the context's
// pinned buffers (at most about 15 MB, kept); larger ones, or when those
// cannot be had, into pageable memory of their own.
constexpr uint32_t kPinnedVerbs = 1u << 18;

struct sx_ctx {
    int device = 0;
    sx_config cfg = {SX_FIT_OFFSET, SX_DENSITY_APPROX, SX_CONSTANTS_VERSION, 0u};
    std::string err;
    sx_tuning tune = {2u, 16u, 0u, 2u};
    sx::WsCtl* pinned = nullptr;       // host-pinned counters of the last synchronous expansion
    std::shared_ptr<DevPool> pool;
    sx::HostEncoding enc{{pinned_get, pinned_put}};  // a scene's host streams while it is encoded (memory reused)
    void* scratch = nullptr;           // device address of `scratch` on this device
};

// Per-tag terms of the single-pass output estimate (see soup_terms).
struct SoupTerm {
    float a = 0.0f, b = 1.0f, w = 0.0f;
    uint32_t flags = 0;
};

struct sx_scene {
    sx_ctx* ctx = nullptr;
    std::shared_ptr<DevPool> pool;  // the context's
    uint32_t n_tags = 0, n_pts = 0, n_paths = 0, n_styles = 0, n_xforms = 0;
    // encoded streams
    uint8_t* d_tags = nullptr;
    float2* d_pts = nullptr;
    sx::StyleD* d_styles = nullptr;
    float* d_xforms = nullptr;
    uint32_t* d_path_map = nullptr;
    // per tag: monoids, slot counts and their exclusive scan (slot bases)
    uint32_t* d_mon = nullptr;
    uint32_t* d_nslots = nullptr;
    uint32_t* d_codes = nullptr;  // the first piece codes of each tag
    uint32_t* d_ordered = nullptr;  // all piece codes of tags with more (slot_cap words)
    uint32_t* d_rich = nullptr;     // per bisection wave, where they start; the tags (a word per tag each)
    uint64_t* d_base = nullptr;
    // per slot: the slot, its record count and record offset
    sx::Slot* d_slots = nullptr;
    uint32_t* d_rc = nullptr;
    uint64_t* d_roff = nullptr;
    void* d_scan_ctl = nullptr;  // three control blocks (tags, slot counts, record counts)
    void* d_status_tags = nullptr;
    void* d_status_nslots = nullptr;
    void* d_status_rc = nullptr;
    // item workspace of the slot / record kernels
    uint4* d_items = nullptr;  // (four to a unit)
    uint4* d_es = nullptr;  // per-slot spiral records (their two halves, an array each)
    uint32_t* d_tile_n = nullptr;
    sx::WsCtl* d_ws_ctl = nullptr;
    uint32_t region_per_piece = 0;  // item units per piece in the per-tile regions
    uint64_t ovf_cap = 0;          // shared overflow units (overflow_units: with a small scene's spill)
    uint64_t slot_cap = 0;         // slots the slot buffers hold
    // allocated capacities (a batch arena is reused for smaller contents)
    uint32_t cap_tags = 0, cap_pts = 0, cap_styles = 0, cap_xforms = 0, cap_paths = 0;
    bool allocated = false;
    bool batch_arena = false;  // owned by a batch, released with it
    hipStream_t last_stream = nullptr;
    // single-pass variant: record counter and the per-tag terms of the
    // output estimate (host)
    unsigned long long* d_soup_n = nullptr;
    std::vector<SoupTerm> est;  // one per tag (see soup_terms)
    float dash_ms = 0.0f;        // device time of the dashing passes (dashed scenes)
};

struct sx_batch {
    sx_ctx* ctx = nullptr;
    sx_scene* arena = nullptr;
    uint32_t n_scenes = 0, cap_scenes = 0;
    sx::GatherDesc* d_desc = nullptr;  // device copy of the descriptors
    sx::GatherDesc* h_desc = nullptr;  // pinned staging
    hipEvent_t staged = nullptr;       // recorded after the last staging upload
};

// Scratch of sx_scan_u32_noalloc: the scan's control block (first 256
// bytes) and its tile status words, one copy per GPU, zero when the code
// object is loaded.  Host code never passes `scratch` itself to a kernel:
// its device address (per device) comes from hipGetSymbolAddress.
static __device__ __align__(256) unsigned char scratch[SX_SCAN_NOALLOC_BYTES];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device `device` (looked up
// once per device); nullptr if the lookup fails.
void* scratch_ptr(int device) {
    if (device < 0 || device >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[device]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
        g_scratch_ptr[device] = p;
    }
    return g_scratch_ptr[device];
}

constexpr uint32_t kMaxBatchScenes = 65535;
constexpr uint32_t kSlotsPerTag = 4;        // initial slot capacity per tag
constexpr uint32_t kRegionPerPiece = 4;     // initial item units per piece in the tile regions
constexpr uint64_t kMinSlots = 4096;
constexpr uint64_t kMinOverflow = 65536;    // initial shared overflow units (minimum)
constexpr uint32_t kMaxSlotCap = 0xfffff000u;  // slots are indexed by u32

int fail(sx_ctx* ctx, int code, const char* msg) noexcept {
    try {
        if (ctx) ctx->err = msg;
    } catch (const std::bad_alloc&) {
        ctx->err.clear();
    }
    return code;
}

int hip_fail(sx_ctx* ctx, hipError_t e, const char* what) noexcept {
    (void)hipGetLastError();  // (reported here, not by the next launch)
    char msg[256];
    snprintf(msg, sizeof(msg), "%s: %s", what, hipGetErrorString(e));
    return fail(ctx, e == hipErrorOutOfMemory ? SX_ENOMEM : SX_EDEVICE, msg);
}

// What an entry point does, with host memory that runs out reported
// (no C++ exception leaves the library).
template <class F>
int guarded(sx_ctx* ctx, F f) noexcept {
    try {
        return f();
    } catch (const std::bad_alloc&) {
        return fail(ctx, SX_ENOMEM, "host memory");
    }
}

// The scene's large blocks go back to its context's pool: the device is idle
// then (hipFree would wait for it too).
void free_scene(sx_scene* s) {
    if (!s) return;
    const bool idle = s->pool->idle();
    auto dfree = [&](auto*& p) {
        s->pool->give((void*)p, idle);
        p = nullptr;
    };
    dfree(s->d_tags);
    dfree(s->d_pts);
    dfree(s->d_styles);
    dfree(s->d_xforms);
    dfree(s->d_path_map);
    dfree(s->d_mon);
    dfree(s->d_nslots);
    dfree(s->d_codes);
    dfree(s->d_ordered);
    dfree(s->d_rich);
    dfree(s->d_base);
    dfree(s->d_slots);
    dfree(s->d_rc);
    dfree(s->d_roff);
    dfree(s->d_scan_ctl);
    dfree(s->d_status_tags);
    dfree(s->d_status_nslots);
    dfree(s->d_status_rc);
    dfree(s->d_items);
    dfree(s->d_es);
    dfree(s->d_tile_n);
    dfree(s->d_ws_ctl);
    dfree(s->d_soup_n);
    delete s;
}

bool invertible(const sx_affine& X) {
    const double det = (double)X.a * X.d - (double)X.b * X.c;
    return std::isfinite(X.a) && std::isfinite(X.b) && std::isfinite(X.c) && std::isfinite(X.d) &&
           std::isfinite(X.e) && std::isfinite(X.f) && det != 0.0;
}

bool similarity(const sx_affine& X) {
    bool rot = (X.a == X.d) && (X.b == -X.c);
    bool refl = (X.a == -X.d) && (X.b == X.c);
    double det = (double)X.a * X.d - (double)X.b * X.c;
    bool fin = std::isfinite(X.a) && std::isfinite(X.b) && std::isfinite(X.c) && std::isfinite(X.d) &&
               std::isfinite(X.e) && std::isfinite(X.f);
    return fin && (rot || refl) && det != 0.0;
}

sx::SceneView view(const sx_scene* s) {
    sx::SceneView v;
    v.tags = s->d_tags;
    v.pts = s->d_pts;
    v.styles = s->d_styles;
    v.xforms = s->d_xforms;
    v.path_map = s->d_path_map;
    v.mon = s->d_mon;
    v.n_tags = s->n_tags;
    v.n_pts = s->n_pts;
    v.n_styles = s->n_styles;
    v.n_xforms = s->n_xforms;
    v.n_paths = s->n_paths;
    v.mon_stride = sx::mon_stride_of(s->n_tags);
    return v;
}

// A scene of few pieces cannot fill the chip with threads of chunk_k records
// each, which then follow one another: it takes chunks of at most
// kSmallChunk.  (At 2^17 slots and two records per slot, chunks of 4 still
// make no more threads than the chip holds at two waves per SIMD.)
constexpr uint64_t kSmallSlots = 1ull << 17;
constexpr uint32_t kSmallChunk = 4;

// Item units of a scene's tile regions, and of its overflow area.  Items that
// a region does not hold take chunks of chunk_k records in the overflow area,
// but a small scene's short chunks can fill a region with items of which
// chunks of chunk_k would have filled only a part: up to a region more per
// tile overflows, and has to have room for a call to be served as with them.
uint64_t region_units(const sx_scene* s) {
    return (uint64_t)sx::slot_tiles(s->slot_cap) * sx::slot_block() * s->region_per_piece;
}
uint64_t overflow_units(const sx_scene* s) {
    return s->ovf_cap + (s->slot_cap <= kSmallSlots ? region_units(s) : 0u);
}

sx::ItemWs workspace(const sx_scene* s) {
    sx::ItemWs w;
    w.units = s->d_items;
    w.es_lo = s->d_es;
    w.es_hi = s->d_es + s->slot_cap;
    w.tile_n = s->d_tile_n;
    w.ctl = s->d_ws_ctl;
    w.tile = sx::slot_block();
    w.region_cap = s->region_per_piece * w.tile;
    w.ovf_base = region_units(s);
    w.ovf_cap = overflow_units(s);
    return w;
}

char* ctl_block(const sx_scene* s, int k) { return (char*)s->d_scan_ctl + k * sx::scan_ctl_bytes(); }

// (Re)allocate the slot buffers for slot_cap slots and the item workspace
// (region_per_piece 64-byte units per piece in the tile regions, one region
// per slot_block() slots of capacity, since pieces never outnumber slots; ovf
// shared units, and a small scene's spill).
// Scan status words are zeroed when allocated.  Ordered on st; allocation is
// synchronous.
hipError_t size_slots(sx_scene* s, uint64_t slot_cap, uint32_t region_per_piece, uint64_t ovf, hipStream_t st) {
    hipError_t e = hipSuccess;
    auto A = [&](hipError_t r) {
        if (e == hipSuccess) e = r;
    };
    const bool idle = (s->d_slots || s->d_items) && s->pool->idle();  // (a new scene has nothing to give back)
    auto dfree = [&](auto*& p) {
        s->pool->give((void*)p, idle);
        p = nullptr;
    };
    auto dalloc = [&](auto** p, size_t bytes) { return s->pool->take((void**)p, bytes); };
    if (slot_cap != s->slot_cap) {
        s->slot_cap = 0;  // (until all of them are there)
        dfree(s->d_slots);
        dfree(s->d_rc);
        dfree(s->d_roff);
        dfree(s->d_status_rc);
        dfree(s->d_tile_n);
        dfree(s->d_es);
        dfree(s->d_ordered);
        A(dalloc(&s->d_slots, slot_cap * sizeof(sx::Slot)));
        A(dalloc(&s->d_ordered, slot_cap * sizeof(uint32_t)));
        A(dalloc(&s->d_es, slot_cap * 2 * sizeof(uint4)));
        A(dalloc(&s->d_rc, (slot_cap + 16) * sizeof(uint32_t)));
        A(dalloc(&s->d_roff, (slot_cap + 1) * sizeof(uint64_t)));
        A(dalloc(&s->d_status_rc, sx::scan_status_bytes((uint32_t)slot_cap)));
        A(dalloc(&s->d_tile_n, (size_t)sx::slot_tiles(slot_cap) * sizeof(uint32_t)));
        if (e == hipSuccess)
            A(sx::launch_zero({{s->d_status_rc, sx::scan_status_bytes((uint32_t)slot_cap)}}, st));
        if (e != hipSuccess) return e;
        s->slot_cap = slot_cap;
    }
    dfree(s->d_items);
    s->region_per_piece = region_per_piece;
    s->ovf_cap = ovf;
    return dalloc(&s->d_items, (region_units(s) + overflow_units(s)) * sx::kUnitWords * sizeof(uint32_t));
}

// Grow the scene's device buffers to hold at least the given sizes (the
// contents are rewritten by the caller).  Ordered on st; allocation is
// synchronous.
hipError_t reserve_scene(sx_scene* s, uint32_t n_tags, uint32_t n_pts, uint32_t n_styles, uint32_t n_xforms,
                         uint32_t n_paths, hipStream_t st, bool streams_only = false) {
    hipError_t e = hipSuccess;
    auto A = [&](hipError_t r) {
        if (e == hipSuccess) e = r;
    };
    const bool first = !s->allocated;
    bool idle = first;  // (nothing to give back)
    auto dalloc = [&](auto** p, size_t bytes) { return s->pool->take((void**)p, bytes); };
    auto regrow = [&](auto*& p, size_t bytes) {
        if (!idle) idle = s->pool->idle();
        s->pool->give((void*)p, idle);
        p = nullptr;
        A(dalloc(&p, bytes));
    };
    if (first || n_tags > s->cap_tags) {
        const uint32_t c = n_tags;
        s->cap_tags = 0;  // (until everything is there)
        const size_t ntag_pad = ((size_t)c + 16 + 15) & ~(size_t)15;
        regrow(s->d_tags, ntag_pad);
        regrow(s->d_mon, 4 * (size_t)sx::mon_stride_of(c) * sizeof(uint32_t));
        regrow(s->d_status_tags, sx::scan_status_bytes(c));
        if (!streams_only) regrow(s->d_nslots, ((size_t)c + 16) * sizeof(uint32_t));
        // kept piece codes: n x keep_codes_of(n) words for any n <= c (at
        // most 2^25, or kKeepCodes per tag)
        if (!streams_only) {
            regrow(s->d_codes, std::min<size_t>(std::max<size_t>((size_t)1 << 25, (size_t)c * sx::kKeepCodes),
                                                (size_t)c * 1024) * sizeof(uint32_t));
            regrow(s->d_base, ((size_t)c + 1) * sizeof(uint64_t));
            regrow(s->d_rich, 2 * (size_t)c * sizeof(uint32_t));
            regrow(s->d_status_nslots, sx::scan_status_bytes(c));
        }
        if (first) {
            A(dalloc(&s->d_scan_ctl, 3 * sx::scan_ctl_bytes()));
            A(dalloc(&s->d_ws_ctl, sizeof(sx::WsCtl)));
        }
        if (e != hipSuccess) return e;
        // the tag padding, the scans' status words (epoch 0: not ready) and counters
        A(sx::launch_zero({{s->d_tags, ntag_pad},
                           {s->d_status_tags, sx::scan_status_bytes(c)},
                           {s->d_status_nslots, streams_only ? 0 : sx::scan_status_bytes(c)},
                           {s->d_scan_ctl, first ? 3 * sx::scan_ctl_bytes() : 0},
                           {s->d_ws_ctl, first ? sizeof(sx::WsCtl) : 0}},
                          st));
        const uint64_t want = std::max<uint64_t>((uint64_t)c * kSlotsPerTag, kMinSlots);
        if (e == hipSuccess && !streams_only && (want > s->slot_cap || !s->d_items)) {
            const uint32_t region = s->region_per_piece ? s->region_per_piece : kRegionPerPiece;
            A(size_slots(s, std::min<uint64_t>(std::max(want, s->slot_cap), kMaxSlotCap), region,
                         std::max<uint64_t>(std::max<uint64_t>(want, s->ovf_cap), kMinOverflow), st));
        }
        if (e == hipSuccess) s->cap_tags = c;
    }
    if (first || n_pts > s->cap_pts) {
        regrow(s->d_pts, (size_t)n_pts * sizeof(float2));
        s->cap_pts = e == hipSuccess ? n_pts : 0;
    }
    if (first || n_styles > s->cap_styles) {
        regrow(s->d_styles, (size_t)n_styles * sizeof(sx::StyleD));
        s->cap_styles = e == hipSuccess ? n_styles : 0;
    }
    if (first || n_xforms > s->cap_xforms) {
        regrow(s->d_xforms, (size_t)n_xforms * 6 * sizeof(float));
        s->cap_xforms = e == hipSuccess ? n_xforms : 0;
    }
    if (first || n_paths > s->cap_paths) {
        regrow(s->d_path_map, (size_t)n_paths * sizeof(uint32_t));
        s->cap_paths = e == hipSuccess ? n_paths : 0;
    }
    if (e == hipSuccess) s->allocated = true;
    return e;
}

bool make_cfg(const sx_ctx* ctx, float tol, int mode, sx::Cfg& cfg) {
    if (!(tol > 0.0f) || !std::isfinite(tol)) return false;
    if (mode != SX_OUT_LINES && mode != SX_OUT_ARCS) return false;
    double tf = sx::kFlatFrac * (double)tol;
    cfg.tau_fit = sx::kFitFrac * (double)tol;
    cfg.tau_flat = tf;
    cfg.inv_sqrt8tf = std::sqrt(1.0 / (8.0 * tf));
    cfg.cbrt_inv120tf = std::cbrt(1.0 / (120.0 * tf));
    cfg.arcs = mode == SX_OUT_ARCS;
    cfg.paper_fit = ctx && ctx->cfg.fit_mode == SX_FIT_PAPER ? 1 : 0;
    cfg.newton = ctx && ctx->cfg.density == SX_DENSITY_NEWTON ? 1 : 0;
    cfg.K = ctx ? ctx->tune.chunk_k : 16u;
    sx::set_break_increments(cfg.xinc);
    return true;
}

const uint64_t* n_slots_dev(const sx_scene* s) { return s->d_base + s->n_tags; }

// Pipeline phases (each one kernel, in this order on one stream).
enum { kPhScanTags, kPhBisectCount, kPhScanSlots, kPhBisectWrite, kPhPieces, kPhTails, kPhScanRecords, kPhRecords,
       kPhN };

// (the last one puts {records, 0 or 1 = workspace too small} into dst, when given)
hipError_t run_one(const sx_ctx* ctx, const sx_scene* s, const sx::Cfg& conf, int ph, void* out, uint64_t cap_records,
                   unsigned long long* stats, hipStream_t st, uint64_t* dst = nullptr) {
    const sx_tuning& t = ctx->tune;
    if (s->n_tags == 0) return hipSuccess;
    sx::Cfg cfg = conf;
    cfg.K_ovf = cfg.K;
    if (s->slot_cap <= kSmallSlots) cfg.K = std::min(cfg.K, kSmallChunk);
    const uint32_t keep = sx::keep_codes_of(s->n_tags);
    const sx::OrderedCodes oc{s->d_ordered, s->slot_cap, s->d_rich, s->d_rich + s->cap_tags, s->d_ws_ctl,
                              sx::bisect_range_of(s->n_tags, t.bisect_range)};
    switch (ph) {
        case kPhScanTags:
            return sx::launch_scan_tags(s->d_tags, s->n_tags, s->d_mon, ctl_block(s, 0), s->d_status_tags, s->d_ws_ctl,
                                        st);
        case kPhBisectCount:
            return sx::launch_bisect(view(s), cfg, keep, (int)t.bisect_waves, s->d_nslots, s->d_codes, oc, stats, st);
        case kPhScanSlots:
            // (a small scene's bases are part of the next phase)
            if (sx::list_is_small(s->n_tags)) return hipSuccess;
            return sx::launch_scan_slots(view(s), cfg, keep, s->d_nslots, s->d_codes, oc, s->d_base, ctl_block(s, 1),
                                         s->d_status_nslots, st);
        case kPhBisectWrite:
            return sx::launch_list(s->n_tags, keep, s->d_nslots, s->d_codes, oc, s->d_base, s->d_slots, s->slot_cap,
                                   st);
        case kPhPieces:
            return sx::launch_slots(view(s), cfg, workspace(s), s->d_slots, n_slots_dev(s), s->slot_cap, s->d_rc,
                                    (int)t.piece_waves, stats, st);
        case kPhTails:
            return sx::launch_tails(view(s), cfg, workspace(s), s->d_base, s->slot_cap, s->d_rc, stats, st);
        case kPhScanRecords:
            return sx::launch_scan_counts_dev(s->d_rc, n_slots_dev(s), (uint32_t)s->slot_cap, s->d_roff,
                                              ctl_block(s, 2), s->d_status_rc, st);
        case kPhRecords:
            return sx::launch_records(view(s), workspace(s), cfg, s->d_roff, s->d_slots, n_slots_dev(s), s->slot_cap,
                                      out, cap_records, dst, st);
    }
    return hipErrorInvalidValue;
}

// Whether everything a launch needs is allocated (a scene or batch whose
// growth failed keeps what it could not replace at capacity 0).
bool allocated(const sx_scene* s) {
    return s->n_tags <= s->cap_tags && s->n_pts <= s->cap_pts && s->n_styles <= s->cap_styles &&
           s->n_xforms <= s->cap_xforms && s->n_paths <= s->cap_paths && s->slot_cap && s->d_items;
}

// the whole pipeline; dst (device) receives {records, 0 or 1 = workspace too small}
int run_all(sx_ctx* ctx, const sx_scene* s, const sx::Cfg& cfg, void* out, uint64_t cap_records, uint64_t* dst,
            hipStream_t st) {
    if (s->n_tags && !allocated(s)) return fail(ctx, SX_ENOMEM, "workspace");
    hipError_t e = s->n_tags == 0 ? sx::launch_no_records(dst, st) : hipSuccess;
    for (int ph = 0; ph < kPhN && e == hipSuccess; ph++) e = run_one(ctx, s, cfg, ph, out, cap_records, nullptr, st, dst);
    return e == hipSuccess ? SX_OK : hip_fail(ctx, e, "pipeline launch");
}

// Synchronous expansion with workspace growth: runs the pipeline, and when
// slots or items did not fit, grows what was short (from the counters the
// run left) and runs again.  The slot and item counts are deterministic
// functions of the scene, tolerance and mode, so the grown run fits.
int run_sized(sx_ctx* ctx, sx_scene* s, const sx::Cfg& cfg, void* out, uint64_t cap_records, uint64_t* n_records,
              hipStream_t st) {
    if (!s->slot_cap || !s->d_items) {  // a growth that failed
        const uint64_t cap = s->slot_cap ? s->slot_cap : std::max<uint64_t>((uint64_t)s->cap_tags * kSlotsPerTag, kMinSlots);
        hipError_t e = size_slots(s, std::min<uint64_t>(cap, kMaxSlotCap), s->region_per_piece, std::max(s->ovf_cap, cap), st);
        if (e != hipSuccess) return hip_fail(ctx, e, "workspace allocation");
    }
    for (int attempt = 0; attempt < 3; attempt++) {
        uint64_t* dst = reinterpret_cast<uint64_t*>(reinterpret_cast<char*>(s->d_ws_ctl) + offsetof(sx::WsCtl, result));
        int r = run_all(ctx, s, cfg, out, cap_records, dst, st);
        if (r != SX_OK) return r;
        hipError_t e = hipMemcpyAsync(ctx->pinned, s->d_ws_ctl, sizeof(sx::WsCtl), hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) return hip_fail(ctx, e, "count readback");
        const sx::WsCtl w = *ctx->pinned;
        *n_records = w.result[0];
        if (w.result[1] == 0) return SX_OK;
        if (w.slots_total > s->slot_cap) {
            if (w.slots_total > kMaxSlotCap) return fail(ctx, SX_ENOMEM, "scene needs more than 2^32 slots");
            const uint64_t cap = std::min<uint64_t>(w.slots_total + w.slots_total / 4 + 64, kMaxSlotCap);
            e = size_slots(s, cap, s->region_per_piece, std::max<uint64_t>(s->ovf_cap, cap), st);
        } else {
            const uint64_t pieces = std::max<uint64_t>(w.slots_total - std::min<uint64_t>(w.slots_total, s->n_tags), 1);
            const uint64_t per = (w.items_total * 5 / 4 + pieces - 1) / pieces;
            const uint32_t region = (uint32_t)std::min<uint64_t>(std::max<uint64_t>(per, kRegionPerPiece), 64);
            e = size_slots(s, s->slot_cap, region, std::max<uint64_t>(w.items_total, kMinOverflow), st);
        }
        if (e != hipSuccess) return hip_fail(ctx, e, "workspace allocation");
    }
    return fail(ctx, SX_EDEVICE, "workspace still too small after resizing");
}

}  // namespace

extern "C" {

const char* sx_version(void) { return "strokex 0.1 (gfx950)"; }

int sx_ctx_create(int device, const sx_config* cfg, sx_ctx** out) {
    if (!out) return SX_EINVAL;
    *out = nullptr;
    sx_config conf = {SX_FIT_OFFSET, SX_DENSITY_APPROX, SX_CONSTANTS_VERSION, 0u};
    if (cfg) {
        if (cfg->fit_mode > SX_FIT_PAPER || cfg->density > SX_DENSITY_NEWTON || cfg->reserved != 0u ||
            (cfg->constants_version != 0u && cfg->constants_version != SX_CONSTANTS_VERSION))
            return SX_EINVAL;
        conf = *cfg;
        conf.constants_version = SX_CONSTANTS_VERSION;
    }
    int n = 0;
    if (hipGetDeviceCount(&n) != hipSuccess || device < 0 || device >= n) return SX_EDEVICE;
    sx_ctx* c = new (std::nothrow) sx_ctx();
    if (!c) return SX_ENOMEM;
    c->device = device;
    c->cfg = conf;
    if (guarded(nullptr, [&] { return c->pool = std::make_shared<DevPool>(device), SX_OK; }) != SX_OK) {
        delete c;
        return SX_ENOMEM;
    }
    if (hipSetDevice(device) != hipSuccess) { delete c; return SX_EDEVICE; }
    if (hipHostMalloc((void**)&c->pinned, sizeof(sx::WsCtl), hipHostMallocDefault) != hipSuccess) {
        (void)hipGetLastError();
        delete c;
        return SX_ENOMEM;
    }
    // the no-allocation scan's scratch on this device (device is current)
    c->scratch = scratch_ptr(device);
    *out = c;
    return SX_OK;
}

int sx_ctx_destroy(sx_ctx* ctx) {
    if (!ctx) return SX_OK;
    if (ctx->pinned) (void)hipHostFree(ctx->pinned);
    ctx->pool->close();
    delete ctx;
    return SX_OK;
}

int sx_set_tuning(sx_ctx* ctx, const sx_tuning* t) {
    if (!ctx || !t) return SX_EINVAL;
    if (t->piece_waves < 1 || t->piece_waves > 3) return fail(ctx, SX_EINVAL, "piece_waves must be 1, 2 or 3");
    if (t->chunk_k < 1 || t->chunk_k > 255) return fail(ctx, SX_EINVAL, "chunk_k must be in [1, 255]");
    if (t->bisect_range != 0 && (t->bisect_range % 64 || t->bisect_range > 1024))
        return fail(ctx, SX_EINVAL, "bisect_range must be a multiple of 64 up to 1024 (0: by size)");
    if (t->bisect_waves != 0 && (t->bisect_waves < 2 || t->bisect_waves > 4))
        return fail(ctx, SX_EINVAL, "bisect_waves must be 2, 3 or 4 (0: 2)");
    ctx->tune = *t;
    if (ctx->tune.bisect_waves == 0) ctx->tune.bisect_waves = 2;
    return SX_OK;
}

int sx_get_config(const sx_ctx* ctx, sx_config* cfg) {
    if (!ctx || !cfg) return SX_EINVAL;
    *cfg = ctx->cfg;
    return SX_OK;
}

int sx_get_tuning(const sx_ctx* ctx, sx_tuning* t) {
    if (!ctx || !t) return SX_EINVAL;
    *t = ctx->tune;
    return SX_OK;
}

const char* sx_last_error(const sx_ctx* ctx) { return ctx ? ctx->err.c_str() : "null context"; }

// Per-tag terms of the single-pass output estimate (the paper sizes its
// atomically filled buffer with Wang's formula on the host, Section 8.1):
// a = sqrt(d (d - 1) M / 8) of the world control polygon (M its largest
// second difference), so that Wang's count at flattening tolerance t is
// a / sqrt(t); b = sqrt(1 + w k), k = d (d - 1) M / chord^2, inflating it for
// the parallel curves of half-width w; flags: 1 curve, 2 line, 4 marker,
// 8 fill, 16 round join or cap.
enum { kEstCurve = 1, kEstLine = 2, kEstMarker = 4, kEstFill = 8, kEstRound = 16 };
static void soup_terms(const sx::HostEncoding& enc, const sx_style* styles, const sx_affine* xforms,
                       std::vector<SoupTerm>& est) {
    const size_t n = enc.tags.size();
    // (squares of FP32 values stay in range: no need of hypot's scaling)
    auto norm = [](double x, double y) { return std::sqrt(x * x + y * y); };
    est.assign(n, SoupTerm{});
    uint32_t off = 0;
    int sty = -1, xfi = -1;
    for (size_t i = 0; i < n; i++) {
        const uint32_t t = enc.tags[i];
        if (t & sx::kTagStyle) sty++;
        if (t & sx::kTagXform) xfi++;
        const sx_style& st = styles[enc.style_stream[sty]];
        const sx_affine& X = xforms[enc.xform_stream[xfi]];
        const bool fill = (st.flags & SX_STYLE_FILL) != 0;
        const double scale = std::sqrt(std::fabs((double)X.a * X.d - (double)X.b * X.c));
        const double w = fill ? 0.0 : (double)st.half_width * scale;
        uint32_t fl = fill ? kEstFill : 0u;
        if (!fill && (st.join == SX_JOIN_ROUND || st.start_cap == SX_CAP_ROUND || st.end_cap == SX_CAP_ROUND))
            fl |= kEstRound;
        const uint32_t c = t & sx::kTagCount;
        double a = 0.0, b = 1.0;
        if (t & sx::kTagEnd) {
            fl |= kEstMarker;
        } else if (c == 1u) {
            fl |= kEstLine;
        } else {
            fl |= kEstCurve;
            double px[4], py[4];
            for (uint32_t j = 0; j <= c; j++) {
                const double x = enc.data[2 * (off + j)], y = enc.data[2 * (off + j) + 1];
                px[j] = (double)X.a * x + (double)X.c * y;
                py[j] = (double)X.b * x + (double)X.d * y;
            }
            double M = 0.0;
            for (uint32_t j = 0; j + 2 <= c; j++)
                M = std::max(M, norm(px[j + 2] - 2.0 * px[j + 1] + px[j], py[j + 2] - 2.0 * py[j + 1] + py[j]));
            const double dd = (double)(c * (c - 1));
            const double ch = norm(px[c] - px[0], py[c] - py[0]);
            a = std::sqrt(dd * M / 8.0);
            b = std::sqrt(1.0 + (ch > 0.0 ? w * dd * M / (ch * ch) : 0.0));
        }
        est[i] = SoupTerm{(float)a, (float)b, (float)w, fl};
        off += c + ((t & sx::kTagEnd) ? 1u : 0u);
    }
}

// A scene until it is handed out.
struct SceneOwner {
    sx_scene* s = nullptr;
    ~SceneOwner() { free_scene(s); }
    sx_scene* give() {
        sx_scene* r = s;
        s = nullptr;
        return r;
    }
};

static int encode_impl(sx_ctx* ctx, const sx_paths* paths, const sx_style* styles, uint32_t n_styles,
                       const sx_affine* xforms, uint32_t n_xforms, void* stream, sx_scene** out,
                       std::vector<uint32_t>* style_stream, bool streams_only = false) {
    if (!ctx || !out) return SX_EINVAL;
    *out = nullptr;
    if (!paths || (paths->n_paths && (!paths->verbs || !paths->verb_off || !paths->pts || !paths->pt_off ||
                                      !paths->style_ix || !paths->xform_ix)))
        return fail(ctx, SX_EINVAL, "null path arrays");
    if ((n_styles && !styles) || (n_xforms && !xforms)) return fail(ctx, SX_EINVAL, "null style/transform table");
    if (hipSetDevice(ctx->device) != hipSuccess) return fail(ctx, SX_EDEVICE, "hipSetDevice");
    sx::HostEncoding own;
    const bool large = paths->n_paths && std::max(paths->verb_off[paths->n_paths], paths->n_paths) > kPinnedVerbs;
    sx::HostEncoding* to = large ? &own : &ctx->enc;
    std::string err;
    for (bool done = false; !done;) {
        try {
            if (!sx::encode_paths(*paths, styles, n_styles, n_xforms, *to, err)) return fail(ctx, SX_EINVAL, err.c_str());
            done = true;
        } catch (const std::bad_alloc&) {
            if (to == &own) return fail(ctx, SX_ENOMEM, "host encoding");
            ctx->enc.tags.reset();
            ctx->enc.data.reset();
            to = &own;
        }
    }
    const sx::HostEncoding& enc = *to;
    // validate the styles and transforms that are actually used
    std::vector<sx::StyleD> sd(enc.style_stream.size());
    for (size_t i = 0; i < enc.style_stream.size(); i++) {
        const sx_style& st = styles[enc.style_stream[i]];
        if (st.flags & ~(uint32_t)SX_STYLE_FILL) return fail(ctx, SX_EINVAL, "reserved style flags");
        if (st.flags & SX_STYLE_FILL) {
            // a fill: offset 0, no joins or caps (width and join/cap fields ignored)
            sd[i] = sx::StyleD{0.0f, 1.0f, sx::kStyleFill};
            continue;
        }
        if (!(st.half_width >= 0.0f) || !std::isfinite(st.half_width)) return fail(ctx, SX_EINVAL, "half_width < 0");
        if (!(st.miter_limit >= 1.0f) || !std::isfinite(st.miter_limit)) return fail(ctx, SX_EINVAL, "miter_limit < 1");
        if (st.join > 2 || st.start_cap > 2 || st.end_cap > 2) return fail(ctx, SX_EINVAL, "bad join/cap");
        sd[i] = sx::StyleD{st.half_width, st.miter_limit,
                           (uint32_t)st.join | ((uint32_t)st.start_cap << 8) | ((uint32_t)st.end_cap << 16)};
    }
    // a transform drawn with a stroke must be a similarity, one drawn with a
    // fill an invertible finite affine map (checked per encoded path)
    for (uint32_t p = 0; p < (uint32_t)enc.path_map.size(); p++) {
        const uint32_t k = enc.path_map[p];
        const sx_affine& X = xforms[paths->xform_ix[k]];
        if (styles[paths->style_ix[k]].flags & SX_STYLE_FILL) {
            if (!invertible(X)) return fail(ctx, SX_EINVAL, "fill transforms must be invertible");
        } else if (!similarity(X)) {
            return fail(ctx, SX_EINVAL, "stroke transforms must be similarities");
        }
    }
    std::vector<float> xd(6 * enc.xform_stream.size());
    for (size_t i = 0; i < enc.xform_stream.size(); i++) {
        const sx_affine& X = xforms[enc.xform_stream[i]];
        const float v[6] = {X.a, X.b, X.c, X.d, X.e, X.f};
        memcpy(&xd[6 * i], v, sizeof(v));
    }
    SceneOwner own_s;
    sx_scene* s = own_s.s = new (std::nothrow) sx_scene();
    if (!s) return fail(ctx, SX_ENOMEM, "scene alloc");
    s->ctx = ctx;
    s->pool = ctx->pool;
    s->n_tags = (uint32_t)enc.tags.size();
    s->n_pts = (uint32_t)(enc.data.size() / 2);
    s->n_paths = (uint32_t)enc.path_map.size();
    s->n_styles = (uint32_t)sd.size();
    s->n_xforms = (uint32_t)enc.xform_stream.size();
    hipStream_t st = (hipStream_t)stream;
    hipError_t e = reserve_scene(s, s->n_tags, s->n_pts, s->n_styles, s->n_xforms, s->n_paths, st, streams_only);
    if (e != hipSuccess) return hip_fail(ctx, e, "scene allocation");
    auto A = [&](hipError_t r) {
        if (e == hipSuccess) e = r;
    };
    if (s->n_tags) A(hipMemcpyAsync(s->d_tags, enc.tags.data(), s->n_tags, hipMemcpyHostToDevice, st));
    if (s->n_pts)
        A(hipMemcpyAsync(s->d_pts, enc.data.data(), enc.data.size() * sizeof(float), hipMemcpyHostToDevice, st));
    if (!sd.empty()) A(hipMemcpyAsync(s->d_styles, sd.data(), sd.size() * sizeof(sx::StyleD), hipMemcpyHostToDevice, st));
    if (!xd.empty()) A(hipMemcpyAsync(s->d_xforms, xd.data(), xd.size() * sizeof(float), hipMemcpyHostToDevice, st));
    if (!enc.path_map.empty())
        A(hipMemcpyAsync(s->d_path_map, enc.path_map.data(), enc.path_map.size() * sizeof(uint32_t),
                         hipMemcpyHostToDevice, st));
    // host vectors die with this call: finish the uploads before returning
    A(hipStreamSynchronize(st));
    if (e != hipSuccess) return hip_fail(ctx, e, "scene upload");
    if (!streams_only) soup_terms(enc, styles, xforms, s->est);
    if (style_stream) *style_stream = enc.style_stream;
    s->last_stream = st;
    *out = own_s.give();
    return SX_OK;
}

int sx_scene_encode(sx_ctx* ctx, const sx_paths* paths, const sx_style* styles, uint32_t n_styles,
                    const sx_affine* xforms, uint32_t n_xforms, void* stream, sx_scene** out) {
    return guarded(ctx, [&] {
        return encode_impl(ctx, paths, styles, n_styles, xforms, n_xforms, stream, out, nullptr);
    });
}

static int encode_dashed(sx_ctx* ctx, const sx_paths* paths, const sx_style* styles, const sx_dash* dashes,
                         uint32_t n_styles, const sx_affine* xforms, uint32_t n_xforms, void* stream,
                         sx_scene** out) {
    if (!ctx || !out) return SX_EINVAL;
    *out = nullptr;
    if (n_styles && !dashes) return fail(ctx, SX_EINVAL, "null dash table");
    // the patterns on the 2^-24 grid, per user style (an odd array repeats once)
    std::vector<std::vector<int64_t>> pats(n_styles);
    std::vector<int64_t> phases(n_styles, 0), periods(n_styles, 0);
    for (uint32_t k = 0; k < n_styles; k++) {
        const sx_dash& d = dashes[k];
        if (d.count > 32u || (d.count && !d.array) || !std::isfinite(d.offset))
            return fail(ctx, SX_EINVAL, "bad dash pattern");
        if (styles && (styles[k].flags & SX_STYLE_FILL)) continue;  // fills are not dashed
        const uint32_t m = (d.count & 1u) ? 2u * d.count : d.count;
        int64_t period = 0;
        for (uint32_t j = 0; j < m; j++) {
            const float v = d.array[j % d.count];
            if (!(v >= 0.0f) || !std::isfinite(v)) return fail(ctx, SX_EINVAL, "bad dash pattern");
            pats[k].push_back(sx::dash_fix((double)v));
            period += pats[k].back();
        }
        if (period <= 0) {
            pats[k].clear();  // nothing to dash: solid
            continue;
        }
        // a period below 2^-10 units would cut every unit of length into
        // thousands of dashes (and as many loop turns per segment)
        if (period < ((int64_t)1 << 14)) return fail(ctx, SX_EINVAL, "dash pattern period below 2^-10 units");
        int64_t ph = sx::dash_fix((double)d.offset) % period;
        phases[k] = ph < 0 ? ph + period : ph;
        periods[k] = period;
    }
    hipStream_t st = (hipStream_t)stream;
    std::vector<uint32_t> sstream;
    SceneOwner own_src, own_dst;
    sx_scene*& src = own_src.s;
    sx_scene*& dst = own_dst.s;
    int r = encode_impl(ctx, paths, styles, n_styles, xforms, n_xforms, stream, &src, &sstream, true);
    if (r != SX_OK) return r;
    const uint32_t n = src->n_tags;
    // per style entry of the scene: its user style's pattern
    std::vector<sx::DashDesc> desc(sstream.size());
    std::vector<int64_t> pat;
    for (size_t e = 0; e < sstream.size(); e++) {
        const uint32_t k = sstream[e];
        desc[e] = sx::DashDesc{(uint32_t)pat.size(), (uint32_t)pats[k].size(), periods[k], phases[k]};
        pat.insert(pat.end(), pats[k].begin(), pats[k].end());
    }
    // coordinates within 2^24 units keep every segment's grid length below
    // 2^53 and a subpath's below 2^63 for any realistic segment count
    {
        const uint32_t np = paths->n_paths ? paths->pt_off[paths->n_paths] : 0u;
        for (uint32_t j = 0; j < 2u * np; j++)
            if (!(std::fabs(paths->pts[j]) <= 16777216.0f))
                return fail(ctx, SX_EINVAL, "dashed paths need coordinates within 2^24 units");
    }
    hipError_t e = hipSuccess;
    auto A = [&](hipError_t x) {
        if (e == hipSuccess) e = x;
    };
    sx::DashBufs b{};
    bool idle = false;  // the device has been waited for
    auto dalloc = [&](auto** p, size_t bytes) { return ctx->pool->take((void**)p, bytes); };
    auto dfree = [&](auto*& p) {
        ctx->pool->give((void*)p, idle);
        p = nullptr;
    };
    // (nothing throws from here on)
    // device time of the three dashing phases (the host reads the sizes and
    // allocates between them)
    hipEvent_t ev[6] = {nullptr, nullptr, nullptr, nullptr, nullptr, nullptr};
    uint64_t n_ch = 0, tot_t = 0, tot_p = 0;
    uint32_t too_fine = 0;
    const size_t nn = (size_t)n + 2;
    A(dalloc(&b.desc, std::max<size_t>(desc.size(), 1) * sizeof(sx::DashDesc)));
    A(dalloc(&b.pat, std::max<size_t>(pat.size(), 1) * sizeof(int64_t)));
    A(dalloc(&b.panels, (size_t)std::max<uint32_t>(n, 1u) * sx::kDashPanels * sizeof(double)));
    A(dalloc(&b.len, nn * sizeof(uint64_t)));
    A(dalloc(&b.cum, nn * sizeof(uint64_t)));
    A(dalloc(&b.sub_start, nn * sizeof(uint64_t)));
    A(dalloc(&b.subix, nn * sizeof(uint32_t)));
    A(dalloc(&b.nch, nn * sizeof(uint32_t)));
    A(dalloc(&b.chb, nn * sizeof(uint64_t)));
    A(dalloc(&b.flag, sizeof(uint32_t)));
    A(dalloc(&b.ctl0, sx::scan_ctl_bytes()));
    A(dalloc(&b.ctl1, sx::scan_ctl_bytes()));
    A(dalloc(&b.ctl2, sx::scan_ctl_bytes()));
    A(dalloc(&b.st0, sx::scan_status_bytes(n)));
    A(dalloc(&b.st1, sx::scan_status_bytes(n)));
    for (auto& x : ev) A(hipEventCreate(&x));
    if (e == hipSuccess && !desc.empty())
        e = hipMemcpyAsync(b.desc, desc.data(), desc.size() * sizeof(sx::DashDesc), hipMemcpyHostToDevice, st);
    if (e == hipSuccess && !pat.empty())
        e = hipMemcpyAsync(b.pat, pat.data(), pat.size() * sizeof(int64_t), hipMemcpyHostToDevice, st);
    if (e == hipSuccess)
        e = sx::launch_zero({{b.ctl0, sx::scan_ctl_bytes()},
                             {b.ctl1, sx::scan_ctl_bytes()},
                             {b.ctl2, sx::scan_ctl_bytes()},
                             {b.st0, sx::scan_status_bytes(n)},
                             {b.st1, sx::scan_status_bytes(n)},
                             {b.flag, sizeof(uint32_t)}},
                            st);
    if (e == hipSuccess && n)
        e = sx::launch_scan_tags(src->d_tags, n, src->d_mon, ctl_block(src, 0), src->d_status_tags, nullptr, st);
    // phase 0: lengths, positions, subpath starts, chunks per tag and their scan
    A(hipEventRecord(ev[0], st));
    if (e == hipSuccess) e = sx::launch_dash(view(src), b, 0, nullptr, nullptr, st);
    A(hipEventRecord(ev[1], st));
    if (e == hipSuccess && n) e = hipMemcpyAsync(&n_ch, b.chb + n, sizeof(uint64_t), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess && n) e = hipMemcpyAsync(&too_fine, b.flag, sizeof(uint32_t), hipMemcpyDeviceToHost, st);
    A(hipStreamSynchronize(st));
    if (e == hipSuccess && (too_fine || n_ch > (uint64_t)INT32_MAX))
        r = fail(ctx, SX_EINVAL, "dash pattern too fine for the segment lengths");
    // phase 1: chunk owners, per-chunk counts and their scan
    if (e == hipSuccess && r == SX_OK && n) {
        b.n_ch = (uint32_t)n_ch;
        const size_t nc = (size_t)n_ch + 2;
        A(dalloc(&b.ch_tag, nc * sizeof(uint32_t)));
        A(dalloc(&b.cnt, nc * sizeof(uint2)));
        A(dalloc(&b.otag, nc * sizeof(uint64_t)));
        A(dalloc(&b.opt, nc * sizeof(uint64_t)));
        A(dalloc(&b.st2, sx::scan_status_bytes(b.n_ch)));
        if (e == hipSuccess) e = sx::launch_zero({{b.st2, sx::scan_status_bytes(b.n_ch)}}, st);
        A(hipEventRecord(ev[2], st));
        if (e == hipSuccess) e = sx::launch_dash(view(src), b, 1, nullptr, nullptr, st);
        A(hipEventRecord(ev[3], st));
        if (e == hipSuccess) e = hipMemcpyAsync(&tot_t, b.otag + b.n_ch, sizeof(uint64_t), hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipMemcpyAsync(&tot_p, b.opt + b.n_ch, sizeof(uint64_t), hipMemcpyDeviceToHost, st);
        A(hipStreamSynchronize(st));
    }
    if (e == hipSuccess && r == SX_OK && (tot_t > UINT32_MAX - 64 || tot_p > UINT32_MAX)) {
        r = fail(ctx, SX_EINVAL, "dashed scene exceeds 32-bit stream sizes");
    } else if (e == hipSuccess && r == SX_OK) {
        dst = new (std::nothrow) sx_scene();
        if (!dst) e = hipErrorOutOfMemory;
    }
    // phase 2: the write pass into the result scene
    if (e == hipSuccess && r == SX_OK) {
        dst->ctx = ctx;
        dst->pool = ctx->pool;
        dst->n_tags = (uint32_t)tot_t;
        dst->n_pts = (uint32_t)tot_p;
        dst->n_paths = src->n_paths;
        dst->n_styles = src->n_styles;
        dst->n_xforms = src->n_xforms;
        e = reserve_scene(dst, dst->n_tags, dst->n_pts, dst->n_styles, dst->n_xforms, dst->n_paths, st);
        A(hipEventRecord(ev[4], st));
        if (e == hipSuccess && n) e = sx::launch_dash(view(src), b, 2, dst->d_tags, dst->d_pts, st);
        A(hipEventRecord(ev[5], st));
        if (e == hipSuccess && src->n_styles)
            e = hipMemcpyAsync(dst->d_styles, src->d_styles, src->n_styles * sizeof(sx::StyleD),
                               hipMemcpyDeviceToDevice, st);
        if (e == hipSuccess && src->n_xforms)
            e = hipMemcpyAsync(dst->d_xforms, src->d_xforms, src->n_xforms * 6 * sizeof(float),
                               hipMemcpyDeviceToDevice, st);
        if (e == hipSuccess && src->n_paths)
            e = hipMemcpyAsync(dst->d_path_map, src->d_path_map, src->n_paths * sizeof(uint32_t),
                               hipMemcpyDeviceToDevice, st);
        A(hipStreamSynchronize(st));
        float ms[3] = {0.0f, 0.0f, 0.0f};
        if (e == hipSuccess && n && hipEventElapsedTime(&ms[0], ev[0], ev[1]) == hipSuccess &&
            hipEventElapsedTime(&ms[1], ev[2], ev[3]) == hipSuccess &&
            hipEventElapsedTime(&ms[2], ev[4], ev[5]) == hipSuccess)
            dst->dash_ms = ms[0] + ms[1] + ms[2];
    }
    idle = ctx->pool->idle();
    dfree(b.desc);
    dfree(b.pat);
    dfree(b.panels);
    dfree(b.len);
    dfree(b.cum);
    dfree(b.sub_start);
    dfree(b.subix);
    dfree(b.nch);
    dfree(b.chb);
    dfree(b.flag);
    dfree(b.ch_tag);
    dfree(b.cnt);
    dfree(b.otag);
    dfree(b.opt);
    dfree(b.ctl0);
    dfree(b.ctl1);
    dfree(b.ctl2);
    dfree(b.st0);
    dfree(b.st1);
    dfree(b.st2);
    for (auto& x : ev)
        if (x) (void)hipEventDestroy(x);
    if (e != hipSuccess || r != SX_OK) return r != SX_OK ? r : hip_fail(ctx, e, "dashed encoding");
    dst->last_stream = st;
    *out = own_dst.give();
    return SX_OK;
}

int sx_scene_encode_dashed(sx_ctx* ctx, const sx_paths* paths, const sx_style* styles, const sx_dash* dashes,
                           uint32_t n_styles, const sx_affine* xforms, uint32_t n_xforms, void* stream,
                           sx_scene** out) {
    return guarded(ctx, [&] {
        return encode_dashed(ctx, paths, styles, dashes, n_styles, xforms, n_xforms, stream, out);
    });
}

int sx_scene_dash_ms(const sx_scene* s, float* ms) {
    if (!s || !ms) return SX_EINVAL;
    *ms = s->dash_ms;
    return SX_OK;
}

int sx_scene_release(sx_ctx* ctx, sx_scene* scene) {
    if (!scene) return SX_OK;
    if (ctx && scene->ctx != ctx) return fail(ctx, SX_EINVAL, "scene belongs to another context");
    if (scene->batch_arena) return fail(ctx, SX_EINVAL, "a batch arena is released with its batch");
    (void)hipStreamSynchronize(scene->last_stream);
    free_scene(scene);
    return SX_OK;
}

int sx_scene_info(const sx_scene* s, uint32_t* n_tags, uint32_t* n_pts, uint32_t* n_paths, uint32_t* n_styles,
                  uint32_t* n_xforms) {
    if (!s) return SX_EINVAL;
    if (n_tags) *n_tags = s->n_tags;
    if (n_pts) *n_pts = s->n_pts;
    if (n_paths) *n_paths = s->n_paths;
    if (n_styles) *n_styles = s->n_styles;
    if (n_xforms) *n_xforms = s->n_xforms;
    return SX_OK;
}

int sx_scene_download(const sx_scene* s, uint8_t* tags, float* data, uint32_t* path_map) {
    if (!s) return SX_EINVAL;
    hipError_t e = hipSuccess;
    if (tags && s->n_tags) e = hipMemcpy(tags, s->d_tags, s->n_tags, hipMemcpyDeviceToHost);
    if (e == hipSuccess && data && s->n_pts)
        e = hipMemcpy(data, s->d_pts, (size_t)s->n_pts * sizeof(float2), hipMemcpyDeviceToHost);
    if (e == hipSuccess && path_map && s->n_paths)
        e = hipMemcpy(path_map, s->d_path_map, (size_t)s->n_paths * sizeof(uint32_t), hipMemcpyDeviceToHost);
    return e == hipSuccess ? SX_OK : SX_EDEVICE;
}

int sx_expand_async(sx_ctx* ctx, const sx_scene* scene, float tolerance, int output_mode, void* out_dev,
                    uint64_t out_capacity_bytes, uint64_t* out_count_dev, void* stream) {
    if (!ctx || !scene) return SX_EINVAL;
    sx::Cfg cfg;
    if (!make_cfg(ctx, tolerance, output_mode, cfg)) return fail(ctx, SX_EINVAL, "bad tolerance or output mode");
    if (!out_count_dev) return fail(ctx, SX_EINVAL, "null count pointer");
    if (out_capacity_bytes && !out_dev) return fail(ctx, SX_EINVAL, "null output buffer");
    hipStream_t st = (hipStream_t)stream;
    const_cast<sx_scene*>(scene)->last_stream = st;
    const uint64_t rec = output_mode == SX_OUT_ARCS ? sizeof(sx_arc) : sizeof(sx_line);
    return run_all(ctx, scene, cfg, out_dev, out_capacity_bytes / rec, out_count_dev, st);
}

int sx_expand(sx_ctx* ctx, const sx_scene* scene, float tolerance, int output_mode, void* out_dev,
              uint64_t out_capacity_bytes, uint64_t* out_count, void* stream) {
    if (!ctx || !scene || !out_count) return SX_EINVAL;
    sx::Cfg cfg;
    if (!make_cfg(ctx, tolerance, output_mode, cfg)) return fail(ctx, SX_EINVAL, "bad tolerance or output mode");
    if (out_capacity_bytes && !out_dev) return fail(ctx, SX_EINVAL, "null output buffer");
    hipStream_t st = (hipStream_t)stream;
    sx_scene* s = const_cast<sx_scene*>(scene);
    s->last_stream = st;
    const uint64_t rec = output_mode == SX_OUT_ARCS ? sizeof(sx_arc) : sizeof(sx_line);
    *out_count = 0;
    if (s->n_tags == 0) return SX_OK;
    int r = run_sized(ctx, s, cfg, out_dev, out_capacity_bytes / rec, out_count, st);
    if (r != SX_OK) return r;
    if (*out_count > out_capacity_bytes / rec) return fail(ctx, SX_ETOOSMALL, "output buffer too small");
    return SX_OK;
}

int sx_run_phase(sx_ctx* ctx, const sx_scene* s, int phase, float tolerance, int output_mode, void* out_dev,
                 uint64_t out_capacity_bytes, void* stream) {
    if (!ctx || !s) return SX_EINVAL;
    sx::Cfg cfg;
    if (!make_cfg(ctx, tolerance, output_mode, cfg)) return fail(ctx, SX_EINVAL, "bad tolerance or output mode");
    if (phase < 0 || phase >= kPhN) return fail(ctx, SX_EINVAL, "bad phase");
    if (phase == kPhRecords && out_capacity_bytes && !out_dev) return fail(ctx, SX_EINVAL, "null output buffer");
    if (s->n_tags == 0) return SX_OK;
    if (!allocated(s)) return fail(ctx, SX_ENOMEM, "workspace");
    hipStream_t st = (hipStream_t)stream;
    const_cast<sx_scene*>(s)->last_stream = st;
    const uint64_t rec = output_mode == SX_OUT_ARCS ? sizeof(sx_arc) : sizeof(sx_line);
    hipError_t e = hipSuccess;
    // (the bisection alone, again and again: its codes go to the same place)
    if (phase == kPhBisectCount)
        e = sx::launch_zero({{&s->d_ws_ctl->ordered_n, sizeof(s->d_ws_ctl->ordered_n)},
                             {&s->d_ws_ctl->rich_n, sizeof(s->d_ws_ctl->rich_n)}},
                            st);
    if (e == hipSuccess) e = run_one(ctx, s, cfg, phase, out_dev, out_capacity_bytes / rec, nullptr, st);
    return e == hipSuccess ? SX_OK : hip_fail(ctx, e, "phase launch");
}

int sx_batch_create(sx_ctx* ctx, sx_batch** out) {
    if (!ctx || !out) return SX_EINVAL;
    *out = nullptr;
    if (hipSetDevice(ctx->device) != hipSuccess) return fail(ctx, SX_EDEVICE, "hipSetDevice");
    sx_batch* b = new (std::nothrow) sx_batch();
    if (!b) return fail(ctx, SX_ENOMEM, "batch alloc");
    b->ctx = ctx;
    b->arena = new (std::nothrow) sx_scene();
    if (!b->arena) {
        delete b;
        return fail(ctx, SX_ENOMEM, "batch alloc");
    }
    b->arena->ctx = ctx;
    b->arena->pool = ctx->pool;
    b->arena->batch_arena = true;
    hipError_t e = hipEventCreateWithFlags(&b->staged, hipEventDisableTiming);
    if (e == hipSuccess) e = reserve_scene(b->arena, 0, 0, 0, 0, 0, nullptr);
    if (e == hipSuccess) e = hipStreamSynchronize(nullptr);
    if (e != hipSuccess) {
        if (b->staged) (void)hipEventDestroy(b->staged);
        free_scene(b->arena);
        delete b;
        return hip_fail(ctx, e, "batch creation");
    }
    *out = b;
    return SX_OK;
}

int sx_batch_destroy(sx_ctx* ctx, sx_batch* b) {
    if (!b) return SX_OK;
    if (ctx && b->ctx != ctx) return fail(ctx, SX_EINVAL, "batch belongs to another context");
    (void)hipStreamSynchronize(b->arena->last_stream);
    (void)hipEventSynchronize(b->staged);
    if (b->d_desc) (void)hipFree(b->d_desc);
    if (b->h_desc) (void)hipHostFree(b->h_desc);
    (void)hipEventDestroy(b->staged);
    free_scene(b->arena);
    delete b;
    return SX_OK;
}

int sx_batch_set(sx_ctx* ctx, sx_batch* b, const sx_scene* const* scenes, uint32_t n, void* stream) {
    if (!ctx || !b || (n && !scenes)) return SX_EINVAL;
    if (b->ctx != ctx) return fail(ctx, SX_EINVAL, "batch belongs to another context");
    if (n > kMaxBatchScenes) return fail(ctx, SX_EINVAL, "too many scenes in one batch");
    uint64_t nt = 0, np = 0, ns = 0, nx = 0, npa = 0;
    for (uint32_t i = 0; i < n; i++) {
        const sx_scene* sc = scenes[i];
        if (!sc || sc->ctx != ctx) return fail(ctx, SX_EINVAL, "null scene or scene of another context");
        if (sc->batch_arena) return fail(ctx, SX_EINVAL, "a batch arena cannot be batched");
        nt += sc->n_tags;
        np += sc->n_pts;
        ns += sc->n_styles;
        nx += sc->n_xforms;
        npa += sc->n_paths;
    }
    if (nt > UINT32_MAX - 64 || np > UINT32_MAX || ns > UINT32_MAX || nx > UINT32_MAX / 6 || npa > UINT32_MAX)
        return fail(ctx, SX_EINVAL, "batch exceeds 32-bit stream sizes");
    hipStream_t st = (hipStream_t)stream;
    // the staging buffer is reused: wait until its previous upload is done
    hipError_t e = hipEventSynchronize(b->staged);
    if (e == hipSuccess && n > b->cap_scenes) {
        if (b->d_desc) (void)hipFree(b->d_desc);
        if (b->h_desc) (void)hipHostFree(b->h_desc);
        b->d_desc = nullptr;
        b->h_desc = nullptr;
        b->cap_scenes = 0;
        e = hipMalloc((void**)&b->d_desc, (size_t)n * sizeof(sx::GatherDesc));
        if (e == hipSuccess) e = hipHostMalloc((void**)&b->h_desc, (size_t)n * sizeof(sx::GatherDesc), hipHostMallocDefault);
        if (e == hipSuccess) b->cap_scenes = n;
    }
    if (e == hipSuccess)
        e = reserve_scene(b->arena, (uint32_t)nt, (uint32_t)np, (uint32_t)ns, (uint32_t)nx, (uint32_t)npa, st);
    if (e != hipSuccess) return hip_fail(ctx, e, "batch allocation");
    uint32_t tb = 0, pb = 0, sb = 0, xb = 0, ab = 0;
    for (uint32_t i = 0; i < n; i++) {
        const sx_scene* sc = scenes[i];
        sx::GatherDesc& d = b->h_desc[i];
        d.tags = sc->d_tags;
        d.pts = sc->d_pts;
        d.styles = sc->d_styles;
        d.xforms = sc->d_xforms;
        d.path_map = sc->d_path_map;
        d.n_tags = sc->n_tags;
        d.n_pts = sc->n_pts;
        d.n_styles = sc->n_styles;
        d.n_xforms = sc->n_xforms;
        d.n_paths = sc->n_paths;
        d.tag_base = tb;
        d.pt_base = pb;
        d.style_base = sb;
        d.xform_base = xb;
        d.path_base = ab;
        d.pad = 0;
        tb += sc->n_tags;
        pb += sc->n_pts;
        sb += sc->n_styles;
        xb += sc->n_xforms;
        ab += sc->n_paths;
    }
    sx_scene* a = b->arena;
    a->n_tags = tb;
    a->n_pts = pb;
    a->n_styles = sb;
    a->n_xforms = xb;
    a->n_paths = ab;
    b->n_scenes = n;
    a->last_stream = st;
    if (n) {
        e = hipMemcpyAsync(b->d_desc, b->h_desc, (size_t)n * sizeof(sx::GatherDesc), hipMemcpyHostToDevice, st);
        if (e == hipSuccess) e = hipEventRecord(b->staged, st);
        if (e == hipSuccess)
            e = sx::launch_gather(b->d_desc, n, a->d_tags, a->d_pts, a->d_styles, a->d_xforms, a->d_path_map, st);
        if (e != hipSuccess) return hip_fail(ctx, e, "batch gather");
    }
    return SX_OK;
}

int sx_batch_info(const sx_batch* b, uint32_t* n_scenes, sx_scene** arena) {
    if (!b) return SX_EINVAL;
    if (n_scenes) *n_scenes = b->n_scenes;
    if (arena) *arena = b->arena;
    return SX_OK;
}

int sx_batch_expand(sx_ctx* ctx, sx_batch* b, float tolerance, int output_mode, void* out_dev,
                    uint64_t out_capacity_bytes, uint64_t* scene_offsets_dev, uint64_t* status_dev, void* stream) {
    if (!ctx || !b || !scene_offsets_dev || !status_dev) return SX_EINVAL;
    if (b->ctx != ctx) return fail(ctx, SX_EINVAL, "batch belongs to another context");
    sx::Cfg cfg;
    if (!make_cfg(ctx, tolerance, output_mode, cfg)) return fail(ctx, SX_EINVAL, "bad tolerance or output mode");
    if (out_capacity_bytes && !out_dev) return fail(ctx, SX_EINVAL, "null output buffer");
    hipStream_t st = (hipStream_t)stream;
    sx_scene* a = b->arena;
    a->last_stream = st;
    const uint64_t rec = output_mode == SX_OUT_ARCS ? sizeof(sx_arc) : sizeof(sx_line);
    int r = run_all(ctx, a, cfg, out_dev, out_capacity_bytes / rec, status_dev, st);
    if (r != SX_OK) return r;
    hipError_t e = sx::launch_scene_offsets(a->d_base, a->d_roff, a->slot_cap, b->d_desc, b->n_scenes, a->n_tags,
                                            scene_offsets_dev, st);
    return e == hipSuccess ? SX_OK : hip_fail(ctx, e, "scene offsets");
}

int sx_debug_piece_stats(sx_ctx* ctx, const sx_scene* s, float tolerance, int output_mode, uint64_t* stats6,
                         void* stream) {
    if (!ctx || !s || !stats6) return SX_EINVAL;
    sx::Cfg cfg;
    if (!make_cfg(ctx, tolerance, output_mode, cfg)) return fail(ctx, SX_EINVAL, "bad tolerance or output mode");
    for (int j = 0; j < 6; j++) stats6[j] = 0;
    if (s->n_tags == 0) return SX_OK;
    hipStream_t st = (hipStream_t)stream;
    sx_scene* sc = const_cast<sx_scene*>(s);
    // size the workspace first, so the instrumented run covers every slot
    uint64_t n_rec = 0;
    int r = run_sized(ctx, sc, cfg, nullptr, 0, &n_rec, st);
    if (r != SX_OK) return r;
    unsigned long long* d = nullptr;
    hipError_t e = hipMalloc((void**)&d, 6 * sizeof(unsigned long long));
    if (e == hipSuccess) e = hipMemsetAsync(d, 0, 6 * sizeof(unsigned long long), st);
    for (int ph = 0; ph <= kPhTails && e == hipSuccess; ph++) {
        const bool counted = ph == kPhBisectCount || ph == kPhPieces || ph == kPhTails;
        e = run_one(ctx, sc, cfg, ph, nullptr, 0, counted ? d : nullptr, st);
    }
    if (e == hipSuccess) e = hipMemcpyAsync(stats6, d, 6 * sizeof(uint64_t), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (d) (void)hipFree(d);
    return e == hipSuccess ? SX_OK : hip_fail(ctx, e, "piece stats");
}

int sx_debug_monoids(sx_ctx* ctx, const sx_scene* s, uint32_t* out4xn_dev, void* stream) {
    if (!ctx || !s || (!out4xn_dev && s->n_tags)) return SX_EINVAL;
    if (s->n_tags > s->cap_tags) return fail(ctx, SX_ENOMEM, "workspace");
    hipStream_t st = (hipStream_t)stream;
    hipError_t e = sx::launch_scan_tags(s->d_tags, s->n_tags, s->d_mon, ctl_block(s, 0), s->d_status_tags, nullptr, st);
    const size_t stride = sx::mon_stride_of(s->n_tags);
    for (int k = 0; k < 4 && e == hipSuccess && s->n_tags; k++)
        e = hipMemcpyAsync(out4xn_dev + k * (size_t)s->n_tags, s->d_mon + k * stride, (size_t)s->n_tags * sizeof(uint32_t),
                           hipMemcpyDeviceToDevice, st);
    return e == hipSuccess ? SX_OK : hip_fail(ctx, e, "monoids");
}

// per-tag record counts and / or offsets after a sized run of the pipeline
static int tag_records(sx_ctx* ctx, const sx_scene* s, float tolerance, int output_mode, uint32_t* counts,
                       uint64_t* offs, void* stream) {
    sx::Cfg cfg;
    if (!make_cfg(ctx, tolerance, output_mode, cfg)) return fail(ctx, SX_EINVAL, "bad tolerance or output mode");
    hipStream_t st = (hipStream_t)stream;
    if (s->n_tags == 0) {
        if (!offs) return SX_OK;
        hipError_t e = hipMemsetAsync(offs, 0, sizeof(uint64_t), st);
        return e == hipSuccess ? SX_OK : hip_fail(ctx, e, "memset");
    }
    uint64_t n_rec = 0;
    int r = run_sized(ctx, const_cast<sx_scene*>(s), cfg, nullptr, 0, &n_rec, st);
    if (r != SX_OK) return r;
    hipError_t e = sx::launch_tag_records(s->d_base, s->d_roff, s->slot_cap, s->n_tags, counts, offs, st);
    return e == hipSuccess ? SX_OK : hip_fail(ctx, e, "tag records");
}

int sx_debug_counts(sx_ctx* ctx, const sx_scene* s, float tolerance, int output_mode, uint32_t* counts_dev,
                    void* stream) {
    if (!ctx || !s || (!counts_dev && s->n_tags)) return SX_EINVAL;
    return tag_records(ctx, s, tolerance, output_mode, counts_dev, nullptr, stream);
}

int sx_debug_offsets(sx_ctx* ctx, const sx_scene* s, float tolerance, int output_mode, uint64_t* offsets_dev,
                     void* stream) {
    if (!ctx || !s || !offsets_dev) return SX_EINVAL;
    return tag_records(ctx, s, tolerance, output_mode, nullptr, offsets_dev, stream);
}

int sx_scan_u32(sx_ctx* ctx, const uint32_t* in_dev, uint64_t* out_dev, uint32_t n, void* stream) {
    if (!ctx || !out_dev || (n && !in_dev)) return SX_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    if (n == 0) {
        hipError_t e = hipMemsetAsync(out_dev, 0, sizeof(uint64_t), st);
        return e == hipSuccess ? SX_OK : hip_fail(ctx, e, "memset");
    }
    void *ctl = nullptr, *status = nullptr;
    hipError_t e = hipMalloc(&ctl, sx::scan_ctl_bytes());
    if (e == hipSuccess) e = hipMalloc(&status, sx::scan_status_bytes(n));
    if (e == hipSuccess) e = hipMemsetAsync(ctl, 0, sx::scan_ctl_bytes(), st);
    if (e == hipSuccess) e = hipMemsetAsync(status, 0, sx::scan_status_bytes(n), st);
    if (e == hipSuccess) e = sx::launch_scan_counts(in_dev, n, out_dev, ctl, status, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (ctl) (void)hipFree(ctl);
    if (status) (void)hipFree(status);
    return e == hipSuccess ? SX_OK : hip_fail(ctx, e, "scan_u32");
}

int sx_scan_u32_noalloc(sx_ctx* ctx, const uint32_t* in_dev, uint64_t* out_dev, uint32_t n, void* stream) {
    if (!ctx || !out_dev || (n && !in_dev)) return SX_EINVAL;
    if (n > SX_SCAN_NOALLOC_MAX) return fail(ctx, SX_EINVAL, "n exceeds SX_SCAN_NOALLOC_MAX");
    static_assert(SX_SCAN_NOALLOC_BYTES >= 256u, "control block");
    if (sx::scan_ctl_bytes() > 256u || sx::scan_status_bytes(SX_SCAN_NOALLOC_MAX) > SX_SCAN_NOALLOC_BYTES - 256u)
        return fail(ctx, SX_EDEVICE, "scan scratch layout");
    if (!ctx->scratch) return fail(ctx, SX_EDEVICE, "scratch address lookup failed");
    hipStream_t st = (hipStream_t)stream;
    char* base = (char*)ctx->scratch;
    hipError_t e = n == 0 ? sx::launch_zero_u64(out_dev, st)
                          : sx::launch_scan_counts(in_dev, n, out_dev, base, base + 256, st);
    return e == hipSuccess ? SX_OK : hip_fail(ctx, e, "scan_u32_noalloc");
}

// ------------------------------------------------------------ single pass
constexpr int kSoupEnabled = 0;

int sx_scene_estimate(const sx_scene* s, float tolerance, int output_mode, uint64_t* out_records) {
    if (!s || !out_records) return SX_EINVAL;
    sx::Cfg cfg;
    if (!make_cfg(s->ctx, tolerance, output_mode, cfg)) return SX_EINVAL;
    const double tf = cfg.tau_flat, rtf = 1.0 / std::sqrt(tf);
    uint64_t total = 0;
    for (const SoupTerm& e : s->est) {
        const double a = e.a, b = e.b, w = e.w;
        const uint32_t fl = e.flags;
        const bool fill = (fl & kEstFill) != 0;
        uint64_t tail = 0;
        if (!fill) tail = (fl & kEstRound) ? (w > tf ? (uint64_t)std::ceil(sx::kHalfPi / std::acos(1.0 - tf / w)) : 2u) + 4u
                                           : 6u;
        uint64_t n = tail;
        if (fl & kEstLine) {
            n += fill ? 1u : 2u;
        } else if (fl & kEstCurve) {
            const double base = a * rtf;
            // both sides inflated, plus room for the evolute bundles of a stroke
            n += (fill ? 1u : 2u) * (uint64_t)std::ceil(base * b) + (fill ? 0u : 2u * (uint64_t)std::ceil(base)) + 2u;
        }
        total += n;
    }
    *out_records = total;
    return SX_OK;
}

int sx_expand_soup(sx_ctx* ctx, sx_scene* s, float tolerance, int output_mode, void* out_dev,
                   uint64_t out_capacity_bytes, uint64_t* out_count, void* stream) {
    if (!ctx || !s || !out_count) return SX_EINVAL;
    sx::Cfg cfg;
    if (!make_cfg(ctx, tolerance, output_mode, cfg)) return fail(ctx, SX_EINVAL, "bad tolerance or output mode");
    if (out_capacity_bytes && !out_dev) return fail(ctx, SX_EINVAL, "null output buffer");
    hipStream_t st = (hipStream_t)stream;
    *out_count = 0;
    if (s->n_tags == 0) return SX_OK;
    // Switched off: soup_kernel has been seen not to finish on gfx950 and the
    // cause is not known (its loops are bounded, and the same sink compiled
    // for the host reproduces the ordered records exactly).  Nothing is
    // launched until the cause is found.
    if (kSoupEnabled == 0) return fail(ctx, SX_EDEVICE, "single-pass expansion is switched off");
    s->last_stream = st;
    const uint64_t rec = output_mode == SX_OUT_ARCS ? sizeof(sx_arc) : sizeof(sx_line);
    hipError_t e = hipSuccess;
    if (!s->d_soup_n) e = hipMalloc((void**)&s->d_soup_n, sizeof(unsigned long long));
    if (e == hipSuccess) e = hipMemsetAsync(s->d_soup_n, 0, sizeof(unsigned long long), st);
    if (e == hipSuccess)
        e = sx::launch_scan_tags(s->d_tags, s->n_tags, s->d_mon, ctl_block(s, 0), s->d_status_tags, nullptr, st);
    if (e == hipSuccess) e = sx::launch_soup(view(s), cfg, out_dev, out_capacity_bytes / rec, s->d_soup_n, st);
    unsigned long long n = 0;
    if (e == hipSuccess) e = hipMemcpyAsync(&n, s->d_soup_n, sizeof(n), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return hip_fail(ctx, e, "single-pass expansion");
    *out_count = n;
    if (n > out_capacity_bytes / rec) return fail(ctx, SX_ETOOSMALL, "output buffer too small");
    return SX_OK;
}

}  // extern "C"
