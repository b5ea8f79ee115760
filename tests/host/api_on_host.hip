// Test shim: the library's host side (sx_api.hip, as it is) over a stand-in
// for the HIP runtime, so that the CPU suite can run its entry points where an
// allocation fails.  Device memory is host memory, copies are memcpy, and a
// launch only checks the addresses it is given and leaves the sizes that the
// host reads back.  Test infrastructure only.
#include <cstdlib>
#include <map>
#include <set>

#include "sx_api.hip"

namespace {
std::map<void*, size_t> g_live;  // allocations, device and pinned
size_t g_dev_bytes, g_pin_most;  // device bytes held, largest pinned request
long g_calls, g_fail = -1;       // allocations so far; the first one that fails (-2: every pinned one)
size_t g_limit = ~(size_t)0;     // device bytes there are
int g_bad;                       // launches given a null address, frees of what is not live
int g_capture;                   // 1: a stream is being captured, relaxed; 2: its capture was ended by a wait
hipError_t g_last = hipSuccess;
int g_new_fail = -1;             // C++ allocations until one fails
sx::WsCtl g_result;              // what the next expansion leaves

hipError_t out(hipError_t e) {
    if (e != hipSuccess) g_last = e;
    return e;
}
struct Quiet {  // the stand-in's own C++ allocations do not fail
    int k = g_new_fail;
    Quiet() { g_new_fail = -1; }
    ~Quiet() { g_new_fail = k; }
};
void need(std::initializer_list<const void*> ps) {
    for (const void* p : ps)
        if (!p) g_bad++;
}
bool fails() { return g_calls++ >= g_fail && g_fail >= 0; }
hipError_t launched() {
    const hipError_t e = g_last;  // as hipGetLastError after a launch
    g_last = hipSuccess;
    return e;
}
}  // namespace

void* operator new(size_t n) {
    if (g_new_fail >= 0 && g_new_fail-- == 0) throw std::bad_alloc();
    if (void* p = malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }

extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
    Quiet q;
    *p = nullptr;
    // (16 bytes: the pool's wait for the device, which no call depends on)
    if ((n > 16 && fails()) || g_dev_bytes + n > g_limit) return out(hipErrorOutOfMemory);
    // (only what the host side touches is backed: the tests stay small)
    *p = calloc(1, n < ((size_t)1 << 22) ? n : (size_t)1 << 22);
    g_live[*p] = n;
    g_dev_bytes += n;
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    const auto it = g_live.find(p);
    if (it == g_live.end()) {
        g_bad++;
        return out(hipErrorInvalidValue);
    }
    g_dev_bytes -= it->second;
    g_live.erase(it);
    free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
    Quiet q;
    *p = nullptr;
    if (n > g_pin_most) g_pin_most = n;
    if (fails() || g_fail == -2) return out(hipErrorOutOfMemory);
    *p = malloc(n);
    g_live[*p] = 0;
    return hipSuccess;
}
hipError_t hipHostFree(void* p) { return hipFree(p); }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
    need({d, s});
    if (d && s) memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t) { return hipMemcpy(d, s, n, k); }
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
    if (!d) return out(hipErrorInvalidValue);
    memset(d, v, n);
    return hipSuccess;
}
hipError_t hipDeviceSynchronize() {
    if (!g_capture) return hipSuccess;
    g_capture = 2;
    return out(hipErrorStreamCaptureUnsupported);
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipGetDeviceCount(int* n) { return *n = 1, hipSuccess; }
hipError_t hipGetLastError() { return launched(); }
const char* hipGetErrorString(hipError_t) { return "stand-in"; }
hipError_t hipGetSymbolAddress(void** p, const void*) { return *p = nullptr, hipErrorInvalidValue; }
hipError_t hipEventCreate(hipEvent_t* e) { return *e = (hipEvent_t)malloc(1), hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { return free(e), hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) { return e ? hipSuccess : hipErrorInvalidHandle; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { return *ms = 0.0f, hipSuccess; }
}

namespace sx {
uint32_t piece_tiles(uint32_t n, uint32_t tile) { return n / tile + 1; }
uint32_t slot_tiles(uint64_t n) { return (uint32_t)(n / 256 + 1); }
uint32_t slot_block() { return 256; }
size_t scan_status_bytes(uint32_t n) { return 16 * ((size_t)n / 1024 + 1); }
size_t scan_ctl_bytes() { return 64; }
bool list_is_small(uint32_t n) { return n <= 4096; }
hipError_t launch_zero(const ZeroList& l, hipStream_t) {
    for (const ZeroPart& x : l.part)
        if (x.bytes) {
            need({x.p});
            if (x.p) memset(x.p, 0, std::min<size_t>(x.bytes, (size_t)1 << 22));
        }
    if (!l.ok()) return hipErrorInvalidValue;
    return launched();
}
hipError_t launch_scan_tags(const uint8_t* tags, uint32_t, uint32_t* mon, void* ctl, void* st, WsCtl*, hipStream_t) {
    return need({tags, mon, ctl, st}), launched();
}
hipError_t launch_scan_counts(const uint32_t* in, uint32_t, uint64_t* o, void* ctl, void* st, hipStream_t) {
    return need({in, o, ctl, st}), launched();
}
hipError_t launch_zero_u64(uint64_t* o, hipStream_t) { return need({o}), launched(); }
hipError_t launch_scan_counts_dev(const uint32_t* in, const uint64_t* n, uint32_t, uint64_t* o, void* ctl, void* st,
                                  hipStream_t) {
    return need({in, n, o, ctl, st}), launched();
}
hipError_t launch_bisect(const SceneView& sv, const Cfg&, uint32_t, int, uint32_t* nslots, uint32_t* codes,
                         const OrderedCodes& oc, unsigned long long*, hipStream_t) {
    return need({sv.tags, sv.pts, sv.mon, nslots, codes, oc.codes, oc.wave_base, oc.rich, oc.ctl}), launched();
}
hipError_t launch_scan_slots(const SceneView& sv, const Cfg&, uint32_t, const uint32_t* nslots, const uint32_t* codes,
                             const OrderedCodes& oc, uint64_t* base, void* ctl, void* st, hipStream_t) {
    return need({sv.tags, nslots, codes, oc.codes, oc.wave_base, oc.rich, base, ctl, st}), launched();
}
hipError_t launch_list(uint32_t, uint32_t, const uint32_t* nslots, const uint32_t* codes, const OrderedCodes& oc,
                       uint64_t* base, Slot* pcs, uint64_t, hipStream_t) {
    return need({nslots, codes, oc.codes, oc.wave_base, base, pcs}), launched();
}
hipError_t launch_slots(const SceneView& sv, const Cfg&, const ItemWs& ws, const Slot* pcs, const uint64_t* n, uint64_t,
                        uint32_t* rc, int, unsigned long long*, hipStream_t) {
    return need({sv.styles, sv.xforms, sv.path_map, ws.units, ws.es_lo, ws.tile_n, ws.ctl, pcs, n, rc}), launched();
}
hipError_t launch_tails(const SceneView&, const Cfg&, const ItemWs& ws, const uint64_t* base, uint64_t, uint32_t* rc,
                        unsigned long long*, hipStream_t) {
    return need({ws.units, ws.tile_n, base, rc}), launched();
}
hipError_t launch_records(const SceneView&, const ItemWs& ws, const Cfg&, const uint64_t* roff, const Slot* pcs,
                          const uint64_t* n, uint64_t slot_cap, void*, uint64_t, uint64_t* dst, hipStream_t) {
    need({ws.units, ws.ctl, roff, pcs, n, dst});
    if (!ws.ctl || !dst) return launched();
    const bool fit = g_result.slots_total <= slot_cap && g_result.ovf_n <= ws.ovf_cap;
    WsCtl w = g_result;
    w.result[0] = 0;
    w.result[1] = fit ? 0 : 1;
    *ws.ctl = w;
    dst[0] = w.result[0];
    dst[1] = w.result[1];
    return launched();
}
hipError_t launch_no_records(uint64_t* dst, hipStream_t) { return need({dst}), launched(); }
hipError_t launch_soup(const SceneView&, const Cfg&, void*, uint64_t, unsigned long long*, hipStream_t) { return launched(); }
hipError_t launch_gather(const GatherDesc* d, uint32_t, uint8_t* tags, float2* pts, StyleD* st, float* xf, uint32_t* pm,
                         hipStream_t) {
    return need({d, tags, pts, st, xf, pm}), launched();
}
hipError_t launch_scene_offsets(const uint64_t* base, const uint64_t* roff, uint64_t, const GatherDesc*, uint32_t,
                                uint32_t, uint64_t* o, hipStream_t) {
    return need({base, roff, o}), launched();
}
hipError_t launch_tag_records(const uint64_t* base, const uint64_t* roff, uint64_t, uint32_t, uint32_t*, uint64_t*,
                              hipStream_t) {
    return need({base, roff}), launched();
}
// (dashing: each tag one chunk, which comes out as it went in)
hipError_t launch_dash(const SceneView& sv, const DashBufs& b, int phase, uint8_t* tags, float2* pts, hipStream_t) {
    need({sv.tags, sv.mon, b.desc, b.pat, b.panels, b.len, b.cum, b.sub_start, b.subix, b.nch, b.chb, b.flag, b.st0, b.st1});
    if (phase == 0 && b.chb) b.chb[sv.n_tags] = sv.n_tags;
    if (phase >= 1) need({b.ch_tag, b.cnt, b.otag, b.opt, b.st2});
    if (phase == 1 && b.otag && b.opt) {
        b.otag[b.n_ch] = sv.n_tags;
        b.opt[b.n_ch] = sv.n_pts;
    }
    if (phase == 2) need({tags, pts});
    return launched();
}
}  // namespace sx

extern "C" {
int ah_zero_ok(void* a, size_t na, void* b, size_t nb) { return sx::ZeroList{{a, na}, {b, nb}}.ok(); }
uint32_t ah_range(uint32_t n, uint32_t asked) { return sx::bisect_range_of(n, asked); }
void ah_fail(long k) { g_calls = 0, g_fail = k; }
long ah_calls() { return g_calls; }
void ah_limit(size_t n) { g_limit = n; }
void ah_new_fail(int k) { g_new_fail = k; }
int ah_new_left() { return g_new_fail; }
int ah_bad() { return g_bad; }
int ah_capture(int on) {
    const int was = g_capture;
    g_capture = on;
    return was;
}
int ah_last() { return (int)launched(); }
uint64_t ah_live() { return g_live.size(); }
uint64_t ah_dev_bytes() { return g_dev_bytes; }
uint64_t ah_pin_most() {
    const uint64_t n = g_pin_most;
    return g_pin_most = 0, n;
}
void ah_result(uint64_t slots, uint64_t items, uint64_t ovf) {
    g_result = {};
    g_result.slots_total = slots;
    g_result.items_total = items;
    g_result.ovf_n = ovf;
}
}
