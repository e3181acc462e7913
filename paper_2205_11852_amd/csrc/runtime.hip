// Error reporting, device contexts, pinned staging and stream-ordered scratch.
#include <cstring>
#include <map>

#include "lc_internal.hpp"

namespace lc {

static thread_local std::string g_err;

void set_error(const char* fmt, ...) {
    char buf[1024];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
}

void clear_error() { g_err.clear(); }

lc_status fail(lc_status code, const char* fmt, ...) {
    char buf[1024];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return code;
}

static std::mutex g_ctx_mu;
static std::map<int, DeviceCtx*> g_ctx;

lc_status get_ctx(DeviceCtx** out) {
    int dev = 0;
    LC_TRY_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(g_ctx_mu);
    auto it = g_ctx.find(dev);
    if (it != g_ctx.end()) {
        *out = it->second;
        return LC_OK;
    }
    auto* c = new DeviceCtx();
    c->device = dev;
    hipDeviceProp_t prop;
    LC_TRY_HIP(hipGetDeviceProperties(&prop, dev));
    c->n_cu = prop.multiProcessorCount;
    c->max_lds_block = prop.sharedMemPerBlock;
    // keep freed stream-ordered memory in the pool between calls
    hipMemPool_t pool;
    if (hipDeviceGetDefaultMemPool(&pool, dev) == hipSuccess) {
        uint64_t thr = UINT64_MAX;
        (void)hipMemPoolSetAttribute(pool, hipMemPoolAttrReleaseThreshold, &thr);
    }
    c->scratch_cap = prop.totalGlobalMem / 16;
    for (PinnedSlot& sl : c->pinned) LC_TRY_HIP(hipEventCreateWithFlags(&sl.ev, hipEventDisableTiming));
    g_ctx[dev] = c;
    *out = c;
    return LC_OK;
}

size_t Stager::push(const void* src, size_t bytes) {
    size_t off = (host_.size() + 255) & ~size_t(255);
    host_.resize(off + bytes);
    if (bytes) std::memcpy(host_.data() + off, src, bytes);
    return off;
}

// The host bytes go through a ring of pinned blocks, so that a call does not
// wait for the copy of the call before it, which the stream makes only after
// the kernels queued before that call (with the scratch cache below,
// back-to-back counts of 5 tasks of 3001 points went from 86 to 79 us a call).
lc_status Stager::commit(hipStream_t s, void** dev_base) {
    const size_t n = host_.size() ? host_.size() : 1;
    std::lock_guard<std::mutex> lk(ctx_->mu);
    PinnedSlot& sl = ctx_->pinned[ctx_->pinned_next];
    ctx_->pinned_next = (ctx_->pinned_next + 1) % kPinnedSlots;
    if (sl.pending) {
        // the last copy out of this block must have finished
        LC_TRY_HIP(hipEventSynchronize(sl.ev));
        sl.pending = false;
    }
    if (sl.size < n) {
        if (sl.p) LC_TRY_HIP(hipHostFree(sl.p));
        sl.p = nullptr;
        sl.size = 0;
        size_t sz = 1 << 14;
        while (sz < n) sz <<= 1;
        if (hipHostMalloc(&sl.p, sz, hipHostMallocDefault) != hipSuccess) {
            sl.p = nullptr;
            return fail(LC_ERR_NOMEM, "pinned staging allocation of %zu bytes failed", sz);
        }
        sl.size = sz;
    }
    if (!host_.empty()) std::memcpy(sl.p, host_.data(), host_.size());
    void* d = nullptr;
    LC_TRY(dev_alloc(&d, n, s));
    hipError_t e = hipSuccess;
    if (!host_.empty()) e = hipMemcpyAsync(d, sl.p, host_.size(), hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipEventRecord(sl.ev, s);
    if (e != hipSuccess) {
        dev_free(d, s);
        return fail(LC_ERR_HIP, "staging copy of %zu bytes failed: %s", host_.size(), hipGetErrorString(e));
    }
    sl.pending = true;
    *dev_base = d;
    return LC_OK;
}

// Scratch cache.  hipFreeAsync takes 20-25 us on the host, more than the
// rest of a small count call, and hipMalloc and hipFree of a mesh (100
// catalogues of 1e5 points) more than building it; a buffer kept here costs
// an event record.  Mesh, counts, xi, map and checked covariance of 32 mocks
// of 5000 points: 1220 -> 947 us; that mesh and one count on it 6.9 -> 1.5 ms.  A buffer is handed
// out for its size class only (at most an eighth larger than asked for), on
// the stream it was freed on or, once its event has passed, on any.  What is
// kept is bounded by a sixteenth of the device's memory (the oldest buffers
// leave first), given up when an allocation fails and released by
// lc_release_caches.  A capturing stream takes its memory from the graph.
static size_t size_class(size_t n) {
    size_t step = 256;
    while (step * 8 < n) step <<= 1;
    return (n + step - 1) / step * step;
}

static bool capturing(hipStream_t s) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &st) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return st != hipStreamCaptureStatusNone;
}

// Gives a cached buffer's memory back to the device (scratch_mu held).
static void scratch_drop(DeviceCtx* c, std::list<ScratchBlock>::iterator it) {
    if (!it->idle) (void)hipEventSynchronize(it->ev);
    if (it->ev) (void)hipEventDestroy(it->ev);
    (void)hipFreeAsync(it->p, nullptr);
    c->scratch_bytes -= it->size;
    c->scratch.erase(it);
}

static void scratch_drop_all(DeviceCtx* c) {
    while (!c->scratch.empty()) scratch_drop(c, c->scratch.begin());
}

lc_status dev_alloc(void** p, size_t bytes, hipStream_t s) {
    const size_t n = size_class(bytes ? bytes : 1);
    *p = nullptr;
    DeviceCtx* c;
    LC_TRY(get_ctx(&c));
    const bool cap = capturing(s);
    std::lock_guard<std::mutex> lk(c->scratch_mu);
    if (!cap) {
        for (auto it = c->scratch.begin(); it != c->scratch.end(); ++it) {
            if (it->size != n) continue;
            if (!it->idle) {
                // (the wait also covers a stream handle that was destroyed
                // and given out again)
                const hipError_t e = it->s == s ? hipStreamWaitEvent(s, it->ev, 0) : hipEventQuery(it->ev);
                if (e != hipSuccess) {
                    (void)hipGetLastError();
                    continue;
                }
            }
            *p = it->p;
            c->scratch_bytes -= n;
            c->scratch_live.emplace(it->p, *it);
            c->scratch.erase(it);
            return LC_OK;
        }
    }
    hipError_t e = hipMallocAsync(p, n, s);
    if (e == hipErrorOutOfMemory && !cap && !c->scratch.empty()) {
        (void)hipGetLastError();
        scratch_drop_all(c);
        (void)hipDeviceSynchronize();
        e = hipMallocAsync(p, n, s);
    }
    if (e != hipSuccess) {
        *p = nullptr;
        (void)hipGetLastError();
        return fail(e == hipErrorOutOfMemory ? LC_ERR_NOMEM : LC_ERR_HIP,
                    "device allocation of %zu bytes failed: %s", bytes, hipGetErrorString(e));
    }
    if (!cap) {
        ScratchBlock b;
        b.p = *p;
        b.size = n;
        c->scratch_live.emplace(b.p, b);
    }
    return LC_OK;
}

static void scratch_put(void* p, hipStream_t s, bool idle) {
    DeviceCtx* c;
    if (!p || get_ctx(&c) != LC_OK) return;
    const bool cap = !idle && capturing(s);
    std::lock_guard<std::mutex> lk(c->scratch_mu);
    auto it = c->scratch_live.find(p);
    if (it == c->scratch_live.end()) {
        (void)hipFreeAsync(p, s);
        return;
    }
    ScratchBlock b = it->second;
    c->scratch_live.erase(it);
    b.s = s;
    b.idle = idle;
    if (!idle && !b.ev && hipEventCreateWithFlags(&b.ev, hipEventDisableTiming) != hipSuccess) b.ev = nullptr;
    if (cap || (!idle && (!b.ev || hipEventRecord(b.ev, s) != hipSuccess))) {
        (void)hipGetLastError();
        if (b.ev) (void)hipEventDestroy(b.ev);
        (void)hipFreeAsync(p, s);
        return;
    }
    c->scratch.push_back(b);
    c->scratch_bytes += b.size;
    while (c->scratch_bytes > c->scratch_cap) scratch_drop(c, c->scratch.begin());
}

void dev_free(void* p, hipStream_t s) { scratch_put(p, s, false); }
void dev_free_idle(void* p) { scratch_put(p, nullptr, true); }

}  // namespace lc

extern "C" const char* lc_last_error(void) { return lc::g_err.c_str(); }

extern "C" void lc_release_caches(void) {
    lc::DeviceCtx* c = nullptr;
    if (lc::get_ctx(&c) != LC_OK) return;
    lc::release_graphs();
    lc::release_tuning();
    {
        std::lock_guard<std::mutex> lk(c->mu);
        for (lc::PinnedSlot& sl : c->pinned) {
            if (sl.pending) (void)hipEventSynchronize(sl.ev);
            sl.pending = false;
            if (sl.p) (void)hipHostFree(sl.p);
            sl.p = nullptr;
            sl.size = 0;
        }
    }
    {
        std::lock_guard<std::mutex> lk(c->scratch_mu);
        lc::scratch_drop_all(c);
    }
    hipMemPool_t pool;
    if (hipDeviceGetDefaultMemPool(&pool, c->device) == hipSuccess) {
        (void)hipDeviceSynchronize();
        (void)hipMemPoolTrimTo(pool, 0);
    }
}
