// Error reporting, device contexts, pinned staging and stream-ordered scratch.
#include <cstring>
#include <iterator>
#include <map>
#include <new>

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
    c->scratch_cap = prop.totalGlobalMem / 16;
    for (PinnedSlot& sl : c->pinned) LC_TRY_HIP(hipEventCreateWithFlags(&sl.ev, hipEventDisableTiming));
    LC_TRY_HIP(hipEventCreateWithFlags(&c->pinned_large.ev, hipEventDisableTiming));
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

// Calls that HIP refuses, breaking the capture, while this thread (or in
// global mode any thread) captures a stream: queries and waits of events,
// synchronous allocation.  They touch no capturing stream here.
class RelaxedCapture {
  public:
    RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode_); }
    ~RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode_); }

  private:
    hipStreamCaptureMode mode_ = hipStreamCaptureModeRelaxed;
};

// The host bytes go through a ring of pinned blocks, so that a call does not
// wait for the copy of the call before it, which the stream makes only after
// the kernels queued before that call (with the scratch cache below,
// back-to-back counts of 5 tasks of 3001 points went from 86 to 79 us a call).
// The ring is one allocation, made once; what is larger than its slots goes
// through a block of its own, which grows with the largest.
static lc_status pinned_room(DeviceCtx* c, PinnedSlot& sl, size_t n) {
    RelaxedCapture relaxed;
    if (sl.pending) {
        // the last copy out of this block must have finished
        LC_TRY_HIP(hipEventSynchronize(sl.ev));
        sl.pending = false;
    }
    if (&sl == &c->pinned_large) {
        if (sl.size >= n) return LC_OK;
        if (sl.p) LC_TRY_HIP(hipHostFree(sl.p));
        sl.p = nullptr;
        sl.size = 0;
        size_t sz = 2 * kPinnedSlot;
        while (sz < n) sz <<= 1;
        if (hipHostMalloc(&sl.p, sz, hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            sl.p = nullptr;
            return fail(LC_ERR_NOMEM, "pinned staging allocation of %zu bytes failed", sz);
        }
        sl.size = sz;
    } else if (!sl.p) {
        void* ring = nullptr;
        if (hipHostMalloc(&ring, kPinnedSlots * kPinnedSlot, hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            return fail(LC_ERR_NOMEM, "pinned staging allocation of %zu bytes failed", kPinnedSlots * kPinnedSlot);
        }
        for (int i = 0; i < kPinnedSlots; i++) {
            c->pinned[i].p = static_cast<unsigned char*>(ring) + i * kPinnedSlot;
            c->pinned[i].size = kPinnedSlot;
        }
    }
    return LC_OK;
}

lc_status Stager::commit(hipStream_t s, void** dev_base) {
    const size_t n = host_.size() ? host_.size() : 1;
    std::lock_guard<std::mutex> lk(ctx_->mu);
    PinnedSlot* slot = &ctx_->pinned_large;
    if (n <= kPinnedSlot) {
        slot = &ctx_->pinned[ctx_->pinned_next];
        ctx_->pinned_next = (ctx_->pinned_next + 1) % kPinnedSlots;
    }
    PinnedSlot& sl = *slot;
    LC_TRY(pinned_room(ctx_, sl, n));
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
// of 5000 points: 1220 -> 947 us; that mesh and one count on it 6.9 -> 1.5 ms.
// A buffer is handed out for its size class only (at most an eighth larger than
// asked for), on the stream it was freed on or, once its event has passed, on
// any.  What is kept is bounded by a sixteenth of the device's memory: beyond
// it the oldest buffers whose work is done go back to the device, at every call
// until it is met (no call waits for them).  An allocation that fails takes
// what is kept, as does lc_release_caches.  A capturing stream takes its memory
// from the graph.
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

// Waits until every stream of the device is idle: what hipFree does first.
// (hipDeviceSynchronize would break the captures of all threads.)
static bool device_wait() {
    RelaxedCapture relaxed;
    void* d = nullptr;
    hipError_t e = hipMalloc(&d, 256);
    if (e == hipSuccess) e = hipFree(d);
    else if (e == hipErrorOutOfMemory) e = hipDeviceSynchronize();
    if (e != hipSuccess) (void)hipGetLastError();
    return e == hipSuccess;
}

static bool passed(const ScratchBlock& b) {
    if (b.idle) return true;
    RelaxedCapture relaxed;
    if (hipEventQuery(b.ev) == hipSuccess) return true;
    (void)hipGetLastError();
    return false;
}

// Whether stream s may use the block (the wait also covers a stream handle that
// was destroyed and given out again).
static bool ready(const ScratchBlock& b, hipStream_t s) {
    if (b.idle || b.s != s) return passed(b);
    if (hipStreamWaitEvent(s, b.ev, 0) == hipSuccess) return true;
    (void)hipGetLastError();
    return false;
}

// Takes the oldest blocks beyond the bound that are done out of the cache
// (scratch_mu held).
static void over_cap(DeviceCtx* c, ScratchList& gone) {
    for (auto it = c->scratch.begin(); it != c->scratch.end() && c->scratch_bytes > c->scratch_cap;) {
        const auto next = std::next(it);
        if (passed(*it)) {
            c->scratch_bytes -= it->size;
            gone.splice(gone.end(), c->scratch, it);
        }
        it = next;
    }
}

// Returns blocks that are done to the device: at once, and without waiting for
// anything (hipFreeAsync leaves them in the pool until some later
// synchronisation).
static void give_back(DeviceCtx* c, ScratchList& gone) {
    if (gone.empty()) return;
    RelaxedCapture relaxed;
    for (ScratchBlock& b : gone) {
        if (b.ev) (void)hipEventDestroy(b.ev);
        (void)hipFree(b.p);
    }
    gone.clear();
    hipMemPool_t pool;
    if (hipDeviceGetDefaultMemPool(&pool, c->device) == hipSuccess) (void)hipMemPoolTrimTo(pool, 0);
}

// Everything cached, back to the device (where HIP refuses the wait, what is
// not done stays).
static void drop_scratch(DeviceCtx* c) {
    ScratchList gone;
    {
        std::lock_guard<std::mutex> lk(c->scratch_mu);
        gone.splice(gone.end(), c->scratch);
        c->scratch_bytes = 0;
    }
    if (!device_wait()) {
        std::lock_guard<std::mutex> lk(c->scratch_mu);
        for (auto it = gone.begin(); it != gone.end();) {
            const auto next = std::next(it);
            if (!passed(*it)) {
                c->scratch_bytes += it->size;
                c->scratch.splice(c->scratch.end(), gone, it);
            }
            it = next;
        }
    }
    give_back(c, gone);
}

static lc_status alloc_failed(size_t bytes, hipError_t e) {
    (void)hipGetLastError();
    return fail(e == hipErrorOutOfMemory ? LC_ERR_NOMEM : LC_ERR_HIP, "device allocation of %zu bytes failed: %s",
                bytes, hipGetErrorString(e));
}

lc_status dev_alloc(void** p, size_t bytes, hipStream_t s) {
    const size_t n = size_class(bytes ? bytes : 1);
    *p = nullptr;
    DeviceCtx* c;
    LC_TRY(get_ctx(&c));
    const bool cap = capturing(s);
    if (cap) {
        const hipError_t e = hipMallocAsync(p, n, s);
        if (e == hipSuccess) return LC_OK;
        *p = nullptr;
        return alloc_failed(bytes, e);
    }
    try {
        ScratchList node, gone;
        {
            std::lock_guard<std::mutex> lk(c->scratch_mu);
            for (auto it = c->scratch.begin(); it != c->scratch.end(); ++it) {
                if (it->size != n || !ready(*it, s)) continue;
                c->scratch_live.emplace(it->p, it);
                c->scratch_bytes -= n;
                c->scratch_out.splice(c->scratch_out.end(), c->scratch, it);
                *p = it->p;
                break;
            }
            over_cap(c, gone);
        }
        give_back(c, gone);
        if (*p) return LC_OK;
        node.emplace_back();
        node.front().size = n;
        void* d = nullptr;
        hipError_t e = hipMallocAsync(&d, n, s);
        if (e == hipErrorOutOfMemory) {
            (void)hipGetLastError();
            drop_scratch(c);
            e = hipMallocAsync(&d, n, s);
        }
        if (e != hipSuccess) return alloc_failed(bytes, e);
        node.front().p = d;
        std::lock_guard<std::mutex> lk(c->scratch_mu);
        try {
            c->scratch_live.emplace(d, node.begin());
        } catch (...) {
            (void)hipFreeAsync(d, s);
            throw;
        }
        c->scratch_out.splice(c->scratch_out.end(), node);
        *p = d;
        return LC_OK;
    } catch (const std::bad_alloc&) {
        return fail(LC_ERR_NOMEM, "out of host memory in a device allocation of %zu bytes", bytes);
    }
}

void dev_free(void* p, hipStream_t s) {
    DeviceCtx* c;
    if (!p || get_ctx(&c) != LC_OK) return;
    const bool cap = capturing(s);
    ScratchList gone;
    {
        std::lock_guard<std::mutex> lk(c->scratch_mu);
        auto it = c->scratch_live.find(p);
        if (it == c->scratch_live.end()) {
            (void)hipFreeAsync(p, s);
            return;
        }
        auto b = it->second;
        c->scratch_live.erase(it);
        b->s = s;
        b->idle = false;
        if (!b->ev && hipEventCreateWithFlags(&b->ev, hipEventDisableTiming) != hipSuccess) b->ev = nullptr;
        if (cap || !b->ev || hipEventRecord(b->ev, s) != hipSuccess) {
            (void)hipGetLastError();
            if (b->ev) (void)hipEventDestroy(b->ev);
            c->scratch_out.erase(b);
            (void)hipFreeAsync(p, s);
            return;
        }
        c->scratch.splice(c->scratch.end(), c->scratch_out, b);
        c->scratch_bytes += b->size;
        over_cap(c, gone);
    }
    give_back(c, gone);
}

void dev_free_unused(void* const* ps, int n) {
    DeviceCtx* c;
    if (get_ctx(&c) != LC_OK) return;
    ScratchList gone;
    {
        std::lock_guard<std::mutex> lk(c->scratch_mu);
        for (int i = 0; i < n; i++) {
            auto it = ps[i] ? c->scratch_live.find(ps[i]) : c->scratch_live.end();
            if (it == c->scratch_live.end()) continue;
            c->scratch_wait.splice(c->scratch_wait.end(), c->scratch_out, it->second);
            c->scratch_live.erase(it);
        }
        gone.splice(gone.end(), c->scratch_wait);
    }
    // any stream may have used them: they count as free after a wait for the
    // whole device, this one or, where HIP refuses it, a later one
    const bool idle = device_wait();
    {
        std::lock_guard<std::mutex> lk(c->scratch_mu);
        if (!idle) {
            c->scratch_wait.splice(c->scratch_wait.end(), gone);
            return;
        }
        for (ScratchBlock& b : gone) {
            b.idle = true;
            c->scratch_bytes += b.size;
        }
        c->scratch.splice(c->scratch.end(), gone);
        over_cap(c, gone);
    }
    give_back(c, gone);
}

}  // namespace lc

extern "C" const char* lc_last_error(void) { return lc::g_err.c_str(); }

extern "C" void lc_release_caches(void) {
    lc::DeviceCtx* c = nullptr;
    if (lc::get_ctx(&c) != LC_OK) return;
    lc::release_graphs();
    lc::release_tuning();
    {
        std::lock_guard<std::mutex> lk(c->mu);
        lc::RelaxedCapture relaxed;
        auto done = [](lc::PinnedSlot& sl) {
            if (sl.pending) (void)hipEventSynchronize(sl.ev);
            sl.pending = false;
        };
        for (lc::PinnedSlot& sl : c->pinned) done(sl);
        done(c->pinned_large);
        if (c->pinned[0].p) (void)hipHostFree(c->pinned[0].p);  // (the whole ring)
        if (c->pinned_large.p) (void)hipHostFree(c->pinned_large.p);
        for (lc::PinnedSlot& sl : c->pinned) sl.p = nullptr;
        c->pinned_large.p = nullptr;
        c->pinned_large.size = 0;
    }
    lc::dev_free_unused(nullptr, 0);
    lc::drop_scratch(c);
    hipMemPool_t pool;
    if (hipDeviceGetDefaultMemPool(&pool, c->device) == hipSuccess) (void)hipMemPoolTrimTo(pool, 0);
}
