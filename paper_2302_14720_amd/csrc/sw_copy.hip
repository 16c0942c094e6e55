// sw_copy.hip -- results to the caller's memory, pageable memory through pinned
// staging buffers.
//
// A pageable hipMemcpy waits for its own staging: 24 us for a record, 36 us for
// 64 KB, 112 us for 256 KB, and 10-17 GB/s for whole configurations, whose
// pages in the caller's memory one thread touches for the first time.  Here
// the device writes pinned slots in stream order (no wait in between) and the
// host moves them on; from kCopySplit bytes on kCopySlots threads of this
// call take a slot each.  Measured, pageable / here: a record 24 / 14 us, 256 KB
// 112 / 21 us, 4 MiB 242 / 204 us, 16 MiB 0.95 / 0.62 ms, 256 MiB 25.4 / 9.5 ms.
#include <string.h>

#include <algorithm>
#include <atomic>
#include <mutex>
#include <thread>

#include "sw_host.h"

namespace swmi {
namespace {

// A stage that has copied no more than this at once is that small: a program that
// reads records and small lattices holds 64 KB, not 4 MiB.
constexpr size_t kCopySmall = (size_t)64 << 10;
constexpr size_t kCopyChunk = (size_t)1 << 20;  // bytes of a slot
// With 2 / 4 / 8 slots (and as many threads): 9.8 MiB 423 / 411 / 445 us, 16 MiB
// 664 / 622 / 653 us, 64 MiB 4.5 / 2.6 / 2.4 ms, 256 MiB 17.8 / 9.9 / 8.9 ms.
constexpr int kCopySlots = 4;
// Below, starting threads costs more than they save; one thread / four: 1.9 MiB
// 97 / 123 us, 4 MiB 214 / 228, 7.6 MiB 347 / 345, 9.8 MiB 440 / 411, 16 MiB
// 683 / 622.
constexpr size_t kCopySplit = (size_t)8 << 20;

struct Stage {
    int device;
    char *pin;
    size_t cap;
    hipEvent_t ev[kCopySlots];
    bool events;
};

// Every device has up to kPerDevice stages of its own; a copy owns one while it
// runs and parks it afterwards, so that eight threads can read at once without
// an allocation in the steady state (making and freeing pinned memory takes
// hundreds of us).  With all of a device's stages taken a copy is a pageable
// one.  When the last sim, batch, server or phi^4 sim of the process is
// destroyed all are given back but for one (at most 4 MiB): freeing
// pinned memory makes the next create 270 us slower (205 -> 475 us at 512^2)
// and its first read 170 us (30 -> 200), which a program that makes one sim
// after another would pay each time.
constexpr int kPerDevice = 8;
constexpr int kMaxDevices = 64;
struct DeviceStages {
    Stage parked[kPerDevice];
    int nparked, live;  // live: parked or owned by a copy
};
std::mutex g_lock;
DeviceStages g_dev[kMaxDevices];
int64_t g_users = 0;

void stage_free(Stage &st) {
    if (st.pin) (void)hipHostFree(st.pin);
    if (st.events)
        for (hipEvent_t e : st.ev) (void)hipEventDestroy(e);
    st = Stage{};
}

// false: none free.
bool stage_take(int device, Stage &st) {
    if (device < 0 || device >= kMaxDevices) return false;
    std::lock_guard<std::mutex> hold(g_lock);
    DeviceStages &d = g_dev[device];
    if (d.nparked > 0) {
        st = d.parked[--d.nparked];
        return true;
    }
    if (d.live == kPerDevice) return false;
    ++d.live;
    st = Stage{};
    st.device = device;
    return true;
}

void stage_give(const Stage &st) {
    std::lock_guard<std::mutex> hold(g_lock);
    DeviceStages &d = g_dev[st.device];
    d.parked[d.nparked++] = st;
}

// Pinned memory for a copy of n bytes; false: none to be had.
bool stage_reserve(Stage &st, size_t n) {
    const size_t want = n <= kCopySmall ? kCopySmall : kCopyChunk * kCopySlots;
    if (st.cap >= want) return true;
    void *p = nullptr;
    if (hipHostMalloc(&p, want, hipHostMallocDefault) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    if (want > kCopySmall && !st.events) {
        for (int i = 0; i < kCopySlots; ++i) {
            if (hipEventCreateWithFlags(&st.ev[i], hipEventDisableTiming) == hipSuccess) continue;
            (void)hipGetLastError();
            for (int j = 0; j < i; ++j) (void)hipEventDestroy(st.ev[j]);
            (void)hipHostFree(p);
            return false;
        }
        st.events = true;
    }
    if (st.pin) (void)hipHostFree(st.pin);
    st.pin = (char *)p;
    st.cap = want;
    return true;
}

// Chunks first, first + step, ... of the copy through slots `slot` .. `slot` +
// nslots - 1, as many in flight as there are slots.
hipError_t copy_chunks(const Stage &st, char *dst, const char *src, size_t n, size_t first, size_t step, int slot,
                       int nslots, hipStream_t s) {
    const size_t chunks = (n + kCopyChunk - 1) / kCopyChunk;
    auto bytes = [&](size_t c) { return std::min(kCopyChunk, n - c * kCopyChunk); };
    auto issue = [&](size_t c, int k) {
        hipError_t e = hipMemcpyAsync(st.pin + (size_t)k * kCopyChunk, src + c * kCopyChunk, bytes(c),
                                      hipMemcpyDeviceToHost, s);
        return e != hipSuccess ? e : hipEventRecord(st.ev[k], s);
    };
    size_t ahead = first;
    for (int k = 0; k < nslots && ahead < chunks; ++k, ahead += step) {
        const hipError_t e = issue(ahead, slot + k);
        if (e != hipSuccess) return e;
    }
    int k = 0;
    for (size_t c = first; c < chunks; c += step) {
        hipError_t e = hipEventSynchronize(st.ev[slot + k]);
        if (e != hipSuccess) return e;
        memcpy(dst + c * kCopyChunk, st.pin + (size_t)(slot + k) * kCopyChunk, bytes(c));
        if (ahead < chunks) {
            e = issue(ahead, slot + k);
            if (e != hipSuccess) return e;
            ahead += step;
        }
        k = k + 1 == nslots ? 0 : k + 1;
    }
    return hipSuccess;
}

hipError_t copy_straight(void *dst, const void *src, size_t n, hipStream_t s) {
    const hipError_t e = hipMemcpyAsync(dst, src, n, hipMemcpyDeviceToHost, s);
    return e != hipSuccess ? e : hipStreamSynchronize(s);
}

// Memory the device reaches by itself (pinned, managed or its own) needs no
// staging: 1 MiB into pinned memory takes 27 us straight and 60 through a slot,
// 268 MB 4.7 and 8.4 ms.  The question costs 0.2 us.
bool device_writes(const void *dst) {
    hipPointerAttribute_t at{};
    if (hipPointerGetAttributes(&at, dst) == hipSuccess) return at.type != hipMemoryTypeUnregistered;
    (void)hipGetLastError();
    return false;
}

hipError_t copy_staged(Stage &st, void *dst, const void *src, size_t n, hipStream_t s) {
    if (!stage_reserve(st, n)) return copy_straight(dst, src, n, s);
    if (n <= st.cap && n <= kCopyChunk) {
        hipError_t e = hipMemcpyAsync(st.pin, src, n, hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e == hipSuccess) memcpy(dst, st.pin, n);
        return e;
    }
    hipError_t e = hipSuccess;
    // hipStreamPerThread names another stream in every thread: only in this one
    // does a copy come after the caller's work
    if (n < kCopySplit || s == hipStreamPerThread) {
        e = copy_chunks(st, (char *)dst, (const char *)src, n, 0, 1, 0, kCopySlots, s);
    } else {
        std::atomic<int> err{(int)hipSuccess};
        auto work = [&](int k) {
            hipError_t w = hipSetDevice(st.device);
            if (w == hipSuccess) w = copy_chunks(st, (char *)dst, (const char *)src, n, (size_t)k, kCopySlots, k, 1, s);
            if (w != hipSuccess) err.store((int)w);
        };
        std::thread th[kCopySlots];
        int started = 1;
        try {
            for (; started < kCopySlots; ++started) th[started] = std::thread(work, started);
        } catch (...) {  // no more threads: this one takes the remaining slots' chunks too
        }
        work(0);
        for (int k = started; k < kCopySlots; ++k) work(k);
        for (int k = 1; k < started; ++k) th[k].join();
        e = (hipError_t)err.load();
    }
    // After an error slots may still be in flight; after a copy that waited for
    // its events alone the runtime's own tidying of the stream (25 us) would fall
    // on the caller's next call.
    const hipError_t w = hipStreamSynchronize(s);
    return e != hipSuccess ? e : w;
}

}  // namespace

hipError_t copy_to_host(void *dst, const void *src, size_t n, hipStream_t s) {
    int device = 0;
    hipError_t e = hipGetDevice(&device);
    if (e != hipSuccess) return e;
    Stage st;
    if (device_writes(dst) || !stage_take(device, st)) return copy_straight(dst, src, n, s);
    e = copy_staged(st, dst, src, n, s);
    stage_give(st);
    return e;
}

StageUser::StageUser() {
    std::lock_guard<std::mutex> hold(g_lock);
    ++g_users;
}

StageUser::~StageUser() {
    std::lock_guard<std::mutex> hold(g_lock);
    if (--g_users > 0) return;
    bool kept = false;
    for (DeviceStages &d : g_dev) {
        while (d.nparked > (kept ? 0 : 1)) {
            stage_free(d.parked[--d.nparked]);
            --d.live;
        }
        kept = kept || d.nparked > 0;
    }
}

}  // namespace swmi
