// Host build of sw_copy.hip against a stand-in for the HIP runtime, to look at
// what copy_to_host asks of it: which thread copies on which stream, where to,
// and what it allocates.  Usage: copy_host SCENARIO; exit status 0 if it holds.
#include <stdio.h>
#include <stdlib.h>

#include <condition_variable>
#include <map>
#include <set>

#include "sw_copy.hip"

namespace {

std::mutex mu;
thread_local int cur_device = 0;

// One device buffer: `fresh` is what the work enqueued on `stream` by the
// thread `owner` leaves in it; a copy that does not come after that work in
// stream order sees `stale`.
struct Buffer {
    std::vector<char> stale, fresh;
    hipStream_t stream;
    std::thread::id owner;

    Buffer(size_t n, hipStream_t s) : stale(n, 0), fresh(n), stream(s), owner(std::this_thread::get_id()) {
        for (size_t i = 0; i < n; ++i) fresh[i] = (char)(1 + i % 251 + (i >> 20));
        std::lock_guard<std::mutex> hold(mu);
        all.insert(this);
    }
    ~Buffer() {
        std::lock_guard<std::mutex> hold(mu);
        all.erase(this);
    }
    static std::set<Buffer *> all;
};
std::set<Buffer *> Buffer::all;

bool waited = false;  // for the stream, since the last copy

// Pinned memory held and made.
std::map<void *, size_t> pinned;
size_t pinned_bytes = 0, pinned_most = 0, pinned_made = 0;

// Holds every thread's next copy until `gather` threads are in one.
std::condition_variable gathered;
int gather = 0, waiting = 0;
thread_local bool held = false;

// Memory the device reaches by itself, and what copies wrote there.
const char *mapped = nullptr;
size_t mapped_bytes = 0, straight = 0;

bool is_mapped(const void *p) { return mapped && p >= mapped && p < mapped + mapped_bytes; }

bool check(bool ok, const char *what) {
    if (!ok) printf("failed: %s\n", what);
    return ok;
}

}  // namespace

extern "C" {
hipError_t hipGetDevice(int *d) {
    *d = cur_device;
    return hipSuccess;
}
hipError_t hipSetDevice(int d) {
    cur_device = d;
    return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned int) {
    *p = malloc(n);
    std::lock_guard<std::mutex> hold(mu);
    pinned[*p] = n;
    pinned_bytes += n;
    pinned_most = std::max(pinned_most, pinned_bytes);
    ++pinned_made;
    return hipSuccess;
}
hipError_t hipHostFree(void *p) {
    std::lock_guard<std::mutex> hold(mu);
    pinned_bytes -= pinned[p];
    pinned.erase(p);
    free(p);
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
    *e = (hipEvent_t)malloc(1);
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) {
    free(e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) {
    std::lock_guard<std::mutex> hold(mu);
    waited = true;
    return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *at, const void *p) {
    at->type = is_mapped(p) ? hipMemoryTypeHost : hipMemoryTypeUnregistered;
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t n, hipMemcpyKind, hipStream_t s) {
    const Buffer *b = nullptr;
    {
        std::unique_lock<std::mutex> hold(mu);
        if (gather && held) {
            held = false;
            if (++waiting == gather) gathered.notify_all();
            gathered.wait(hold, [] { return waiting >= gather; });
        }
        for (const Buffer *x : Buffer::all)
            if (src >= x->stale.data() && src < x->stale.data() + x->stale.size()) b = x;
    }
    if (!b) return hipErrorInvalidValue;
    const size_t at = (const char *)src - b->stale.data();
    if (is_mapped(dst)) straight += n;
    {
        std::lock_guard<std::mutex> hold(mu);
        waited = false;
    }
    const bool ordered = s == b->stream && (s != hipStreamPerThread || std::this_thread::get_id() == b->owner);
    memcpy(dst, (ordered ? b->fresh.data() : b->stale.data()) + at, n);
    return hipSuccess;
}
}

namespace {

bool copies(size_t n, hipStream_t s) {
    Buffer b(n, s);
    std::vector<char> out(n, 0);
    if (swmi::copy_to_host(out.data(), b.stale.data(), n, s) != hipSuccess) return false;
    return out == b.fresh;
}

// Sizes below and above every limit, each with a remainder.
const size_t kSizes[] = {1, 320, (size_t)64 << 10, ((size_t)64 << 10) + 1, (size_t)1 << 20, ((size_t)3 << 20) + 7,
                         (size_t)8 << 20, ((size_t)33 << 20) + 11};

bool every_size(hipStream_t s) {
    swmi::StageUser user;
    bool ok = true;
    for (size_t n : kSizes) {
        ok = check(copies(n, s), "copy") && ok;
        ok = check(waited, "stream not waited for") && ok;
    }
    return ok;
}

// Into memory that the device reaches by itself: one copy, straight there.
bool into_mapped() {
    swmi::StageUser user;
    bool ok = true;
    for (size_t n : kSizes) {
        Buffer b(n, (hipStream_t)0x1000);
        std::vector<char> out(n, 0);
        mapped = out.data();
        mapped_bytes = n;
        straight = 0;
        ok = check(swmi::copy_to_host(out.data(), b.stale.data(), n, b.stream) == hipSuccess, "copy") && ok;
        ok = check(out == b.fresh, "bytes") && check(straight == n, "not straight") && ok;
        mapped = nullptr;
    }
    return ok;
}

// `threads` threads on each of `devices` devices, all in a copy at once.
bool at_once(int devices, int threads, size_t n) {
    {
        std::lock_guard<std::mutex> hold(mu);
        gather = devices * threads;
        waiting = 0;
    }
    std::atomic<int> good{0};
    std::vector<std::thread> th;
    for (int i = 0; i < devices * threads; ++i)
        th.emplace_back([=, &good] {
            cur_device = i % devices;
            held = true;
            good += copies(n, (hipStream_t)(uintptr_t)(0x1000 + 16 * i));
        });
    for (std::thread &t : th) t.join();
    gather = 0;
    return check(good == devices * threads, "copies at once");
}

// Reading again makes no pinned memory, however many threads and devices read,
// and what is held stays below 32 MiB a device; the last object leaves 4 MiB.
bool steady(int devices, int threads) {
    bool ok = true;
    {
        swmi::StageUser user;
        for (size_t n : {(size_t)320, ((size_t)2 << 20) + 5, ((size_t)9 << 20) + 5}) {
            ok = at_once(devices, threads, n) && ok;
            const size_t made = pinned_made;
            for (int k = 0; k < 3; ++k) ok = at_once(devices, threads, n) && ok;
            ok = check(pinned_made == made, "pinned memory made in the steady state") && ok;
        }
        ok = check(pinned_most <= (size_t)devices * (33u << 20), "pinned memory held") && ok;
    }
    return check(pinned_bytes <= (size_t)4 << 20, "pinned memory left") && ok;
}

}  // namespace

int main(int argc, char **argv) {
    const std::string what = argc > 1 ? argv[1] : "";
    bool ok = false;
    if (what == "stream") ok = every_size((hipStream_t)0x1000);
    if (what == "null_stream") ok = every_size(nullptr);
    if (what == "per_thread_stream") ok = every_size(hipStreamPerThread);
    if (what == "into_mapped") ok = into_mapped();
    if (what == "eight_threads") ok = steady(1, 8);
    if (what == "more_threads") ok = steady(1, 19);
    if (what == "six_devices") ok = steady(6, 2);
    return ok ? 0 : 1;
}
