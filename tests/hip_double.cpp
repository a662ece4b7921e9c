// A stand-in for the HIP runtime, linked with the host half of zs_encode_device.hip on a machine without a GPU: what
// the packer's host code does when a runtime call fails, when the stream is being captured, and when more calls are
// under way than there are slots of pinned memory.  No kernel runs; the launch of scan_kernel leaves a fixed set
// of totals where the kernel would, and the copy of the totals delivers the same ones.
// The scenario is the program's argument; the exit status is 0 when everything in it held.
#include <hip/hip_runtime_api.h>

#include <atomic>
#include <condition_variable>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <set>
#include <string>
#include <thread>
#include <vector>

#include "zipserv.h"

namespace {

struct Totals { // the layout of the packer's
    uint64_t h_units, l_units, n_high;
    uint32_t max_h, max_l, win_lo, predicted_lo;
};
const Totals kTotals = {250, 12, 4000, 250, 12, 117, 0};

std::mutex mutex;
std::map<const void *, std::string> &names() // of the kernels, by their host address (registered before main)
{
    static std::map<const void *, std::string> all;
    return all;
}
thread_local hipError_t last = hipSuccess;
std::atomic<int> copies{0};
std::set<void *> slots_seen; // pinned slots that a launch of scan_kernel was given
std::atomic<bool> malloc_fails{false}, mapping_fails{false}, capturing{false}, sync_fails{false};
std::string launch_fails; // name of the kernel whose launch fails
int wait_for = 0, waiting = 0;  // hipStreamSynchronize returns once that many threads are in it
std::condition_variable all_in;

hipError_t error(hipError_t e) { return last = e; }
} // namespace

extern "C" {
void **__hipRegisterFatBinary(const void *) { static void *p; return &p; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *)
{
    names()[host] = name;
}
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *, dim3 *, size_t *, hipStream_t *) { return hipSuccess; }
hipError_t hipLaunchKernel(const void *f, dim3, dim3, void **args, size_t, hipStream_t)
{
    const std::string &name = names()[f];
    if (!launch_fails.empty() && name.find(launch_fails) != std::string::npos) return error(hipErrorLaunchFailure);
    if (name.find("scan_kernel") != std::string::npos) {
        Totals *host = *static_cast<Totals **>(args[6]);
        if (host && !capturing) *host = kTotals;
        std::lock_guard<std::mutex> lock(mutex);
        if (host) slots_seen.insert(host);
    }
    return hipSuccess;
}
hipError_t hipGetLastError()
{
    const hipError_t e = last;
    last = hipSuccess;
    return e;
}
hipError_t hipHostMalloc(void **p, size_t bytes, unsigned)
{
    if (malloc_fails) return error(hipErrorOutOfMemory);
    *p = std::aligned_alloc(4096, (bytes + 4095) / 4096 * 4096);
    return hipSuccess;
}
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned)
{
    if (mapping_fails) return error(hipErrorInvalidValue);
    *d = h;
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *to, const void *, size_t bytes, hipMemcpyKind, hipStream_t)
{
    ++copies;
    if (!capturing) std::memcpy(to, &kTotals, bytes);
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *status)
{
    *status = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t)
{
    if (capturing) return error(hipErrorStreamCaptureUnsupported);
    if (sync_fails) return error(hipErrorLaunchFailure);
    std::unique_lock<std::mutex> lock(mutex);
    ++waiting;
    all_in.notify_all();
    all_in.wait(lock, [] { return waiting >= wait_for; });
    return hipSuccess;
}
int zs_compute_units(void) { return 256; }
}

namespace {
int call()
{
    alignas(256) static thread_local uint8_t W[64 * 64 * 2], ws[ZS_ENCODE_WORKSPACE_BYTES];
    static thread_local std::vector<uint8_t> room(zs_encode_bound(64, 64) + 256);
    uint8_t *blob = room.data() + (256 - reinterpret_cast<uintptr_t>(room.data()) % 256) % 256;
    zs_desc d;
    std::memset(&d, 0xEE, sizeof d);
    const int rc = zs_encode_device(reinterpret_cast<uint16_t *>(W), 64, 64, 64, blob, zs_encode_bound(64, 64), &d, ws, sizeof ws,
                                    reinterpret_cast<hipStream_t>(0x10));
    if (rc != ZS_OK) return rc;
    const bool same = d.h_bytes == 16 * kTotals.h_units && d.l_bytes == 16 * kTotals.l_units && d.n_high == kTotals.n_high &&
                      d.n_fallback == 4096 - kTotals.n_high && d.max_h_units == kTotals.max_h && d.max_l_units == kTotals.max_l &&
                      d.base_exp == (int)kTotals.win_lo - 1;
    return same ? 0 : 1000;
}
int failures = 0;
void check(bool ok, const char *what, int got)
{
    if (!ok) std::printf("%s: %d\n", what, got), ++failures;
}
void calls(int n, int want_rc, int want_copies, const char *what)
{
    copies = 0;
    for (int i = 0; i < n; ++i) {
        const int rc = call();
        check(rc == want_rc, (std::string(what) + ", status").c_str(), rc);
        const hipError_t left = hipGetLastError();
        if (want_rc == ZS_OK) check(left == hipSuccess, (std::string(what) + ", error left behind").c_str(), left);
    }
    check(copies == want_copies, (std::string(what) + ", copies").c_str(), copies);
}
} // namespace

int main(int argc, char **argv)
{
    const std::string scenario = argc > 1 ? argv[1] : "";
    if (scenario == "plain") {
        calls(40, ZS_OK, 0, "pinned");
        check(slots_seen.size() == 1, "slots used one call after the other", (int)slots_seen.size());
    } else if (scenario == "no_pinned_memory") {
        malloc_fails = true;
        calls(3, ZS_OK, 3, "no pinned memory");
    } else if (scenario == "no_mapping") { // and the slots are there again when it works
        mapping_fails = true;
        calls(20, ZS_OK, 20, "no device address");
        mapping_fails = false;
        calls(3, ZS_OK, 0, "afterwards");
    } else if (scenario == "threads") { // one more than there are slots, all under way at a time
        constexpr int kThreads = 17;
        wait_for = kThreads;
        std::vector<std::thread> threads;
        std::atomic<int> good{0};
        for (int i = 0; i < kThreads; ++i) threads.emplace_back([&] { good += call() == ZS_OK; });
        for (auto &t : threads) t.join();
        check(good == kThreads, "calls at a time that succeed", good);
        check(copies == 1, "copies among them", copies);
        check(slots_seen.size() == kThreads - 1, "slots among them", (int)slots_seen.size());
        calls(3, ZS_OK, 0, "afterwards");
    } else if (scenario == "failed_wait") { // the GPU may still write the slot: nobody else gets it
        sync_fails = true;
        calls(1, ZS_ERR_HIP, 0, "failed wait");
        void *const lost = *slots_seen.begin();
        slots_seen.clear();
        sync_fails = false;
        calls(3, ZS_OK, 0, "afterwards");
        check(!slots_seen.count(lost), "the slot is used again", 1);
    } else if (scenario == "failed_launch") { // is not taken for a failure of what comes after it
        malloc_fails = argc > 2;
        mapping_fails = argc <= 2;
        for (const char *k : {"sample_kernel", "hist_kernel", "recount_kernel", "scan_kernel", "pack_kernel"}) {
            launch_fails = k;
            const int rc = call();
            check(rc == ZS_ERR_HIP, (std::string(k) + " not launched, status").c_str(), rc);
            hipGetLastError();
        }
    } else if (scenario == "capture") { // refused, as every call that waits; no slot is lost by it
        capturing = true;
        copies = 0;
        for (int i = 0; i < 40; ++i) {
            const int rc = call();
            check(rc == ZS_ERR_HIP, "under capture, status", rc);
            hipGetLastError();
        }
        capturing = false;
        calls(3, ZS_OK, 0, "afterwards");
    } else {
        return 2;
    }
    return failures ? 1 : 0;
}
