// workspace.h -- the library's workspace memory: a stream-ordered pool per
// device and the block kept for calls on the null stream (host side only; one
// translation unit includes it).
#pragma once

#include <hip/hip_runtime_api.h>

#include <atomic>
#include <cstdint>
#include <cstdio>
#include <mutex>

#include "../../include/mxattn.h"

namespace mxattn {
namespace {

// Detail of the calling thread's last HIP error (mxattn_last_error).
thread_local char g_last_error[256] = "";

void set_error(const char* what, hipError_t e) {
    std::snprintf(g_last_error, sizeof g_last_error, "%s: %s", what, hipGetErrorString(e));
}

constexpr int kMaxDevices = 64;

// Workspace memory comes from a stream-ordered pool that belongs to the
// library, one per device, created on first use.  Its release threshold has
// no limit, so the forward's workspace is recycled between calls instead of
// being returned to the driver at every synchronization; the device's
// default pool, which other libraries share, keeps its attributes.
// mxattn_release_workspace() hands the cached memory back.  If the pool
// cannot be created, workspace comes from the default pool (unchanged).
struct PoolSlot {
    std::once_flag once;
    std::atomic<hipMemPool_t> pool{nullptr};
};
PoolSlot g_pools[kMaxDevices];

hipMemPool_t private_pool(int dev) {
    if (dev < 0 || dev >= kMaxDevices) return nullptr;
    PoolSlot& slot = g_pools[dev];
    std::call_once(slot.once, [dev, &slot] {
        hipMemPoolProps props{};
        props.allocType = hipMemAllocationTypePinned;
        props.handleTypes = hipMemHandleTypeNone;
        props.location.type = hipMemLocationTypeDevice;
        props.location.id = dev;
        hipMemPool_t pool = nullptr;
        if (hipMemPoolCreate(&pool, &props) != hipSuccess || !pool) {
            (void)hipGetLastError();
            return;
        }
        uint64_t threshold = UINT64_MAX;
        if (hipMemPoolSetAttribute(pool, hipMemPoolAttrReleaseThreshold, &threshold) != hipSuccess) {
            (void)hipGetLastError();
            (void)hipMemPoolDestroy(pool);
            return;
        }
        slot.pool.store(pool);
    });
    return slot.pool.load();
}

hipError_t workspace_alloc(void** p, size_t bytes, hipStream_t s) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return hipErrorInvalidDevice;
    if (hipMemPool_t pool = private_pool(dev)) return hipMallocFromPoolAsync(p, bytes, pool, s);
    return hipMallocAsync(p, bytes, s);
}

// A stream-ordered allocation and its free cost the host about 15 us, several
// times the launches of a short call.  So each device keeps one block for the
// calls on its null stream, which is never destroyed and runs them in the order
// they were enqueued: the next call may overwrite the block without waiting.
// `m` is held while a call is enqueued, so that two threads' launches cannot
// interleave on one block; a call that finds it held, one on another stream
// (whose handle may be destroyed and given out again while its work still
// runs, or which may be captured) and one that needs more than kKeptMost take
// their workspace from the pool as they go.  Host time of a call of 2 heads x
// 512 tokens through the C ABI: 22.3 us with the pool, 5.8 us with the block.
constexpr size_t kKeptMost = (size_t)64 << 20;
struct KeptBlock {
    std::mutex m;
    void* p = nullptr;
    size_t bytes = 0;
};
KeptBlock g_kept[kMaxDevices];

// The workspace of one call, given back when the call has been enqueued.
class Workspace {
  public:
    // The status of taking `bytes` for a call on `s`.
    int take(size_t bytes, hipStream_t s) {
        stream_ = s;
        int dev = -1;
        if (s == nullptr && bytes <= kKeptMost && hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < kMaxDevices) {
            KeptBlock& k = g_kept[dev];
            std::unique_lock<std::mutex> lock(k.m, std::try_to_lock);
            if (lock.owns_lock()) {
                if (k.bytes < bytes) grow(k, bytes);
                if (k.bytes >= bytes) {
                    lock_ = std::move(lock);
                    p_ = k.p;
                    return MXATTN_OK;
                }
            }
        }
        hipError_t e = workspace_alloc(&p_, bytes, s);
        if (e != hipSuccess || !p_) {
            p_ = nullptr;
            set_error("workspace allocation", e);
            return MXATTN_ERR_OOM;
        }
        return MXATTN_OK;
    }
    uint8_t* get() const { return static_cast<uint8_t*>(p_); }
    // Gives the workspace back; the call's status, or that of the free.
    int give_back(int st) {
        if (lock_.owns_lock()) {
            lock_.unlock();
            return st;
        }
        hipError_t e = hipFreeAsync(p_, stream_);
        if (st == MXATTN_OK && e != hipSuccess) {
            set_error("hipFreeAsync", e);
            st = MXATTN_ERR_HIP;
        }
        return st;
    }

  private:
    // A block of at least `bytes` (the next power of two from 1 MiB on) in place
    // of k's; k is empty if it cannot be had, and as it was if its own block
    // cannot be freed.  Either way the call's workspace comes from the pool, and
    // no error is left for the launches that follow.
    static void grow(KeptBlock& k, size_t bytes) {
        if (k.p && hipFreeAsync(k.p, nullptr) != hipSuccess) {
            (void)hipGetLastError();
            return;
        }
        k.p = nullptr;
        k.bytes = 0;
        size_t n = (size_t)1 << 20;
        while (n < bytes) n *= 2;
        void* p = nullptr;
        if (workspace_alloc(&p, n, nullptr) != hipSuccess || !p) {
            (void)hipGetLastError();
            return;
        }
        k.p = p;
        k.bytes = n;
    }
    void* p_ = nullptr;
    hipStream_t stream_ = nullptr;
    std::unique_lock<std::mutex> lock_;
};

// Gives k's block back to the pool if no call can still use it, without waiting
// for one; MXATTN_ERR_HIP if that fails.  The block stays where the null stream
// has work, and where a stream that synchronizes with the null stream is being
// captured (an operation on the null stream is not allowed then: the free and
// the wait below ended the process).  The query of the capture is allowed
// always and disturbs none.
int release_kept(KeptBlock& k) {
    if (!k.p) return MXATTN_OK;
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(nullptr, &capture) != hipSuccess) {
        (void)hipGetLastError();
        return MXATTN_OK;
    }
    // (queries and waits are allowed then also while another stream is captured)
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    const char* what = "hipStreamQuery";
    hipError_t e = hipStreamQuery(nullptr);
    if (e == hipSuccess) {
        what = "hipFreeAsync";
        e = hipFreeAsync(k.p, nullptr);
        if (e == hipSuccess) {
            k.p = nullptr;
            k.bytes = 0;
            // the free is through before the trim; the stream holds nothing else
            what = "hipStreamSynchronize";
            e = hipStreamSynchronize(nullptr);
        }
    }
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    if (e == hipSuccess) return MXATTN_OK;
    (void)hipGetLastError();
    if (e == hipErrorNotReady) return MXATTN_OK;
    set_error(what, e);
    return MXATTN_ERR_HIP;
}

int release_workspace() {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) {
        set_error("hipGetDevice", e);
        return MXATTN_ERR_HIP;
    }
    if (dev < 0 || dev >= kMaxDevices) return MXATTN_OK;
    int st = MXATTN_OK;
    {
        std::lock_guard<std::mutex> lock(g_kept[dev].m);
        st = release_kept(g_kept[dev]);
    }
    hipMemPool_t pool = g_pools[dev].pool.load();
    if (!pool) return st;  // no workspace was ever taken on this device
    e = hipMemPoolTrimTo(pool, 0);
    if (e != hipSuccess) {
        set_error("hipMemPoolTrimTo", e);
        return MXATTN_ERR_HIP;
    }
    return st;
}

}  // namespace
}  // namespace mxattn
