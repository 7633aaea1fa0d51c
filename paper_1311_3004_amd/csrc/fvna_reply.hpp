// fvna_reply.hpp -- pinned host memory through which kernels answer the host.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <mutex>

namespace fvna {

// Pinned host memory that answers are written to by the kernels that form them.
//
// Small ones (the clock and its window state, sums, a window of at most
// REPLY_CELLS cells): one launch and one wait bring an answer, where a copy to
// the caller's pageable memory took a round trip of 15 to 20 us each.  Clock
// 20 -> 12 us, statistics 39 -> 12, one row of a window 91 -> 21, sums
// 47 -> 20; two steps of 96 x 64, one row and the time 150 -> 47.
//
// Large ones go through two chunks (stream_out), one filled by the copy engine
// while the host copies the other out.
//
// Each part is allocated when it is first needed and given back with its owner;
// where there is no memory to pin, get() and chunk() are null and the answer
// takes the copies.  Whoever asks holds the lock from the launch until the
// answer is copied out: the members of a batch share one.
constexpr size_t REPLY_HEAD = 1024;
constexpr long long REPLY_CELLS = 8192;
constexpr long long REPLY_CHUNK = 131072;   // cells of a chunk: 1 MiB
// Cells from which the chunks are used: pinning them costs about 0.5 ms once,
// what they save of 4 MiB.
constexpr long long REPLY_BIG = 4 * REPLY_CHUNK;

struct Reply {
    std::recursive_mutex mu;
    size_t tail = 0;                        // bytes beyond head and window (the clocks of a batch)
    Reply() = default;
    Reply(const Reply&) = delete;
    Reply& operator=(const Reply&) = delete;
    ~Reply()
    {
        if (p) (void)hipHostFree(p);
        if (big) (void)hipHostFree(big);
        for (hipEvent_t e : ready)
            if (e) (void)hipEventDestroy(e);
    }
    char* get() { return once(p, tried, REPLY_HEAD + 3 * REPLY_CELLS * sizeof(double) + tail); }
    double* cells() { return get() ? (double*)(p + REPLY_HEAD) : nullptr; }
    char* end() { return get() ? p + REPLY_HEAD + 3 * REPLY_CELLS * sizeof(double) : nullptr; }
    // the first of two chunks with their events, null if there are none
    double* chunks()
    {
        for (hipEvent_t& e : ready)
            if (!e && hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) {
                e = nullptr;
                (void)hipGetLastError();
                return nullptr;
            }
        return (double*)once(big, big_tried, 2 * REPLY_CHUNK * sizeof(double));
    }
    hipEvent_t event(int k) const { return ready[k & 1]; }

private:
    char *p = nullptr, *big = nullptr;
    bool tried = false, big_tried = false;
    hipEvent_t ready[2] = {nullptr, nullptr};
    static char* once(char*& m, bool& done, size_t bytes)
    {
        if (!done) {
            done = true;
            if (hipHostMalloc((void**)&m, bytes, hipHostMallocPortable) != hipSuccess) {
                m = nullptr;
                (void)hipGetLastError();
            }
        }
        return m;
    }
};

// n 64-bit words of device memory to the reply.
static __global__ void k_words(const unsigned long long* __restrict__ src, unsigned long long* __restrict__ dst, int n)
{
    for (int k = threadIdx.x; k < n; k += blockDim.x) dst[k] = src[k];
}

// `bytes` (a multiple of 8, at most REPLY_HEAD) of device memory to h, once
// everything enqueued before is done.
inline hipError_t read_words(Reply& r, hipStream_t s, const void* src, void* h, size_t bytes)
{
    std::lock_guard<std::recursive_mutex> lock(r.mu);
    char* pin = r.get();
    if (pin) {
        hipLaunchKernelGGL(k_words, dim3(1), dim3(64), 0, s, (const unsigned long long*)src, (unsigned long long*)pin,
                           (int)(bytes / 8));
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const hipError_t e = hipStreamSynchronize(s);
    if (e != hipSuccess) return e;
    if (!pin) return hipMemcpy(h, src, bytes, hipMemcpyDeviceToHost);
    std::memcpy(h, pin, bytes);
    return hipSuccess;
}

// `fields` arrays of rows x n cells to dst[0 ..], fill(f, row, nrows, out)
// launching the kernel that writes rows row .. row + nrows - 1 of array f to
// out.  stage: device memory for the cells of one array or REPLY_CHUNK of them.
// False (and nothing launched) if there is too little for it, the chunks are
// not to be had or too short for a row; err is the first error of a launch, copy or wait.
template <typename Fill>
bool stream_out(Reply& r, hipStream_t s, int fields, long long rows, long long n, double* stage, double* const* dst,
                Fill&& fill, hipError_t& err)
{
    std::lock_guard<std::recursive_mutex> lock(r.mu);
    err = hipSuccess;
    double* const pin = fields * rows * n >= REPLY_BIG && n <= REPLY_CHUNK ? r.chunks() : nullptr;
    if (!pin) return false;
    const long long per = std::min<long long>(REPLY_CHUNK / n, 65535), parts = (rows + per - 1) / per;
    const long long total = fields * parts;
    auto row0 = [&](long long k) { return (k % parts) * per; };
    auto size = [&](long long k) { return std::min(per, rows - row0(k)) * n; };
    auto launch = [&](long long k) {
        fill((int)(k / parts), row0(k), size(k) / n, stage);
        err = hipGetLastError();
        if (err == hipSuccess)
            err = hipMemcpyAsync(pin + (k & 1) * REPLY_CHUNK, stage, (size_t)size(k) * sizeof(double),
                                 hipMemcpyDeviceToHost, s);
        if (err == hipSuccess) err = hipEventRecord(r.event((int)(k & 1)), s);
    };
    launch(0);
    for (long long k = 0; k < total && err == hipSuccess; ++k) {
        if (k + 1 < total) launch(k + 1);
        if (err == hipSuccess) err = hipEventSynchronize(r.event((int)(k & 1)));
        if (err == hipSuccess)
            std::memcpy(dst[k / parts] + row0(k) * n, pin + (k & 1) * REPLY_CHUNK,
                        (size_t)size(k) * sizeof(double));
    }
    if (err != hipSuccess) (void)hipStreamSynchronize(s);      // nothing writes to the chunks any more
    return true;
}

}  // namespace fvna
