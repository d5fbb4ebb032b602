#pragma once
// Large device buffers to pageable host memory (internal to the host code).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstring>
#include <thread>

#include "device_scope.h"

namespace sk {

// hipMemcpy into pageable memory runs at 10 to 18 GB/s: one thread copies out of the runtime's staging buffer and takes the page
// faults of memory that was never touched, while the link (56 GB/s into pinned memory) waits.  Here LANES threads, the caller among them,
// each take the next piece: link -> own pinned piece -> destination.  An epoch of sixteen U-Net
// steps that reads its 124 MB of weights at the end: 64.0 -> 53.5 ms, with the up-convolutions put in order on the device instead of here (how fast
// such copies are depends on the machine: the same epoch on the old path took 57 to 64 ms on five of them).
// Owned by a plan (LANES * PIECE = 8 MB of pinned memory, given back with it); used like the rest of the plan by one thread at a time.
struct HostReader {
    static constexpr int LANES = 4;
    static constexpr size_t PIECE = 2u << 20;
    char *pinned[LANES] = {};
    hipStream_t stream[LANES] = {};
    int device = 0;

    // without its buffers it reads with hipMemcpy
    void open()
    {
        bool ok = hipGetDevice(&device) == hipSuccess;
        for (int i = 0; ok && i < LANES; ++i)
            ok = hipHostMalloc(reinterpret_cast<void **>(&pinned[i]), PIECE, hipHostMallocDefault) == hipSuccess &&
                 hipStreamCreateWithFlags(&stream[i], hipStreamNonBlocking) == hipSuccess;
        if (!ok) {
            close();
            (void)hipGetLastError();
        }
    }
    void close()
    {
        for (int i = 0; i < LANES; ++i) {
            if (pinned[i]) (void)hipHostFree(pinned[i]);
            if (stream[i]) (void)hipStreamDestroy(stream[i]);
            pinned[i] = nullptr;
            stream[i] = nullptr;
        }
    }

    // hipMemcpy(dst, src, bytes, hipMemcpyDeviceToHost), also in what it waits for: what was issued to the null stream, a graph's replay
    // among it, which the lanes' own streams do not wait for
    hipError_t read(void *dst, const void *src, size_t bytes) const
    {
        const size_t pieces = (bytes + PIECE - 1) / PIECE;
        if (pieces < 2 || !stream[LANES - 1]) return hipMemcpy(dst, src, bytes, hipMemcpyDeviceToHost);
        const DeviceScope on(device);
        if (on.status != hipSuccess) return on.status;
        const hipError_t waited = hipStreamSynchronize(nullptr);
        if (waited != hipSuccess) return waited;
        std::atomic<size_t> next{0};
        std::atomic<int> error{hipSuccess};
        auto lane = [&](int i) {
            hipError_t e = hipSetDevice(device);
            for (size_t p; e == hipSuccess && (p = next++) < pieces;) {
                const size_t at = p * PIECE, len = std::min(PIECE, bytes - at);
                e = hipMemcpyAsync(pinned[i], static_cast<const char *>(src) + at, len, hipMemcpyDeviceToHost, stream[i]);
                if (e == hipSuccess) e = hipStreamSynchronize(stream[i]);
                if (e == hipSuccess) std::memcpy(static_cast<char *>(dst) + at, pinned[i], len);
            }
            if (e != hipSuccess) error = e;
        };
        std::thread helper[LANES];
        for (int i = 1; i < LANES && (size_t)i < pieces; ++i) {
            try {
                helper[i] = std::thread(lane, i);
            } catch (...) {                         // no thread, or no memory for one (nothing may leave through the C entry points)
                break;                              // the lanes that run take every piece
            }
        }
        lane(0);
        for (auto &h : helper)
            if (h.joinable()) h.join();
        return static_cast<hipError_t>(error.load());
    }

    // what launch(stream) makes at src, from a kernel on the plan's device, whichever device the caller is on
    template <class Launch> hipError_t read_made(void *dst, const void *src, size_t bytes, Launch &&launch) const
    {
        const DeviceScope on(device);
        if (on.status != hipSuccess) return on.status;
        const hipError_t made = launch(static_cast<hipStream_t>(nullptr));      // (the null stream: what read waits for)
        return made == hipSuccess ? read(dst, src, bytes) : made;
    }
};

}  // namespace sk
