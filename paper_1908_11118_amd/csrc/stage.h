// stage.h -- small results from the device to the caller's host arrays: one launch and one
// wait through pinned memory instead of a blocking copy per array.
#pragma once
#include <algorithm>
#include <cstring>
#include <initializer_list>
#include <mutex>

#include "host_util.h"
#include "regc_dev.h"

namespace regc {

// A device array and where it goes (null: not asked for).
struct Piece {
    void *dst;
    const void *src;
    size_t bytes;                 // a multiple of 4
};

constexpr size_t kStageBytes = (size_t)256 << 10;

struct Stage {
    int device = 0;               // that the arrays are on
    uint32_t *mem = nullptr;      // pinned, of kStageBytes, allocated at the first use
    std::mutex mutex;
    ~Stage()
    {
        if (mem) (void)hipHostFree(mem);
    }
};

// Waits for the stream and fills the host arrays: in one launch and one wait while they are
// small (64 walkers, ten records: 12 copies 150 us, three launches and waits 25), else a copy
// each.  A copy each also where the launch would not run on the arrays' device (another one
// is current: the null stream is that one's) and where there is no pinned memory to be had.
inline int fetch(Stage &st, hipStream_t stream, std::initializer_list<Piece> pieces)
{
    PackArgs a{};
    size_t total = 0;
    for (const Piece &p : pieces)
        if (p.dst && p.bytes) {
            total += p.bytes;
            a.src[a.n] = static_cast<const uint32_t *>(p.src);
            a.end[a.n++] = (uint32_t)std::min<size_t>(total / 4, UINT32_MAX);
        }
    if (!total) {
        REGC_HIP(hipStreamSynchronize(stream));
        return REGC_OK;
    }
    int current = -1;
    if (total <= kStageBytes && hipGetDevice(&current) == hipSuccess && current == st.device) {
        std::lock_guard<std::mutex> lock(st.mutex);
        if (!st.mem && hipHostMalloc((void **)&st.mem, kStageBytes, hipHostMallocDefault) != hipSuccess) {
            st.mem = nullptr;
            (void)hipGetLastError();
        }
        if (st.mem) {
            REGC_HIP(launch_pack(a, st.mem, stream));
            REGC_HIP(hipStreamSynchronize(stream));
            const char *from = reinterpret_cast<const char *>(st.mem);
            for (const Piece &p : pieces)
                if (p.dst && p.bytes) {
                    std::memcpy(p.dst, from, p.bytes);
                    from += p.bytes;
                }
            return REGC_OK;
        }
    }
    REGC_HIP(hipStreamSynchronize(stream));
    for (const Piece &p : pieces)
        if (p.dst && p.bytes) REGC_HIP(hipMemcpy(p.dst, p.src, p.bytes, hipMemcpyDeviceToHost));
    return REGC_OK;
}

}  // namespace regc
