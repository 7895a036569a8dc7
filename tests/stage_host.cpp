// stage.h on the host alone: the HIP calls it makes are defined here, over host memory.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../paper_1908_11118_amd/csrc/stage.h"

static int current_device, launches, copies, waits;
static bool no_pinned;

extern "C" {
hipError_t hipGetDevice(int *d) { *d = current_device; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipStreamSynchronize(hipStream_t) { ++waits; return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned)
{
    *p = no_pinned ? nullptr : std::malloc(n);
    return no_pinned ? hipErrorOutOfMemory : hipSuccess;
}
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipMalloc(void **, size_t) { return hipErrorOutOfMemory; }
hipError_t hipFree(void *) { return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind)
{
    ++copies;
    std::memcpy(d, s, n);
    return hipSuccess;
}
}

namespace regc {
void set_error(const char *, ...) {}
hipError_t launch_pack(const PackArgs &a, uint32_t *dst, hipStream_t)
{
    ++launches;
    uint32_t k = 0;
    for (int p = 0; p < a.n; ++p)
        for (uint32_t q = 0; k < a.end[p]; ++k, ++q) dst[k] = a.src[p][q];
    return hipSuccess;
}
}  // namespace regc

// words per piece; returns "launches copies" of a fetch into fresh arrays, or "wrong"
static void run(const char *what, int device, int current, bool pinned, size_t words)
{
    std::vector<uint32_t> a(words), b(7), x(words, 0u), y(7, 0u);
    for (size_t k = 0; k < words; ++k) a[k] = (uint32_t)(3 * k + 1);
    for (size_t k = 0; k < 7; ++k) b[k] = (uint32_t)(100 + k);
    regc::Stage st;
    st.device = device;
    current_device = current;
    no_pinned = !pinned;
    launches = copies = waits = 0;
    const int rc = regc::fetch(st, nullptr, {{x.data(), a.data(), 4 * words}, {nullptr, a.data(), 4}, {y.data(), b.data(), 28}});
    std::printf("%s %d %d %d %s\n", what, launches, copies, waits, rc == 0 && x == a && y == b ? "right" : "wrong");
}

int main()
{
    run("same", 0, 0, true, 1000);
    run("other", 0, 1, true, 1000);
    run("unpinned", 0, 0, false, 1000);
    run("large", 0, 0, true, regc::kStageBytes / 4);
    run("second", 1, 1, true, 1000);
    return 0;
}
