// Device scratch of the calls that synchronise before they return (mesh,
// distinct vertices, distances): taken at the start of a call and given back
// at its end, when the device has finished with it, so a buffer has one user
// at a time whatever the threads and streams.  Buffers given back are kept
// for the next call up to kKeep bytes in all, kKeepAlone while there is no
// volume (distances and vertices need none); they are freed when a volume is
// destroyed, when an allocation of the library fails and on demand.
// Allocating and freeing per call cost 4 of the 9.9 ms of a mesh, its vertices
// and two distance calls (28,700 blocks, 1.0 M points), and 30 of 150 us of the
// vertices of 300,000 triangles.
#include <hip/hip_runtime.h>

#include <mutex>
#include <new>
#include <vector>

#include "internal.hpp"

namespace sc {

namespace {
constexpr size_t kKeep = size_t(1) << 30, kKeepAlone = size_t(128) << 20;
std::mutex g_mu;
int g_volumes = 0;
std::vector<Scratch>& kept()
{
    static std::vector<Scratch> v;
    return v;
}
}  // namespace

Scratch scratch_take(size_t bytes)
{
    Scratch s{};
    if (hipGetDevice(&s.device) != hipSuccess) return s;
    // sizes in steps of at most a quarter, so that calls of nearly the same size share a buffer
    size_t step = 4096;
    while (step * 8 < bytes) step *= 2;
    bytes = (bytes + step - 1) / step * step;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        auto& v = kept();
        size_t best = v.size();
        for (size_t i = 0; i < v.size(); ++i)
            if (v[i].device == s.device && v[i].bytes >= bytes && (best == v.size() || v[i].bytes < v[best].bytes))
                best = i;
        if (best < v.size()) {
            s = v[best];
            v.erase(v.begin() + (long)best);
            return s;
        }
    }
    void* p = nullptr;
    if (!device_alloc_bytes(&p, bytes)) return s;
    s.p = static_cast<unsigned char*>(p);
    s.bytes = bytes;
    return s;
}

void scratch_give(Scratch& s, bool idle)
{
    if (!s.p) return;
    bool keep = idle;
    if (keep) {
        std::lock_guard<std::mutex> lk(g_mu);
        auto& v = kept();
        size_t sum = s.bytes;
        for (const Scratch& k : v) sum += k.bytes;
        keep = sum <= (g_volumes > 0 ? kKeep : kKeepAlone);
        if (keep) try {
            v.push_back(s);
        } catch (const std::bad_alloc&) {
            keep = false;
        }
    }
    if (!keep) (void)hipFree(s.p);
    s = Scratch{};
}

void scratch_trim()
{
    std::vector<Scratch> old;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        old.swap(kept());
    }
    for (Scratch& s : old) (void)hipFree(s.p);
}

void scratch_volumes(int change)
{
    {
        std::lock_guard<std::mutex> lk(g_mu);
        g_volumes += change;
    }
    if (change < 0) scratch_trim();
}

bool device_alloc_bytes(void** p, size_t bytes)
{
    for (int attempt = 0; attempt < 2; ++attempt) {
        const hipError_t e = hipMalloc(p, bytes);
        if (e == hipSuccess) return true;
        (void)hipGetLastError();
        *p = nullptr;
        if (e != hipErrorOutOfMemory) break;
        if (attempt == 0) scratch_trim();
    }
    return false;
}

}  // namespace sc

extern "C" void sc_release_scratch(void) { sc::scratch_trim(); }
