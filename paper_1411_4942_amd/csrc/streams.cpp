// Side streams and pinned slots (see streams.hpp).
#include "streams.hpp"

#include <array>
#include <cstdint>
#include <cstring>
#include <map>
#include <mutex>

namespace pm {

hipError_t side_streams(hipStream_t out[2])
{
    static std::mutex mu;
    static std::map<int, std::array<hipStream_t, 2>> made;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lk(mu);
    auto it = made.find(dev);
    if (it == made.end()) {
        std::array<hipStream_t, 2> ss{};
        for (auto &x : ss)
            if ((e = hipStreamCreateWithFlags(&x, hipStreamNonBlocking)) != hipSuccess) return e;
        it = made.emplace(dev, ss).first;
    }
    out[0] = it->second[0];
    out[1] = it->second[1];
    return hipSuccess;
}

namespace {

std::mutex g_slot_mu;
char *g_slot_base = nullptr;
bool g_slot_tried = false;
uint32_t g_slot_used = 0;  // one bit per slot
static_assert(HostSlot::kSlots == 32, "one bit per slot");

}  // namespace

HostSlot::HostSlot() : p(nullptr)
{
    std::lock_guard<std::mutex> lk(g_slot_mu);
    if (!g_slot_tried) {
        g_slot_tried = true;
        void *q = nullptr;
        if (hipHostMalloc(&q, kBytes * kSlots, hipHostMallocPortable) == hipSuccess)
            g_slot_base = (char *)q;
        else
            (void)hipGetLastError();
    }
    if (!g_slot_base || g_slot_used == 0xFFFFFFFFu) return;
    const int i = __builtin_ctz(~g_slot_used);
    g_slot_used |= 1u << i;
    p = g_slot_base + (size_t)i * kBytes;
}

HostSlot::~HostSlot()
{
    if (!p) return;
    std::lock_guard<std::mutex> lk(g_slot_mu);
    g_slot_used &= ~(1u << (int)(((char *)p - g_slot_base) / (ptrdiff_t)kBytes));
}

hipError_t HostSlot::read_back(void *dst, const void *dev, size_t bytes, hipStream_t s)
{
    void *to = p && bytes <= kBytes ? p : dst;
    const hipError_t e = hipMemcpyAsync(to, dev, bytes, hipMemcpyDeviceToHost, s);
    const hipError_t w = hipStreamSynchronize(s);
    if (e == hipSuccess && w == hipSuccess && to != dst) std::memcpy(dst, to, bytes);
    return e != hipSuccess ? e : w;
}

}  // namespace pm
