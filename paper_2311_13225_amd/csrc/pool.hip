// Device memory of the library's handles and temporaries. A freed block is kept for the next request of about its size:
// giving memory back to the driver takes 250 us a block, and the driver clears every block before it hands it out again (some
// 50 GB/s), so that a program which builds graphs or selects hot sets in a loop soon waits for the clearing (measured: the
// 4.7 ms build of a 124 M edge graph at 51 ms a call, 2.5 GB given back by each).
// Bounds: at most POOL_BYTES per device are kept, the longest-unused blocks go first, and only while a handle of the library
// exists; everything kept is given back when an allocation fails and when the last handle is destroyed. A block enters the pool only after its device has
// finished all work (as the driver's own free does), so it may be handed to any thread and any stream.
#include "common.hpp"

#include <map>
#include <mutex>
#include <unordered_map>
#include <vector>

namespace no {

constexpr size_t POOL_BYTES = (size_t)8 << 30;       // per device; 3 % of its memory

namespace {
struct Block { void* p; size_t bytes; int dev; uint64_t age; };
// (never destroyed: handles may be released while the process ends)
std::mutex& g_mutex = *new std::mutex;
auto& g_live = *new std::unordered_map<void*, Block>;         // handed out
auto& g_kept = *new std::multimap<size_t, Block>;             // by size
auto& g_kept_bytes = *new std::unordered_map<int, size_t>;    // by device
uint64_t g_clock = 0;
int64_t g_handles = 0;
thread_local int t_scope = 0;                        // ReleaseScope depth of this thread
thread_local int t_quiet_dev = -1;                   // the device this scope has already waited for

void take_out(std::multimap<size_t, Block>::iterator it) { g_kept_bytes[it->second.dev] -= it->second.bytes; g_kept.erase(it); }

void give_back(std::vector<Block>& blocks) {
    for (Block& b : blocks) (void)hipFree(b.p);
    blocks.clear();
}

void take_all(int dev, std::vector<Block>& out) {    // dev < 0: of every device
    for (auto it = g_kept.begin(); it != g_kept.end();) {
        auto at = it++;
        if (dev >= 0 && at->second.dev != dev) continue;
        out.push_back(at->second);
        take_out(at);
    }
}

// Sizes are rounded up (an eighth of their power of two at most) so that requests of nearly the same size find each other.
size_t rounded(size_t bytes) {
    size_t step = 512;
    if (bytes >= ((size_t)256 << 20)) step = (size_t)2 << 20;
    else while (step * 16 < bytes) step *= 2;
    return (bytes + step - 1) / step * step;
}

void wait_for_device(int dev) {
    if (t_scope > 0 && t_quiet_dev == dev) return;
    int cur = dev;
    (void)hipGetDevice(&cur);
    if (cur != dev) (void)hipSetDevice(dev);
    (void)hipDeviceSynchronize();
    if (cur != dev) (void)hipSetDevice(cur);
    t_quiet_dev = dev;
}
}  // namespace

ReleaseScope::ReleaseScope() { if (t_scope++ == 0) t_quiet_dev = -1; }
ReleaseScope::~ReleaseScope() { --t_scope; }

hipError_t device_alloc(void** out, size_t bytes) {
    *out = nullptr;
    bytes = rounded(bytes);
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    {
        std::lock_guard<std::mutex> l(g_mutex);
        for (auto it = g_kept.lower_bound(bytes); it != g_kept.end() && it->first <= bytes + bytes / 4; ++it)
            if (it->second.dev == dev) {
                const Block b = it->second;
                take_out(it);
                g_live[b.p] = b;
                *out = b.p;
                return hipSuccess;
            }
    }
    void* p = nullptr;
    e = hipMalloc(&p, bytes);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        std::vector<Block> back;
        { std::lock_guard<std::mutex> l(g_mutex); take_all(dev, back); }
        give_back(back);
        e = hipMalloc(&p, bytes);
        if (e != hipSuccess) return e;
    }
    std::lock_guard<std::mutex> l(g_mutex);
    g_live[p] = Block{p, bytes, dev, 0};
    *out = p;
    return hipSuccess;
}

void device_free(void* p) {
    if (!p) return;
    Block b;
    {
        std::lock_guard<std::mutex> l(g_mutex);
        auto it = g_live.find(p);
        if (it == g_live.end()) return;
        b = it->second;
        g_live.erase(it);
    }
    wait_for_device(b.dev);
    std::vector<Block> back;
    {
        std::lock_guard<std::mutex> l(g_mutex);
        if (g_handles == 0) {      // (the temporaries of a call that failed to make the first handle)
            back.push_back(b);
        } else {
            b.age = ++g_clock;
            g_kept.emplace(b.bytes, b);
            g_kept_bytes[b.dev] += b.bytes;
        }
        size_t& kept = g_kept_bytes[b.dev];
        while (kept > POOL_BYTES) {
            auto oldest = g_kept.end();
            for (auto it = g_kept.begin(); it != g_kept.end(); ++it)
                if (it->second.dev == b.dev && (oldest == g_kept.end() || it->second.age < oldest->second.age)) oldest = it;
            back.push_back(oldest->second);
            take_out(oldest);
        }
    }
    give_back(back);
}

void handle_created() {
    std::lock_guard<std::mutex> l(g_mutex);
    ++g_handles;
}

void handle_destroyed() {
    std::vector<Block> back;
    {
        std::lock_guard<std::mutex> l(g_mutex);
        if (--g_handles == 0) take_all(-1, back);
    }
    give_back(back);
}

}  // namespace no
