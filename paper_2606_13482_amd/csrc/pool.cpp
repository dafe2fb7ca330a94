// Large device blocks kept between uses.  Memory that the driver has taken back is
// cleared before it is handed out again, at 30 to 40 GB/s on this system: a program
// that makes and drops operators (1.9 GB of pair blocks and 0.5 GB of matrix at 7680
// unknowns) spends 55 to 120 ms each time in hipMalloc or hipFree once the clean
// memory is used up, against 4 ms of kernels.
//
// A block of at least 1 MiB that is given up is kept for the next request of its
// size (up to a quarter less) on its device.  The kept blocks are bounded (4 GiB, or
// 1/64 of the device's memory if that is less; the oldest go first), those unused for two
// seconds are released at the next request or return, and all are released when an
// allocation of the library fails, before it is tried again.
#include <chrono>
#include <mutex>
#include <unordered_map>
#include <vector>

#include "bie_internal.hpp"

namespace bie {

namespace {

typedef std::chrono::steady_clock Clock;
constexpr size_t SMALLEST = size_t(1) << 20, GRAIN = size_t(2) << 20, LARGEST = size_t(4) << 30;
constexpr std::chrono::seconds IDLE(2);

struct Block {
    void *p;
    size_t bytes;
    int device;
    size_t limit;   // of the kept blocks on its device
    Clock::time_point since;
};
struct State {
    std::mutex mu;
    std::unordered_map<void *, Block> used;
    std::vector<Block> kept;   // oldest first
    std::unordered_map<int, size_t> limit;
};
State &state()   // never destroyed: blocks may outlive static objects
{
    static State *s = new State();
    return *s;
}

// the limit of device, which is current: asked when a block is taken, for it may be
// given up while another device is
size_t limit_of(State &st, int device)
{
    const auto it = st.limit.find(device);
    if (it != st.limit.end()) return it->second;
    size_t free = 0, total = 0;
    if (hipMemGetInfo(&free, &total) != hipSuccess) return 0;
    return st.limit[device] = std::min(LARGEST, total / 64);
}

void release(const std::vector<Block> &bs)
{
    for (const Block &b : bs) (void)hipFree(b.p);
}

// takes out of kept what has been idle too long
void take_idle(State &st, std::vector<Block> &out)
{
    const Clock::time_point now = Clock::now();
    std::vector<Block> left;
    for (const Block &b : st.kept) (now - b.since > IDLE ? out : left).push_back(b);
    st.kept.swap(left);
}

}  // namespace

bool pool_release()
{
    int device = 0;
    if (hipGetDevice(&device) != hipSuccess) return false;
    State &st = state();
    std::vector<Block> out, left;
    {
        std::lock_guard<std::mutex> lk(st.mu);
        for (const Block &b : st.kept) (b.device == device ? out : left).push_back(b);
        st.kept.swap(left);
    }
    release(out);
    return !out.empty();
}

hipError_t pool_get(void **p, size_t bytes)
{
    if (bytes < SMALLEST) return device_malloc(p, bytes);
    bytes = (bytes + GRAIN - 1) / GRAIN * GRAIN;
    int device = 0;
    const hipError_t e = hipGetDevice(&device);
    if (e != hipSuccess) return e;
    State &st = state();
    std::vector<Block> idle;
    *p = nullptr;
    {
        std::lock_guard<std::mutex> lk(st.mu);
        size_t best = st.kept.size();
        for (size_t i = 0; i < st.kept.size(); ++i) {
            const Block &b = st.kept[i];
            if (b.device == device && b.bytes >= bytes && b.bytes - bytes <= bytes / 4 &&
                (best == st.kept.size() || b.bytes < st.kept[best].bytes))
                best = i;
        }
        if (best < st.kept.size()) {
            const Block b = st.kept[best];
            st.used[b.p] = b;
            st.kept.erase(st.kept.begin() + int64_t(best));
            *p = b.p;
        }
        take_idle(st, idle);
    }
    release(idle);
    if (*p) return hipSuccess;
    const hipError_t e2 = device_malloc(p, bytes);
    if (e2 != hipSuccess) return e2;
    std::lock_guard<std::mutex> lk(st.mu);
    st.used[*p] = Block{ *p, bytes, device, limit_of(st, device), Clock::now() };
    return hipSuccess;
}

void pool_put(void *p)
{
    if (!p) return;
    State &st = state();
    std::vector<Block> out;
    {
        std::lock_guard<std::mutex> lk(st.mu);
        const auto it = st.used.find(p);
        if (it == st.used.end()) {
            out.push_back(Block{ p, 0, 0, 0, {} });
        } else {
            Block b = it->second;
            st.used.erase(it);
            b.since = Clock::now();
            if (b.bytes > b.limit) {
                out.push_back(b);
            } else {
                st.kept.push_back(b);
                size_t sum = 0;
                for (const Block &k : st.kept) sum += k.device == b.device ? k.bytes : 0;
                for (size_t i = 0; i < st.kept.size() && sum > b.limit;) {
                    if (st.kept[i].device != b.device) {
                        ++i;
                        continue;
                    }
                    sum -= st.kept[i].bytes;
                    out.push_back(st.kept[i]);
                    st.kept.erase(st.kept.begin() + int64_t(i));
                }
            }
        }
        take_idle(st, out);
    }
    release(out);
}

}  // namespace bie
