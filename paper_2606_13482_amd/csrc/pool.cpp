// Large device blocks kept between uses.  Memory that the driver has taken back is
// cleared before it is handed out again, at 30 to 40 GB/s on this system: a program
// that makes and drops operators (1.9 GB of pair blocks and 0.5 GB of matrix at 7680
// unknowns) spends 55 to 120 ms each time in hipMalloc or hipFree once the clean
// memory is used up, against 4 ms of kernels.
//
// A block of at least 1 MiB that is given up is kept for the next request of its
// size (up to a quarter less) on its device.  The kept blocks are bounded (4 GiB, or
// 1/64 of the device's memory if that is less; the oldest go first, but not where they
// hold more than the newcomer, which is then not kept), those unused for two
// seconds are released at the next request or return, and all are released when an
// allocation of the library fails, before it is tried again, or when the caller asks
// for it (bie_release_memory).
#include <chrono>
#include <list>
#include <mutex>
#include <unordered_map>

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
typedef std::list<Block> Blocks;
// A block stays in the list node that was made for it: giving one up moves nodes and
// takes no host memory.
struct State {
    std::mutex mu;
    Blocks used, kept;   // kept: oldest first
    std::unordered_map<void *, Blocks::iterator> at;   // the used ones
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

void release(const Blocks &bs)
{
    for (const Block &b : bs) (void)hipFree(b.p);
}

// moves the kept blocks that f names to out
template <typename F>
void take(State &st, Blocks &out, F f)
{
    for (auto it = st.kept.begin(); it != st.kept.end();) {
        const auto b = it++;
        if (f(*b)) out.splice(out.end(), st.kept, b);
    }
}

void take_idle(State &st, Blocks &out)
{
    const Clock::time_point now = Clock::now();
    take(st, out, [&](const Block &b) { return now - b.since > IDLE; });
}

}  // namespace

bool pool_release()
{
    int device = 0;
    if (hipGetDevice(&device) != hipSuccess) return false;
    State &st = state();
    Blocks out;
    {
        std::lock_guard<std::mutex> lk(st.mu);
        take(st, out, [&](const Block &b) { return b.device == device; });
    }
    release(out);
    return !out.empty();
}

size_t pool_release_all()
{
    State &st = state();
    Blocks out;
    {
        std::lock_guard<std::mutex> lk(st.mu);
        out.swap(st.kept);
    }
    release(out);
    size_t bytes = 0;
    for (const Block &b : out) bytes += b.bytes;
    return bytes;
}

hipError_t pool_get(void **p, size_t bytes)
{
    if (bytes < SMALLEST) return device_malloc(p, bytes);
    bytes = (bytes + GRAIN - 1) / GRAIN * GRAIN;
    int device = 0;
    const hipError_t e = hipGetDevice(&device);
    if (e != hipSuccess) return e;
    State &st = state();
    Blocks idle;
    *p = nullptr;
    {
        std::lock_guard<std::mutex> lk(st.mu);
        auto best = st.kept.end();
        for (auto b = st.kept.begin(); b != st.kept.end(); ++b)
            if (b->device == device && b->bytes >= bytes && b->bytes - bytes <= bytes / 4 &&
                (best == st.kept.end() || b->bytes < best->bytes))
                best = b;
        if (best != st.kept.end()) {
            st.at.emplace(best->p, best);
            st.used.splice(st.used.end(), st.kept, best);
            *p = best->p;
        }
        take_idle(st, idle);
    }
    release(idle);
    if (*p) return hipSuccess;
    const hipError_t e2 = device_malloc(p, bytes);
    if (e2 != hipSuccess) return e2;
    std::lock_guard<std::mutex> lk(st.mu);
    Blocks one(1, Block{ *p, bytes, device, limit_of(st, device), Clock::now() });
    st.at.emplace(*p, one.begin());
    st.used.splice(st.used.end(), one);
    return hipSuccess;
}

void pool_put(void *p)
{
    if (!p) return;
    State &st = state();
    Blocks out;
    bool foreign = false;
    {
        std::lock_guard<std::mutex> lk(st.mu);
        const auto it = st.at.find(p);
        if (it == st.at.end()) {
            foreign = true;
        } else {
            const auto b = it->second;
            st.at.erase(it);
            b->since = Clock::now();
            st.kept.splice(st.kept.end(), st.used, b);
            const int device = b->device;
            const size_t limit = b->limit;
            size_t sum = 0, old = 0;   // of the device's kept blocks; of those that would go
            for (const Block &k : st.kept) sum += k.device == device ? k.bytes : 0;
            for (const Block &k : st.kept) {
                if (sum - old <= limit) break;
                if (k.device == device && k.p != p) old += k.bytes;
            }
            if (sum - old > limit || old > b->bytes)   // dropped rather than blocks that took longer to get
                out.splice(out.end(), st.kept, b);
            else
                take(st, out, [&](const Block &k) {
                    if (k.device != device || sum <= limit) return false;
                    sum -= k.bytes;
                    return true;
                });
        }
        take_idle(st, out);
    }
    if (foreign) (void)hipFree(p);
    release(out);
}

}  // namespace bie
