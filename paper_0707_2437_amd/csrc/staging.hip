// Host-array transfers: device memory to the caller's pageable arrays through
// pinned staging, and the device memory pool of DevScratch.
//
// What bounds a large copy out is the host side: the runtime's pageable copy
// moves one stretch after another on one thread, which also takes the page
// faults of a new array. Here DMA into a ring of pinned chunks runs ahead of a
// few threads that copy 256 KiB pieces from the ring to the array, in order of
// their arrival. Populations of a 1024^2 lattice into a new array (75 MB) 7.2
// -> 2.6 ms, the first time 7.3 -> 3.3; 4096^2 (1.2 GB) 115 -> 39 ms. DMA
// alone at the link's 57 GB/s would take 1.3 and 21 ms. Copies in are left to
// the runtime: 37 GB/s, and staging with any number of threads no faster.
#include <atomic>
#include <condition_variable>
#include <cstring>
#include <mutex>
#include <thread>

#include "host.h"

namespace lbm {
namespace {

constexpr size_t kPiece = 256 << 10;
// Below this a copy is the runtime's. A team of threads would gain there too
// (25 MB 1.6 -> 0.8 ms), but a program that hands smaller reads on to a
// threaded host library, whose own threads spin between calls, is slowed by
// the scheduler more than that: 32 reads of 9 MB each followed by a
// multi-threaded copy, 31 ms without the team, 50 to 110 with it.
constexpr size_t kStageFrom = 32 << 20;
constexpr int kMaxWorkers = 6;  // 12 us each to start; DMA-bound from 4 (huge pages) or 8 (small ones)
// A DMA takes 13 us to set up and 18 us per MiB. A new ring costs 1.6 us per
// 4 KiB page at its first touch, shared by the team: larger slots gain 0.4 ms
// on 75 MB and lose 2 on the first read of a program.
constexpr int kSlots = 8;
constexpr size_t kSlot = 1 << 20;
constexpr int kPieces = (int)(kSlot / kPiece);
constexpr int kKeepRings = 2;
constexpr size_t kKeepScratch = (size_t)256 << 20;
constexpr int kMaxDevices = 16;

// The device of stream st's work (of the null stream: the current one), which
// need not be the calling thread's current device.
hipError_t stream_device(hipStream_t st, int* device)
{
    hipDevice_t d = 0;
    if (st && hipStreamGetDevice(st, &d) == hipSuccess) {
        *device = d;
        return hipSuccess;
    }
    return hipGetDevice(device);
}

// Makes a device current for its life.
struct OnDevice {
    int before = -1;
    hipError_t e;
    explicit OnDevice(int device)
    {
        e = hipGetDevice(&before);
        if (e == hipSuccess && before == device) before = -1;
        else if (e == hipSuccess) e = hipSetDevice(device);
    }
    ~OnDevice()
    {
        if (before >= 0) (void)hipSetDevice(before);
    }
};

struct Ring {
    char* p = nullptr;
    int device = -1;
    hipEvent_t ev[kSlots] = {};
};

// What outlives one call: at most kKeepRings rings and kKeepScratch bytes of
// device scratch per device, while any lattice or pool lives; and one page of
// totals, whose lines are given back to it (a page freed with the last object
// costs the next one 50 us to 1 ms).
std::mutex g_lock;
int g_users = 0;
constexpr int kLines = 64;           // of a page, 64 bytes each
char* g_page = nullptr;
unsigned long long g_lines_used = 0; // bit per line
Ring g_kept[kKeepRings];
hipMemPool_t g_scratch[kMaxDevices] = {};

void free_ring(Ring& r)
{
    for (hipEvent_t& ev : r.ev)
        if (ev) (void)hipEventDestroy(ev);
    if (r.p) (void)hipHostFree(r.p);
    r = Ring();
}

struct RingLease {
    Ring r;
    bool sound = false;  // every call on it succeeded
    hipError_t take(int device)  // events are recorded on streams of their own device only
    {
        {
            std::lock_guard<std::mutex> hold(g_lock);
            for (Ring& k : g_kept)
                if (k.p && k.device == device) {
                    r = k;
                    k = Ring();
                    return hipSuccess;
                }
        }
        r.device = device;
        OnDevice on(device);
        hipError_t e = on.e;
        if (e == hipSuccess) e = hipHostMalloc((void**)&r.p, kSlots * kSlot, hipHostMallocDefault);
        if (e != hipSuccess) r.p = nullptr;
        for (hipEvent_t& ev : r.ev)
            if (e == hipSuccess) e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
        return e;
    }
    ~RingLease()
    {
        if (sound) {
            std::lock_guard<std::mutex> hold(g_lock);
            if (g_users > 0)
                for (Ring& k : g_kept)
                    if (!k.p) {
                        k = r;
                        return;
                    }
        }
        free_ring(r);
    }
};

// Whether the runtime copies to p with one DMA by itself: pinned, managed or
// device memory.
bool direct(const void* p)
{
    hipPointerAttribute_t a{};
    if (hipPointerGetAttributes(&a, p) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return a.type != hipMemoryTypeUnregistered;
}

// The chunks of all parts in order, each within one part.
struct Plan {
    const HostPart* part;
    int nparts;
    int total = 0;
    Plan(const HostPart* p, int n) : part(p), nparts(n)
    {
        for (int k = 0; k < n; ++k) total += chunks(k);
    }
    int chunks(int k) const { return part[k].dst ? (int)((part[k].bytes + kSlot - 1) / kSlot) : 0; }
    void at(int c, char** dst, const char** src, size_t* len) const
    {
        int k = 0;
        while (c >= chunks(k)) c -= chunks(k++);
        const size_t o = (size_t)c * kSlot, left = part[k].bytes - o;
        *dst = (char*)part[k].dst + o;
        *src = (const char*)part[k].src + o;
        *len = left < kSlot ? left : kSlot;
    }
};

// State shared with the workers. A worker claims the pieces of the chunks in
// order; it waits for the next chunk's DMA, whose end the caller reports, or
// that it gave up.
struct Shared {
    const Plan& plan;
    char* ring;
    std::mutex lock;  // of ready and stop
    std::condition_variable more;
    int ready = 0;  // chunks whose DMA has ended
    bool stop = false;
    std::atomic<long> claim{0};             // next piece
    std::atomic<int> left[kSlots] = {};  // pieces of the slot's chunk not yet copied (a short chunk's last are empty)
    Shared(const Plan& p, char* r) : plan(p), ring(r) {}

    char* slot(int c) const { return ring + (size_t)(c % kSlots) * kSlot; }
    std::atomic<int>& pending(int c) { return left[c % kSlots]; }
    void report(int chunks, bool give_up)
    {
        {
            std::lock_guard<std::mutex> hold(lock);
            ready = chunks;
            stop = give_up;
        }
        more.notify_all();
    }
    void copy_piece(int c, long q)
    {
        char* dst;
        const char* src;
        size_t len;
        plan.at(c, &dst, &src, &len);
        const size_t o = (size_t)q * kPiece;
        if (o < len) std::memcpy(dst + o, slot(c) + o, len - o < kPiece ? len - o : kPiece);
        pending(c).fetch_sub(1, std::memory_order_release);
    }
    void work()
    {
        for (;;) {
            const long k = claim.fetch_add(1, std::memory_order_relaxed);
            const int c = (int)(k / kPieces);
            if (c >= plan.total) return;
            {
                std::unique_lock<std::mutex> hold(lock);
                more.wait(hold, [&] { return ready > c || stop; });
                if (stop) return;
            }
            copy_piece(c, k % kPieces);
        }
    }
};

hipError_t staged(const Plan& plan, RingLease& lease, hipStream_t st)
{
    hipError_t e = hipSuccess;
    Shared sh(plan, lease.r.p);
    int sent = 0;
    // starts the DMA of every chunk whose slot is free
    auto send = [&] {
        while (e == hipSuccess && sent < plan.total && sh.pending(sent).load(std::memory_order_acquire) == 0) {
            char* dst;
            const char* src;
            size_t len;
            plan.at(sent, &dst, &src, &len);
            sh.pending(sent).store(kPieces, std::memory_order_relaxed);
            e = hipMemcpyAsync(sh.slot(sent), src, len, hipMemcpyDeviceToHost, st);
            if (e == hipSuccess) e = hipEventRecord(lease.r.ev[sent % kSlots], st);
            ++sent;
        }
    };
    std::thread team[kMaxWorkers];
    int workers = 0;
    for (int c = 0; c < plan.total; ++c) {
        send();
        while (e == hipSuccess && sent <= c) {
            std::this_thread::yield();
            send();
        }
        if (e == hipSuccess) e = hipEventSynchronize(lease.r.ev[c % kSlots]);
        if (e != hipSuccess) break;
        sh.report(c + 1, false);
        if (c == 0) {  // only now: what the stream had to do before is done
            try {
                while (workers < kMaxWorkers) {
                    team[workers] = std::thread([&sh] { sh.work(); });
                    ++workers;
                }
            } catch (...) {
                // no more threads to be had; with none at all this one copies
            }
        }
        if (workers == 0)
            for (long q = 0; q < kPieces; ++q) sh.copy_piece(c, q);
    }
    if (e != hipSuccess) sh.report(0, true);
    for (int k = 0; k < workers; ++k) team[k].join();
    // the ring goes back only when no DMA writes to it any more
    const hipError_t es = hipStreamSynchronize(st);
    if (e == hipSuccess) e = es;
    lease.sound = e == hipSuccess;
    return e;
}

}  // namespace

void staging_retain()
{
    std::lock_guard<std::mutex> hold(g_lock);
    ++g_users;
}

void staging_release()
{
    Ring gone[kKeepRings];
    {
        std::lock_guard<std::mutex> hold(g_lock);
        if (--g_users > 0) return;
        for (int k = 0; k < kKeepRings; ++k) {
            gone[k] = g_kept[k];
            g_kept[k] = Ring();
        }
        for (hipMemPool_t m : g_scratch)
            if (m) (void)hipMemPoolTrimTo(m, 0);
    }
    for (Ring& r : gone) free_ring(r);
}

// A line of the page, or memory of its own beyond kLines objects: an
// allocation for each takes 15 us, 50 while others are alive.
hipError_t totals_alloc(double** p)
{
    constexpr unsigned kind = hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent;
    *p = nullptr;
    std::lock_guard<std::mutex> hold(g_lock);
    if (!g_page) {
        const hipError_t e = hipHostMalloc((void**)&g_page, (size_t)kLines * 64, kind);
        if (e != hipSuccess) {
            g_page = nullptr;
            return e;
        }
    }
    for (int k = 0; k < kLines; ++k)
        if (!(g_lines_used >> k & 1)) {
            g_lines_used |= 1ull << k;
            *p = (double*)(g_page + (size_t)k * 64);
            return hipSuccess;
        }
    return hipHostMalloc((void**)p, 64, kind);
}

void totals_free(double* p)
{
    if (!p) return;
    {
        std::lock_guard<std::mutex> hold(g_lock);
        if (g_page && (char*)p >= g_page && (char*)p < g_page + (size_t)kLines * 64) {
            g_lines_used &= ~(1ull << (((char*)p - g_page) / 64));
            return;
        }
    }
    (void)hipHostFree(p);
}

// Gives idle scratch of a device back to it: true if there may be memory that
// was not to be had before. Waits for the device, since a block is idle only
// when the calls that used it are done; its callers have run out of memory.
static bool return_scratch(int device)
{
    hipMemPool_t m = nullptr;
    if (device >= 0 && device < kMaxDevices) {
        std::lock_guard<std::mutex> hold(g_lock);
        m = g_scratch[device];
    }
    if (!m) return false;
    OnDevice on(device);
    (void)hipDeviceSynchronize();
    const bool some = hipMemPoolTrimTo(m, 0) == hipSuccess;
    (void)hipGetLastError();
    return some;
}

hipError_t device_malloc(void** p, size_t bytes)
{
    hipError_t e = hipMalloc(p, bytes);
    int device = 0;
    if (e == hipErrorOutOfMemory && hipGetDevice(&device) == hipSuccess && return_scratch(device)) e = hipMalloc(p, bytes);
    if (e != hipSuccess) *p = nullptr;
    return e;
}

hipError_t scratch_alloc(void** p, size_t bytes, hipStream_t st)
{
    *p = nullptr;
    int device = 0;
    hipError_t e = stream_device(st, &device);
    hipMemPool_t m = nullptr;
    if (e == hipSuccess && device < kMaxDevices) {
        std::lock_guard<std::mutex> hold(g_lock);
        if (!g_scratch[device]) {
            hipMemPoolProps props{};
            props.allocType = hipMemAllocationTypePinned;
            props.location.type = hipMemLocationTypeDevice;
            props.location.id = device;
            uint64_t keep = kKeepScratch;
            hipMemPool_t fresh = nullptr;
            if (hipMemPoolCreate(&fresh, &props) == hipSuccess) {
                if (hipMemPoolSetAttribute(fresh, hipMemPoolAttrReleaseThreshold, &keep) == hipSuccess)
                    g_scratch[device] = fresh;
                else
                    (void)hipMemPoolDestroy(fresh);
            }
        }
        m = g_scratch[device];
    }
    if (e == hipSuccess) e = m ? hipMallocFromPoolAsync(p, bytes, m, st) : hipMallocAsync(p, bytes, st);
    if (e == hipErrorOutOfMemory && m && return_scratch(device)) e = hipMallocFromPoolAsync(p, bytes, m, st);
    if (e != hipSuccess) *p = nullptr;
    return e;
}

hipError_t copy_out(const HostPart* part, int nparts, hipStream_t st)
{
    size_t bytes = 0;
    bool stage = true;
    for (int k = 0; k < nparts; ++k) {
        if (!part[k].dst) continue;
        bytes += part[k].bytes;
        if (direct(part[k].dst)) stage = false;
    }
    if (stage && bytes >= kStageFrom) {
        RingLease lease;
        int device = 0;
        hipError_t e = stream_device(st, &device);
        if (e == hipSuccess) e = lease.take(device);
        if (e == hipSuccess && (e = staged(Plan(part, nparts), lease, st)) != hipErrorOutOfMemory) return e;
        // no pinned memory left, or none to be had while another thread
        // captures a graph: as small copies go
        (void)hipGetLastError();
    }
    hipError_t e = hipSuccess;
    for (int k = 0; k < nparts && e == hipSuccess; ++k)
        if (part[k].dst) e = hipMemcpyAsync(part[k].dst, part[k].src, part[k].bytes, hipMemcpyDeviceToHost, st);
    // also after a failure: no copy of an earlier part may outlive the call
    const hipError_t es = hipStreamSynchronize(st);
    return e == hipSuccess ? es : e;
}

}  // namespace lbm
