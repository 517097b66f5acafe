// Reads of per-node values to the host: fields and populations as arrays of
// doubles (lbcg_fields, lbcg_populations).
//
// A copy to pageable memory runs at 10 to 18 GB/s here: the runtime copies
// through buffers of its own on the calling thread, which also takes the page
// faults of a fresh destination.  Reads of kMinBytes and more therefore go
// through two pinned slots in chunks: while the device fills and sends one,
// the calling thread and kHelpers others copy the other out in pieces.  Fields
// of 256^3 nodes (0.8 GB) 79 -> 23 ms (28 with 3 helpers), of 96^3 2.4 -> 1.1
// ms, of 45 x 38 x 53 (4.4 MB) 0.26 -> 0.20 ms; 3 MB are even.
//
// The slots and helpers are one set per process, given back with the last
// handle; a read that finds them in use by another thread, or cannot have them,
// takes the plain copies.  To make and give them back costs 0.24 ms, what reads
// of kFirstBytes in all gain: before that many bytes have been read since they
// were last given back there are none, so that a program that holds one lattice
// at a time and reads it once does not pay for them each time (45 x 38 x 53: 0.40
// ms a read and lattice with them, 0.26 with plain copies).  Helpers started for
// each read were slower where the program's own threads keep the CPUs busy: the
// read then waits for each to be run once (16 boxes, each read followed by a
// conversion on 16 threads: 52 ms in all against 12, and 18 with plain copies).
#include <hip/hip_runtime.h>
#include <sched.h>

#include <atomic>
#include <condition_variable>
#include <cstdint>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <thread>

#include "lbcg_sim.h"

namespace lbcg {

namespace {

constexpr size_t kSlotBytes = size_t(8) << 20;
constexpr size_t kMinBytes = size_t(4) << 20;
constexpr size_t kFirstBytes = size_t(12) << 20;
constexpr int kHelpers = 7;
constexpr int64_t kPiece = 32768;  // doubles

// Whether a read into p gains by the slots: pageable memory.  (The device writes
// to pinned memory itself, as fast: 64^3 nodes 0.30 ms against 0.36 through the
// slots; and only the runtime can write to a device's.)
bool pageable(const void *p) {
    hipPointerAttribute_t at{};
    if (hipPointerGetAttributes(&at, p) != hipSuccess) {
        (void)hipGetLastError();  // pageable memory is not known to the runtime
        return true;
    }
    return at.type == hipMemoryTypeUnregistered;
}
// Whether the rows of N doubles can go through the slots: all pageable, and none
// over another (the threads copy rows at the same time; in the plain copies the
// last row stands).
bool for_slots(int rows, double *const *dst, int64_t N) {
    for (int r = 0; r < rows; ++r) {
        if (!dst[r]) continue;
        const uintptr_t a = reinterpret_cast<uintptr_t>(dst[r]), len = sizeof(double) * uintptr_t(N);
        for (int q = 0; q < r; ++q) {
            const uintptr_t b = reinterpret_cast<uintptr_t>(dst[q]);
            if (dst[q] && a < b + len && b < a + len) return false;
        }
        if (!pageable(dst[r])) return false;
    }
    return true;
}

// Helper threads: the other CPUs that this thread may run on, to a limit.
int helper_count() {
    cpu_set_t set;
    CPU_ZERO(&set);
    const int n = sched_getaffinity(0, sizeof(set), &set) == 0 ? CPU_COUNT(&set) - 1 : 0;
    return n < 0 ? 0 : (n < kHelpers ? n : kHelpers);
}

// One read in progress.  Every chunk has the same number of pieces, numbered
// on through the chunks (the last chunk's may be short or empty); whoever is
// free takes the next one of those that have arrived, so that a helper that
// the system is slow to run holds up nothing but a piece that it has taken.
struct Read {
    double *dst[2 * D3Q19::Q];
    int rows;
    int64_t N, chunk, chunks, per_row, pieces;
    const char *slot[2];
    std::atomic<int64_t> next{0};       // first piece not taken
    std::atomic<int64_t> arrived{0};    // pieces that have arrived
    std::atomic<int64_t> done[2] = {};  // pieces copied out of each slot

    int64_t count(int64_t c) const { return (N - c * chunk) < chunk ? (N - c * chunk) : chunk; }
    bool waiting() const { return next.load() < arrived.load(); }
    // Copies pieces until none is left of those that have arrived.
    void work() {
        int64_t g = next.load(std::memory_order_relaxed);
        for (;;) {
            if (g >= arrived.load(std::memory_order_acquire)) return;
            if (!next.compare_exchange_weak(g, g + 1, std::memory_order_relaxed)) continue;
            const int64_t c = g / pieces, k = g - c * pieces, r = k / per_row, a = (k - r * per_row) * kPiece;
            const int64_t cnt = count(c), n = cnt - a < kPiece ? cnt - a : kPiece;
            if (dst[r] && n > 0)
                std::memcpy(dst[r] + c * chunk + a, reinterpret_cast<const double *>(slot[c & 1]) + r * cnt + a,
                            sizeof(double) * size_t(n));
            done[c & 1].fetch_add(1, std::memory_order_release);
            g = next.load(std::memory_order_relaxed);
        }
    }
    // until chunk c is copied
    void drained(int64_t c) const {
        while (done[c & 1].load(std::memory_order_acquire) < (c / 2 + 1) * pieces) std::this_thread::yield();
    }
};

// The pinned slots and the helpers.
struct Pool {
    char *mem = nullptr;
    std::thread helpers[kHelpers];
    int started = 0;
    std::mutex m;
    std::condition_variable cv;
    std::shared_ptr<Read> read;  // the read in progress
    bool stop = false;

    void help() {
        for (;;) {
            std::shared_ptr<Read> r;
            {
                std::unique_lock<std::mutex> lock(m);
                cv.wait(lock, [this] { return stop || (read && read->waiting()); });
                if (stop) return;
                r = read;
            }
            r->work();
        }
    }
    bool open() {
        RelaxedCapture relaxed;
        const hipError_t e = hipHostMalloc(reinterpret_cast<void **>(&mem), 2 * kSlotBytes, hipHostMallocPortable);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            mem = nullptr;
            return false;
        }
        const int want = helper_count();
        try {
            for (; started < want; ++started) helpers[started] = std::thread([this] { help(); });
        } catch (...) {  // fewer helpers, then
        }
        return true;
    }
    ~Pool() {
        {
            std::lock_guard<std::mutex> lock(m);
            stop = true;
        }
        cv.notify_all();
        for (int h = 0; h < started; ++h) helpers[h].join();
        if (mem) (void)hipHostFree(mem);
    }
    void set(const std::shared_ptr<Read> &r) {
        std::lock_guard<std::mutex> lock(m);
        read = r;
    }
    void arrive(Read &r, int64_t c) {
        {
            std::lock_guard<std::mutex> lock(m);
            r.arrived.store((c + 1) * r.pieces, std::memory_order_release);
        }
        cv.notify_all();
    }
};

std::mutex g_use;                   // held for the length of a read through the pool
std::atomic<int64_t> g_handles{0};
size_t g_plain = 0;                 // bytes of such reads since there were slots (under g_use)
Pool *g_pool = nullptr;             // never freed at exit: its helpers may still wait

hipError_t queue_chunk(lbcg_sim *s, RowsLaunch launch, const Read &rd, int64_t c, double *dev, double *host) {
    double *const *dst = rd.dst;
    const int64_t cnt = rd.count(c);
    hipError_t e = launch(s, c * rd.chunk, cnt, dev);
    for (int r = 0; r < rd.rows && e == hipSuccess;) {  // runs of wanted rows
        if (!dst[r]) {
            ++r;
            continue;
        }
        int r1 = r + 1;
        while (r1 < rd.rows && dst[r1]) ++r1;
        e = hipMemcpyAsync(host + r * cnt, dev + r * cnt, sizeof(double) * size_t((r1 - r) * cnt),
                           hipMemcpyDeviceToHost, s->stream);
        r = r1;
    }
    return e;
}

hipError_t read_slots(lbcg_sim *s, RowsLaunch launch, int rows, double *const *dst, Pool &pool) {
    const std::shared_ptr<Read> shared = std::make_shared<Read>();
    Read &rd = *shared;
    for (int r = 0; r < rows; ++r) rd.dst[r] = dst[r];
    rd.rows = rows;
    rd.N = s->g.N;
    // a chunk fits a slot and half of the device staging
    const int64_t half = s->staging_nodes * (2 * s->Q > 6 ? 2 * s->Q : 6) / 2, fit = int64_t(kSlotBytes / sizeof(double));
    rd.chunk = (half < fit ? half : fit) / rows;
    rd.chunks = (rd.N + rd.chunk - 1) / rd.chunk;
    rd.per_row = (rd.chunk + kPiece - 1) / kPiece;
    rd.pieces = rd.per_row * rows;
    for (int k = 0; k < 2; ++k) rd.slot[k] = pool.mem + size_t(k) * kSlotBytes;
    auto queue = [&](int64_t c) {
        const int k = int(c & 1);
        return queue_chunk(s, launch, rd, c, s->staging + k * half,
                           reinterpret_cast<double *>(pool.mem + size_t(k) * kSlotBytes));
    };
    hipError_t e = queue(0);
    pool.set(shared);
    for (int64_t c = 0; c < rd.chunks && e == hipSuccess; ++c) {
        // chunk c is the last work queued.  (No events: they belong to the device
        // current in the calling thread, which need not be the handle's.)
        e = hipStreamSynchronize(s->stream);
        if (e != hipSuccess) break;
        pool.arrive(rd, c);
        if (c + 1 < rd.chunks) {
            if (c > 0) rd.drained(c - 1);
            e = queue(c + 1);
        }
        rd.work();
    }
    // every piece that has arrived is copied, also after an error: no helper
    // writes to the caller's memory later, and nothing is left in flight
    rd.work();
    const int64_t in = rd.arrived.load() / rd.pieces;
    for (int64_t c = in < 2 ? 0 : in - 2; c < in; ++c) rd.drained(c);
    pool.set(nullptr);
    if (e != hipSuccess) (void)hipStreamSynchronize(s->stream);
    return e;
}

}  // namespace

void slots_use() { g_handles.fetch_add(1); }

void slots_release() {
    if (g_handles.fetch_sub(1) != 1) return;
    std::lock_guard<std::mutex> lock(g_use);
    if (g_handles.load() != 0) return;
    delete g_pool;
    g_pool = nullptr;
    g_plain = 0;
}

// The pool for a read of so many bytes, for the thread that holds g_use; null if
// it does not pay yet or cannot be had.
static Pool *pool(size_t bytes) {
    if (!g_pool) {
        g_plain = bytes < kFirstBytes ? g_plain + bytes : kFirstBytes;
        if (g_plain < kFirstBytes) return nullptr;
        g_pool = new (std::nothrow) Pool;
        if (g_pool && !g_pool->open()) {
            delete g_pool;
            g_pool = nullptr;
        }
    }
    return g_pool;
}

hipError_t read_rows(lbcg_sim *s, RowsLaunch launch, int rows, double *const *dst) {
    const int64_t N = s->g.N, C = s->staging_nodes;
    int64_t wanted = 0;
    for (int r = 0; r < rows; ++r) wanted += dst[r] ? 1 : 0;
    const size_t bytes = size_t(wanted) * sizeof(double) * size_t(N);
    if (bytes >= kMinBytes && for_slots(rows, dst, N)) {
        std::unique_lock<std::mutex> lock(g_use, std::try_to_lock);
        Pool *p = lock.owns_lock() ? pool(bytes) : nullptr;
        if (p) {
            try {
                return read_slots(s, launch, rows, dst, *p);
            } catch (const std::bad_alloc &) {  // thrown before anything is queued
            }
        }
    }
    for (int64_t n0 = 0; n0 < N; n0 += C) {
        const int64_t cnt = (N - n0) < C ? (N - n0) : C;
        hipError_t e = launch(s, n0, cnt, s->staging);
        for (int r = 0; r < rows && e == hipSuccess; ++r)
            if (dst[r])
                e = hipMemcpyAsync(dst[r] + n0, s->staging + int64_t(r) * cnt, sizeof(double) * size_t(cnt),
                                   hipMemcpyDeviceToHost, s->stream);
        if (e == hipSuccess) e = hipStreamSynchronize(s->stream);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace lbcg
