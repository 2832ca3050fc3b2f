// C ABI of libtictac: argument checks, graph validation and levelling, the dependency
// sets of small graphs (large ones are propagated by the kernels), grouping of compute
// ops into classes of identical dependency sets, the tables that the kernels read, and
// the calls into the kernel launchers.  Everything per timing sample runs in the kernels.
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <exception>
#include <future>
#include <memory>
#include <mutex>
#include <numeric>
#include <system_error>

#include "chain_plan.h"
#include "frontier_plan.h"
#include "internal.h"

namespace tictac {

static thread_local char g_err[512] = "";

void set_error(const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
}

// No exception leaves an entry point: each is a function try block that ends in TT_CATCH.
static int caught()
{
    try {
        throw;
    } catch (const std::bad_alloc &) {
        set_error("out of host memory");
    } catch (const std::exception &e) {             // (a length or a thread that the host cannot provide)
        set_error("out of host resources: %s", e.what());
    } catch (...) {
        set_error("out of host resources");
    }
    return TICTAC_ERR_NO_MEM;
}
#define TT_CATCH catch (...) { return caught(); }

#define HIP_TRY(expr)                                                                        \
    do {                                                                                     \
        hipError_t e_ = (expr);                                                              \
        if (e_ != hipSuccess) {                                                              \
            set_error("%s failed: %s (%s:%d)", #expr, hipGetErrorString(e_), __FILE__, __LINE__); \
            return TICTAC_ERR_HIP;                                                           \
        }                                                                                    \
    } while (0)

// Device memory of the handles.  A program that takes in one graph after another allocates and frees blocks of the
// same sizes all the time, and hipMalloc and hipFree cost tens of microseconds each, large blocks much more.  Freed
// blocks are therefore kept, up to kPoolMax bytes per process (the oldest go first), and given back to the runtime when
// an allocation fails and by tictac_trim_memory.  A block is freed only after the device has finished what was queued (as hipFree does), so the
// next owner may use it on any stream.
constexpr size_t kPoolMax = (size_t)1 << 30;
struct PoolBlock { void *p; size_t bytes; int device; };
static std::mutex g_pool_mutex;
static std::vector<PoolBlock> g_pool;               // oldest first
static size_t g_pool_bytes = 0;

// sizes in steps of an eighth, so that blocks of nearly equal requests serve each other
static size_t pool_size(size_t bytes)
{
    size_t step = 4096;
    while (step * 16 < bytes) step *= 2;
    return (bytes + step - 1) / step * step;
}

static hipError_t pool_alloc(void **p, size_t bytes)
{
    *p = nullptr;
    const size_t want = pool_size(bytes);
    int device = 0;
    hipError_t e = hipGetDevice(&device);
    if (e != hipSuccess) return e;
    {
        std::lock_guard<std::mutex> lock(g_pool_mutex);
        for (size_t i = g_pool.size(); i-- > 0;)
            if (g_pool[i].bytes == want && g_pool[i].device == device) {
                *p = g_pool[i].p;
                g_pool_bytes -= want;
                g_pool.erase(g_pool.begin() + i);
                return hipSuccess;
            }
    }
    e = hipMalloc(p, want);
    if (e != hipErrorOutOfMemory) return e;
    (void)hipGetLastError();
    {
        std::lock_guard<std::mutex> lock(g_pool_mutex);
        for (const PoolBlock &b : g_pool) (void)hipFree(b.p);
        g_pool.clear();
        g_pool_bytes = 0;
    }
    e = hipMalloc(p, want);
    if (e != hipSuccess) (void)hipGetLastError();       // (else the next launch would report it)
    return e;
}

// (the device has finished with the block)
static void pool_put(void *p, size_t bytes, int device) noexcept
{
    if (!p) return;
    const size_t want = pool_size(bytes);
    if (want > kPoolMax) { (void)hipFree(p); return; }
    std::lock_guard<std::mutex> lock(g_pool_mutex);
    try {
        g_pool.push_back({p, want, device});
    } catch (const std::bad_alloc &) {
        (void)hipFree(p);
        return;
    }
    g_pool_bytes += want;
    size_t n = 0;
    while (g_pool_bytes > kPoolMax) { g_pool_bytes -= g_pool[n].bytes; (void)hipFree(g_pool[n++].p); }
    g_pool.erase(g_pool.begin(), g_pool.begin() + n);
}

// Gives a block of a handle back once the device has finished with it.
static hipError_t release(Block &b, int device)
{
    if (!b.p) return hipSuccess;
    const hipError_t e = hipDeviceSynchronize();
    if (e != hipSuccess) return e;
    pool_put(b.p, b.bytes, device);
    b = Block();
    return hipSuccess;
}

// Pinned host memory for transfers (pinning costs milliseconds, and copies from or to pageable memory are staged by the
// runtime and take three to four times as long).  Blocks that nobody uses are kept for the next taker, any thread, up to
// kPinnedKept bytes per process.
constexpr size_t kStageMax = (size_t)96 << 20, kPinnedKept = (size_t)192 << 20;
static std::mutex g_pinned_mutex;
static std::vector<Block> g_pinned;                 // oldest first
static size_t g_pinned_bytes = 0;

// Holds a block while its owner lives.  NULL when the request is empty, beyond the cap, or cannot be pinned: the caller then
// copies from or to its own pageable memory.
class Stage {
    Block b;
public:
    Stage() = default;
    Stage(const Stage &) = delete;
    Stage &operator=(const Stage &) = delete;
    ~Stage() { give_back(); }

    void *take(size_t bytes)
    {
        give_back();
        if (bytes == 0 || bytes > kStageMax) return nullptr;
        {
            std::lock_guard<std::mutex> lock(g_pinned_mutex);
            for (size_t i = g_pinned.size(); i-- > 0;)
                if (g_pinned[i].bytes >= bytes) {
                    b = g_pinned[i];
                    g_pinned.erase(g_pinned.begin() + i);
                    g_pinned_bytes -= b.bytes;
                    return b.p;
                }
        }
        const size_t want = (bytes + ((size_t)1 << 20) - 1) & ~(((size_t)1 << 20) - 1);
        if (hipHostMalloc(&b.p, want, hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            b.p = nullptr;
            return nullptr;
        }
        b.bytes = want;
        return b.p;
    }
    // (no copy from or to it is under way)
    void give_back() noexcept
    {
        if (!b.p) return;
        std::lock_guard<std::mutex> lock(g_pinned_mutex);
        try {
            g_pinned.push_back(b);
            g_pinned_bytes += b.bytes;
        } catch (const std::bad_alloc &) {
            (void)hipHostFree(b.p);
        }
        b = Block();
        while (g_pinned_bytes > kPinnedKept) {
            g_pinned_bytes -= g_pinned[0].bytes;
            (void)hipHostFree(g_pinned[0].p);
            g_pinned.erase(g_pinned.begin());
        }
    }
};

// Gives back what the pool and the staging blocks keep; what the runtime does not take stays.
static hipError_t trim_memory()
{
    hipError_t err = hipSuccess;
    auto drop = [&](void *p, bool pinned) {
        const hipError_t e = pinned ? hipHostFree(p) : hipFree(p);
        if (e != hipSuccess) { (void)hipGetLastError(); err = e; }
        return e == hipSuccess;
    };
    {
        std::lock_guard<std::mutex> lock(g_pool_mutex);
        for (size_t i = g_pool.size(); i-- > 0;)
            if (drop(g_pool[i].p, false)) {
                g_pool_bytes -= g_pool[i].bytes;
                g_pool.erase(g_pool.begin() + i);
            }
    }
    std::lock_guard<std::mutex> lock(g_pinned_mutex);
    for (size_t i = g_pinned.size(); i-- > 0;)
        if (drop(g_pinned[i].p, true)) {
            g_pinned_bytes -= g_pinned[i].bytes;
            g_pinned.erase(g_pinned.begin() + i);
        }
    return err;
}

constexpr size_t kCopyInMax = (size_t)512 << 10;

// Collects host arrays (and device-only reservations) into one device block: one allocation, one copy of each array
// into a pinned staging block and one host-to-device copy.  The arrays must live until commit(), and finish() waits for the
// copy (so does the destructor, where an error has come between).
struct Packer {
    struct Part { void **dst; const void *src; size_t bytes, off; };    // (src NULL: only kernels write it)
    std::vector<Part> parts;
    size_t host_bytes = 0, device_only = 0;     // the copied arrays come first
    size_t alignment = 256;                     // of what comes behind them
    bool by_kernel = true;                      // (false: not by a kernel, for which a busy device may have no room)
    Stage staging;
    hipStream_t stream = nullptr;
    bool under_way = false;

    Packer() = default;
    ~Packer() { if (under_way) (void)hipStreamSynchronize(stream); }
    hipError_t finish()
    {
        const hipError_t e = hipStreamSynchronize(stream);
        if (e == hipSuccess) under_way = false;
        return e;
    }

    static size_t align(size_t x, size_t to = 256) { return (x + to - 1) & ~(to - 1); }

    template <typename T>
    void add(T **dst, const T *src, size_t n)
    {
        *dst = nullptr;
        if (!n) return;
        host_bytes = align(host_bytes);
        parts.push_back({reinterpret_cast<void **>(dst), src, n * sizeof(T), host_bytes});
        host_bytes += n * sizeof(T);
    }
    template <typename T>
    void add(T **dst, const std::vector<T> &src) { add(dst, src.data(), src.size()); }
    template <typename T>
    void reserve(T **dst, size_t n_bytes, size_t at = 256)
    {
        *dst = nullptr;
        if (!n_bytes) return;
        alignment = std::max(alignment, at);
        device_only = align(device_only, at);
        parts.push_back({reinterpret_cast<void **>(dst), nullptr, n_bytes, device_only});
        device_only += align(n_bytes);
    }
    // What the block held is released first.  On an error no array of the packer is there, and what has been allocated
    // belongs to the block.
    hipError_t commit(Block &block, int device, hipStream_t s)
    {
        for (const Part &p : parts) *p.dst = nullptr;
        hipError_t e = release(block, device);
        const size_t behind = device_only ? align(host_bytes, alignment) : align(host_bytes), total = behind + device_only;
        if (e != hipSuccess || !total) return e;
        std::vector<char> pageable;
        char *st = stage(pageable);
        e = pool_alloc(&block.p, total);
        if (e != hipSuccess) return e;
        block.bytes = total;
        return send(static_cast<char *>(block.p), behind, st, pageable, s);
    }
    // The same into memory that a block has reserved, where nothing is allocated on the device.
    hipError_t commit_at(void *to, size_t room, hipStream_t s)
    {
        for (const Part &p : parts) *p.dst = nullptr;
        if (host_bytes > room || device_only) return hipErrorInvalidValue;
        std::vector<char> pageable;
        char *st = stage(pageable);
        return send(static_cast<char *>(to), 0, st, pageable, s);
    }

private:
    char *stage(std::vector<char> &pageable)
    {
        char *st = static_cast<char *>(staging.take(host_bytes));
        if (!st && host_bytes) {
            pageable.resize(host_bytes);
            st = pageable.data();
        }
        return st;
    }
    hipError_t send(char *to, size_t behind, char *st, const std::vector<char> &pageable, hipStream_t s)
    {
        hipError_t e = hipSuccess;
        for (const Part &p : parts)
            if (p.src) memcpy(st + p.off, p.src, p.bytes);
        stream = s;
        if (host_bytes) {
            under_way = true;
            // (small blocks: a kernel reads the pinned memory itself)
            if (by_kernel && pageable.empty() && host_bytes <= kCopyInMax) {
                e = launch_copy_in(to, st, host_bytes, s);
            } else {
                e = hipMemcpyAsync(to, st, host_bytes, hipMemcpyHostToDevice, s);
                if (!pageable.empty() && e == hipSuccess) e = hipStreamSynchronize(s);
            }
        }
        for (const Part &p : parts)
            if (e == hipSuccess) *p.dst = to + (p.src ? 0 : behind) + p.off;
        return e;
    }
};

int device_cu_count(int device)
{
    static thread_local int known_device = -1, known_count = 0;
    if (device == known_device) return known_count;
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || n <= 0) {
        (void)hipGetLastError();
        n = 256;
    }
    known_device = device;
    known_count = n;
    return n;
}

hipError_t ensure_dynamic_lds(const void *kernel, size_t bytes)
{
    // (one table for the process: the attribute belongs to the kernel on a device, not to a thread)
    struct Entry { int device; const void *kernel; size_t bytes; };
    static std::vector<Entry> known;
    static std::mutex mutex;
    int device = 0;
    hipError_t err = hipGetDevice(&device);
    if (err != hipSuccess) return err;
    std::lock_guard<std::mutex> lock(mutex);
    for (Entry &e : known)
        if (e.kernel == kernel && e.device == device) {
            if (bytes <= e.bytes) return hipSuccess;
            err = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
            if (err == hipSuccess) e.bytes = bytes;
            return err;
        }
    err = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (err == hipSuccess) known.push_back({device, kernel, bytes});
    return err;
}

hipError_t cached_blocks_per_cu(int *per_cu, const void *kernel, int threads, size_t lds)
{
    struct Entry { const void *kernel; int threads; size_t lds; int per_cu; };
    static thread_local std::vector<Entry> known;
    for (const Entry &e : known)
        if (e.kernel == kernel && e.threads == threads && e.lds == lds) { *per_cu = e.per_cu; return hipSuccess; }
    int n = 0;
    const hipError_t err = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, threads, lds);
    if (err != hipSuccess) return err;
    if (n < 1) n = 1;
    if (known.size() < 256) known.push_back({kernel, threads, lds, n});
    *per_cu = n;
    return hipSuccess;
}

hipError_t ensure_workspace(Dag *d, size_t bytes)
{
    if (bytes <= d->work_bytes) return hipSuccess;
    if (d->d_work) {
        hipError_t e = hipDeviceSynchronize();   // earlier users of the old block are done
        if (e != hipSuccess) return e;
        pool_put(d->d_work, d->work_bytes, d->device);
        d->d_work = nullptr;
        d->work_bytes = 0;
    }
    const size_t want = bytes + bytes / 8;
    const hipError_t e = pool_alloc(&d->d_work, want);
    if (e != hipSuccess) return e;
    d->work_bytes = want;
    return hipSuccess;
}

// Device copy of a channel table [R].  A table equal to the one already there is not sent
// again; a new one is copied synchronously after the work queued on the stream (which may
// still read the old table) has finished.
static hipError_t ensure_chan_table(Dag *d, const int32_t *chan, hipStream_t s)
{
    const size_t bytes = (size_t)d->R * sizeof(int32_t);
    if (d->d_chan && d->h_chan.size() == (size_t)d->R && memcmp(d->h_chan.data(), chan, bytes) == 0)
        return hipSuccess;
    hipError_t e;
    if (!d->d_chan) {
        e = pool_alloc((void **)&d->d_chan, bytes);
        if (e != hipSuccess) return e;
    }
    e = hipStreamSynchronize(s);
    if (e != hipSuccess) return e;
    d->h_chan.clear();
    e = hipMemcpy(d->d_chan, chan, bytes, hipMemcpyHostToDevice);
    if (e != hipSuccess) return e;
    d->h_chan.assign(chan, chan + d->R);
    return hipSuccess;
}

static void free_dag(Dag *d)
{
    if (!d) return;
    int device = 0;
    const bool other = hipGetDevice(&device) == hipSuccess && device != d->device;
    if (other) (void)hipSetDevice(d->device);
    // (whatever still runs on the blocks is waited for, on any stream; only then may another handle take them)
    const bool idle = hipDeviceSynchronize() == hipSuccess;
    const Block blocks[] = {
        d->graph_block, d->quad_block, d->class_block, {d->d_work, d->work_bytes}, {d->d_chan, (size_t)d->R * sizeof(int32_t)},
        d->send_block, d->chain.block, d->sliced_block, d->frontier.block};
    for (const auto &b : blocks) {
        if (!b.p) continue;
        if (idle) pool_put(b.p, b.bytes, d->device);
        else (void)hipFree(b.p);
    }
    if (other) (void)hipSetDevice(device);
    delete d;
}

// Groups the compute ops by identical dependency rows.  `rows` holds the rows of the
// compute ops in op_time column order.  Classes are numbered by their first member;
// a class with more than `max_members` ops is split into consecutive pieces (the
// pieces have the same row, which every kernel handles like distinct classes).
static void group_classes(const std::vector<uint64_t> &rows, int32_t N, int32_t W, int32_t max_members,
                          std::vector<uint64_t> &cls_dep, std::vector<int32_t> &cls_ptr,
                          std::vector<int32_t> &cls_cols, int32_t &n_distinct)
{
    // open-addressing table from row hash to the distinct row's number; scanning the ops in
    // ascending order numbers the distinct rows by first member and keeps members ascending
    size_t cap = 16;
    while (cap < (size_t)N * 2) cap <<= 1;
    std::vector<int32_t> slot(cap, -1);
    std::vector<int32_t> first;                 // first member of every distinct row
    std::vector<int32_t> cls_of(N), count;
    for (int32_t j = 0; j < N; ++j) {
        uint64_t h = 0x9E3779B97F4A7C15ull;
        for (int32_t w = 0; w < W; ++w) {
            h ^= rows[(size_t)j * W + w] + 0x9E3779B97F4A7C15ull + (h << 6) + (h >> 2);
            h *= 0xFF51AFD7ED558CCDull;
        }
        size_t q = (h ^ (h >> 29)) & (cap - 1);
        for (;;) {
            const int32_t c = slot[q];
            if (c < 0) {
                slot[q] = (int32_t)first.size();
                cls_of[j] = (int32_t)first.size();
                first.push_back(j);
                count.push_back(1);
                break;
            }
            if (W == 0 || memcmp(&rows[(size_t)first[c] * W], &rows[(size_t)j * W], (size_t)W * 8) == 0) {
                cls_of[j] = c;
                ++count[c];
                break;
            }
            q = (q + 1) & (cap - 1);
        }
    }
    n_distinct = (int32_t)first.size();
    // members of every distinct row, ascending (counting sort by row number)
    std::vector<int32_t> start(n_distinct + 1, 0);
    for (int32_t c = 0; c < n_distinct; ++c) start[c + 1] = start[c] + count[c];
    std::vector<int32_t> members(N), fill(start.begin(), start.end() - 1);
    for (int32_t j = 0; j < N; ++j) members[fill[cls_of[j]]++] = j;
    cls_dep.clear(); cls_ptr.clear(); cls_cols.clear();
    cls_ptr.push_back(0);
    for (int32_t c = 0; c < n_distinct; ++c)
        for (int32_t k = start[c]; k < start[c + 1]; k += max_members) {
            const int32_t e = std::min(start[c + 1], k + max_members);
            for (int32_t m = k; m < e; ++m) cls_cols.push_back(members[m]);
            cls_ptr.push_back((int32_t)cls_cols.size());
            for (int32_t w = 0; w < W; ++w) cls_dep.push_back(rows[(size_t)first[c] * W + w]);
        }
}

// Whether four lanes with one class should make one addition (Sums::quads in device_utils.h): a tenth of the columns have the
// class of the column 32 further on, that is, eight lanes and more add to one place one after the other.  Simulation with an order
// each, 20 000 samples, by quads and not: inception3 (a third of the columns) 225 and 244 us, several channels, 65 536, 932 and
// 988; 300 classes, one in thirty with 700 columns (two thirds) 240 and 251; 300 with 64 (half) 533 and 570; with 16, 12 and 17 or 1
// to 3 each (none) the test costs 1 to 5 %, 100 samples 4 to 8 %.
static bool long_class_runs(const std::vector<int32_t> &col_cls)
{
    size_t far = 0;
    for (size_t j = 0; j + 32 < col_cls.size(); j += 4) far += col_cls[j] == col_cls[j + 32];
    return far * 16 >= col_cls.size();
}

// The same grouping from the device's: rep[j] the lowest op with the row of op j.  first_col: the first member of every
// class (piece), whose row is the row of the class.
static void group_reps(const int32_t *rep, int32_t N, int32_t max_members, std::vector<int32_t> &cls_ptr,
                       std::vector<int32_t> &cls_cols, std::vector<int32_t> &first_col, std::vector<int32_t> &col_cls, int32_t &n_distinct)
{
    std::vector<int32_t> set_of(N), start((size_t)N + 1, 0);
    int32_t sets = 0;
    for (int32_t j = 0; j < N; ++j) {               // (whether an op starts a set could go either way: no branch)
        const bool fresh = rep[j] == j;
        const int32_t seen = set_of[rep[j]], set = fresh ? sets : seen;
        set_of[j] = set;
        sets += fresh;
        ++start[set + 1];
    }
    n_distinct = sets;
    start.resize((size_t)sets + 1);
    for (int32_t c = 0; c < n_distinct; ++c) start[c + 1] += start[c];
    cls_cols.resize(N);
    {
        std::vector<int32_t> fill(start.begin(), start.end() - 1);
        for (int32_t j = 0; j < N; ++j) cls_cols[fill[set_of[j]]++] = j;
    }
    int32_t largest = 0;
    for (int32_t c = 0; c < n_distinct; ++c) largest = std::max(largest, start[c + 1] - start[c]);
    if (largest <= max_members) {                   // (nothing to split)
        first_col.resize(n_distinct);
        for (int32_t c = 0; c < n_distinct; ++c) first_col[c] = cls_cols[start[c]];
        cls_ptr = std::move(start);
        col_cls = std::move(set_of);
        return;
    }
    cls_ptr.reserve(n_distinct + 64);
    first_col.reserve(n_distinct + 64);
    cls_ptr.assign(1, 0);
    first_col.clear();
    for (int32_t c = 0; c < n_distinct; ++c)
        for (int32_t k = start[c]; k < start[c + 1]; k += max_members) {
            cls_ptr.push_back(std::min(start[c + 1], k + max_members));
            first_col.push_back(cls_cols[start[c]]);
        }
}

// Levels (longest path from a root, in ops before it) and a topological order of a validated graph.  False: the graph has a
// cycle.  (A graph whose predecessors all have lower ids, as traced graphs have as a rule, has its ids for an order.)
static bool find_levels(int32_t n, const int32_t *row_ptr, const int32_t *col_idx, std::vector<int32_t> &level,
                        std::vector<int32_t> &order, int32_t &n_levels)
{
    level.assign(n, 0);
    order.clear();
    n_levels = 0;
    const int32_t E = row_ptr[n];
    std::vector<int32_t> sptr(n + 1, 0), sidx(E), waiting(n);
    for (int32_t e = 0; e < E; ++e) sptr[col_idx[e] + 1]++;
    for (int32_t v = 0; v < n; ++v) sptr[v + 1] += sptr[v];
    {
        std::vector<int32_t> fill(sptr.begin(), sptr.end() - 1);
        for (int32_t v = 0; v < n; ++v)
            for (int32_t e = row_ptr[v]; e < row_ptr[v + 1]; ++e) sidx[fill[col_idx[e]]++] = v;
    }
    order.reserve(n);
    for (int32_t v = 0; v < n; ++v) {
        waiting[v] = row_ptr[v + 1] - row_ptr[v];
        if (waiting[v] == 0) order.push_back(v);
    }
    for (size_t q = 0; q < order.size(); ++q) {
        const int32_t u = order[q];
        n_levels = std::max(n_levels, level[u] + 1);
        for (int32_t e = sptr[u]; e < sptr[u + 1]; ++e) {
            const int32_t v = sidx[e];
            level[v] = std::max(level[v], level[u] + 1);
            if (--waiting[v] == 0) order.push_back(v);
        }
    }
    return (int32_t)order.size() == n;
}

// Dependency rows of the compute ops as sets: of_op[v] the set of op v (-1 for a recv), sets numbered by their first
// member in ascending op id, rows [sets][W].  Formed on the host, set by set: an op whose predecessors are compute ops of
// one set, or whose predecessors' rows all lie within the largest of them, has that set; only the others form a union.
struct HostSets {
    std::vector<int32_t> of_op, count;
    std::vector<uint64_t> rows;
    int32_t n = 0;
};
static void host_sets(int32_t n, int32_t W, const int32_t *row_ptr, const int32_t *col_idx, const std::vector<int32_t> &recv_of_op,
                      const std::vector<int32_t> &order, HostSets &h)
{
    h.of_op.assign(n, -1);
    size_t cap = 1024;
    std::vector<int32_t> slot(cap, -1);
    std::vector<uint64_t> hash_of;
    std::vector<uint64_t> tmp(W);
    for (int32_t i = 0; i < n; ++i) {
        const int32_t v = order.empty() ? i : order[i];
        if (recv_of_op[v] >= 0) continue;
        const int32_t beg = row_ptr[v], end = row_ptr[v + 1];
        int32_t best = -1;
        bool mixed = false;
        for (int32_t e = beg; e < end; ++e) {
            const int32_t c = h.of_op[col_idx[e]];
            if (c < 0) { mixed = true; continue; }              // a recv
            if (best < 0) best = c;
            else if (c != best) {
                mixed = true;
                if (h.count[c] > h.count[best]) best = c;
            }
        }
        bool same = best >= 0;
        if (same && mixed) {
            const uint64_t *rb = &h.rows[(size_t)best * W];
            for (int32_t e = beg; e < end && same; ++e) {
                const int32_t u = col_idx[e], c = h.of_op[u];
                if (c == best) continue;
                if (c < 0) {
                    const int32_t r = recv_of_op[u];
                    same = (rb[r >> 6] >> (r & 63)) & 1ull;
                } else {
                    const uint64_t *rc = &h.rows[(size_t)c * W];
                    uint64_t more = 0;
                    for (int32_t w = 0; w < W; ++w) more |= rc[w] & ~rb[w];
                    same = more == 0;
                }
            }
        }
        if (same) { h.of_op[v] = best; continue; }
        std::fill(tmp.begin(), tmp.end(), 0);
        for (int32_t e = beg; e < end; ++e) {
            const int32_t u = col_idx[e], c = h.of_op[u];
            if (c < 0) tmp[recv_of_op[u] >> 6] |= 1ull << (recv_of_op[u] & 63);
            else for (int32_t w = 0; w < W; ++w) tmp[w] |= h.rows[(size_t)c * W + w];
        }
        uint64_t hash = 0x9E3779B97F4A7C15ull;
        int32_t bits = 0;
        for (int32_t w = 0; w < W; ++w) {
            hash += (tmp[w] ^ (tmp[w] >> 31)) * (0xFF51AFD7ED558CCDull + 2 * (uint64_t)w);
            hash ^= hash >> 29;
            bits += __builtin_popcountll(tmp[w]);
        }
        hash ^= hash >> 32;
        if ((size_t)h.n * 2 >= cap) {
            cap *= 4;
            slot.assign(cap, -1);
            for (int32_t c = 0; c < h.n; ++c) {
                size_t q = hash_of[c] & (cap - 1);
                while (slot[q] >= 0) q = (q + 1) & (cap - 1);
                slot[q] = c;
            }
        }
        size_t q = hash & (cap - 1);
        for (; slot[q] >= 0; q = (q + 1) & (cap - 1))
            if (hash_of[slot[q]] == hash && (W == 0 || memcmp(&h.rows[(size_t)slot[q] * W], tmp.data(), (size_t)W * 8) == 0)) break;
        if (slot[q] < 0) {
            slot[q] = h.n++;
            hash_of.push_back(hash);
            h.count.push_back(bits);
            h.rows.insert(h.rows.end(), tmp.begin(), tmp.end());
        }
        h.of_op[v] = slot[q];
    }
    if (order.empty()) return;
    // numbered by first member
    std::vector<int32_t> to(h.n, -1), count(h.n);
    std::vector<uint64_t> rows(h.rows.size());
    int32_t k = 0;
    for (int32_t v = 0; v < n; ++v) {
        int32_t &c = h.of_op[v];
        if (c < 0) continue;
        if (to[c] < 0) {
            to[c] = k;
            count[k] = h.count[c];
            std::copy(h.rows.begin() + (size_t)c * W, h.rows.begin() + (size_t)(c + 1) * W, rows.begin() + (size_t)k * W);
            ++k;
        }
        c = to[c];
    }
    h.count.swap(count);
    h.rows.swap(rows);
}

// The same classes from sets of ops.  cls_of_set: the first class of every set.
static void group_sets(const HostSets &h, const std::vector<int32_t> &recv_of_op, int32_t N, int32_t W, int32_t max_members,
                       std::vector<uint64_t> &cls_dep, std::vector<int32_t> &cls_ptr, std::vector<int32_t> &cls_cols,
                       int32_t &n_distinct, std::vector<int32_t> &cls_of_set)
{
    std::vector<int32_t> start(h.n + 1, 0);
    for (int32_t c : h.of_op)
        if (c >= 0) ++start[c + 1];
    for (int32_t c = 0; c < h.n; ++c) start[c + 1] += start[c];
    cls_cols.resize(N);
    {
        std::vector<int32_t> fill(start.begin(), start.end() - 1);
        int32_t j = 0;
        for (int32_t c : h.of_op)
            if (c >= 0) cls_cols[fill[c]++] = j++;
    }
    n_distinct = h.n;
    cls_of_set.resize(h.n);
    cls_ptr.reserve(h.n + 8);
    cls_dep.reserve(h.rows.size() + (size_t)8 * W);
    cls_ptr.assign(1, 0);
    for (int32_t c = 0; c < h.n; ++c) {
        cls_of_set[c] = (int32_t)cls_ptr.size() - 1;
        for (int32_t k = start[c]; k < start[c + 1]; k += max_members) {
            cls_ptr.push_back(std::min(start[c + 1], k + max_members));
            cls_dep.insert(cls_dep.end(), h.rows.begin() + (size_t)c * W, h.rows.begin() + (size_t)(c + 1) * W);
        }
    }
}

// ---- the tables of the propagation kernels (k1_propagate.hip) ----
// The condensed graph: a compute op whose predecessors come down to one node has that node's row; every other compute op is
// a node of its own.  Nodes k in topological order, their inputs in[ptr[k] .. ptr[k + 1]): ~i for recv i, else a node.
struct Condensed {
    std::vector<int32_t> val;               // of every op: ~i for recv i, else the node whose row it has
    std::vector<int32_t> op, ptr, in;
    std::vector<int32_t> lvl_ptr, lvl, pos; // positions by level: of each level, and level and position of every node
    int32_t M = 0, n_levels = 0, max_width = 0;
    size_t list_entries = 0;                // of the nodes with more than four nodes or two recvs among their inputs

    const int32_t *begin(int32_t k) const { return &in[0] + ptr[k]; }
    const int32_t *end(int32_t k) const { return &in[0] + ptr[k + 1]; }
};

// Whether a branch on the number of predecessors of an op would go either way: in a sample of 256 ops more than a quarter have
// another number than the op before, and there are two and more on average.  Then the passes over all ops do as if all had four
// (layered graphs with one to four each, every graph seen once: 100 000 ops, levels and condensation 1.44 -> 0.85 ms; a build of 1 800 ops
// 255 -> 232 us, of 960 155 -> 145).  Where the branch is foreseen they do what there is to do: 30 000 ops with three each 1.4 ms, 1.65 with
// four; inception3, chains of ops with 1.5 on average, 136 us, 157 with four; and of a graph of a few hundred ops that is built again and
// again the branches are remembered (700 ops 101 us, 103 with four, 152 and 147 once; 960 ops 92 either way).
static bool mixed_degrees(int32_t n, const int32_t *row_ptr)
{
    if (n < 800 || row_ptr[n] / 2 < n) return false;
    int32_t changes = 0;
    for (int32_t i = 1; i <= 256; ++i) {
        const int32_t v = 1 + (int32_t)((int64_t)i * (n - 2) / 256);
        changes += row_ptr[v + 1] - row_ptr[v] != row_ptr[v] - row_ptr[v - 1];
    }
    return changes > 64;
}

template <bool MIXED>
static void condense(const Dag &d, const int32_t *row_ptr, const int32_t *col_idx, const std::vector<int32_t> &recv_of_op,
                     const std::vector<int32_t> &level, const std::vector<int32_t> &order, Condensed &g)
{
    const int32_t n = d.n;
    g.val.resize(n);
    g.op.resize(n); g.ptr.resize(n + 1);
    g.in.resize((size_t)d.E + 1);           // (one more: begin() of an empty list)
    int32_t *in = g.in.data(), *val = g.val.data(), at = 0, M = 0;
    std::vector<int32_t> used(d.n_levels + 1, 0);
    for (int32_t i = 0; i < n; ++i) {
        const int32_t v = order.empty() ? i : order[i];
        if (recv_of_op[v] >= 0) { val[v] = ~recv_of_op[v]; continue; }
        const int32_t first = at, e0 = row_ptr[v], deg = row_ptr[v + 1] - e0;
        const int32_t *pred = col_idx + e0;
        // (few predecessors, as most ops have: each value is written and kept if it differs from those before, without a
        // branch that could go either way; where numbers of predecessors vary the last one stands in for those missing)
        if (MIXED && (uint32_t)(deg - 1) < 4u) {
            const int32_t x0 = val[pred[0]], x1 = val[pred[std::min(1, deg - 1)]], x2 = val[pred[std::min(2, deg - 1)]], x3 = val[pred[deg - 1]];
            const int32_t k1 = x1 != x0, k2 = (x2 != x0) & (x2 != x1), k3 = (x3 != x0) & (x3 != x1) & (x3 != x2);
            in[at] = x0;
            in[at += 1] = x1;
            in[at += k1] = x2;
            in[at += k2] = x3;
            at += k3;
            const int32_t nr = (x0 < 0) + ((x1 < 0) & k1) + ((x2 < 0) & k2) + ((x3 < 0) & k3);
            g.list_entries += nr > 2 ? 1 + (size_t)(at - first) : 0;
            const bool same = (at == first + 1) & (x0 >= 0);        // (the row of that node)
            val[v] = same ? x0 : M;
            at = same ? first : at;
            g.op[M] = v;
            g.ptr[M + 1] = at;
            used[level[v]] |= !same;
            M += !same;
            continue;
        }
        if (deg <= 4) {
            if (deg > 0) in[at++] = val[pred[0]];
            if (deg > 1) {
                const int32_t x = val[pred[1]];
                in[at] = x;
                at += x != in[first];
            }
            if (deg > 2) {
                const int32_t x = val[pred[2]];
                in[at] = x;
                at += (x != in[first]) & (x != in[at - 1]);
            }
            if (deg > 3) {
                const int32_t x = val[pred[3]], mid = std::min(first + 1, at - 1);
                in[at] = x;
                at += (x != in[first]) & (x != in[mid]) & (x != in[at - 1]);
            }
        } else if (deg <= 16) {
            for (int32_t e = 0; e < deg; ++e) {
                const int32_t x = val[pred[e]];
                bool seen = false;
                for (int32_t k = first; k < at; ++k) seen |= in[k] == x;
                if (!seen) in[at++] = x;
            }
        } else {
            for (int32_t e = 0; e < deg; ++e) in[at++] = val[pred[e]];
            std::sort(in + first, in + at);
            at = (int32_t)(std::unique(in + first, in + at) - in);
        }
        if (at == first + 1 && in[first] >= 0) {
            val[v] = in[first];
            at = first;
            continue;
        }
        if (at - first > 2) {
            int32_t nr = 0;
            for (int32_t k = first; k < at; ++k) nr += in[k] < 0;
            if (nr > 2 || at - first - nr > 4) g.list_entries += 1 + (size_t)(at - first);
        }
        val[v] = M;
        g.op[M++] = v;
        g.ptr[M] = at;
        used[level[v]] = 1;
    }
    g.M = M;
    // Nodes are grouped by the level of their op in the full graph (an input of a node lies on a
    // strictly lower level, and close to it, which keeps inputs inside the kernel's LDS ring);
    // levels without nodes are dropped.
    for (int32_t l = 0; l < d.n_levels; ++l) { const int32_t u = used[l]; used[l] = g.n_levels; g.n_levels += u; }
    g.lvl.resize(g.M);
    g.pos.resize(g.M);
    g.lvl_ptr.assign(g.n_levels + 1, 0);
    for (int32_t k = 0; k < g.M; ++k) ++g.lvl_ptr[(g.lvl[k] = used[level[g.op[k]]]) + 1];
    for (int32_t l = 0; l < g.n_levels; ++l) {
        g.max_width = std::max(g.max_width, g.lvl_ptr[l + 1]);
        g.lvl_ptr[l + 1] += g.lvl_ptr[l];
    }
    std::vector<int32_t> fill(g.lvl_ptr.begin(), g.lvl_ptr.end() - 1);
    for (int32_t k = 0; k < g.M; ++k) g.pos[k] = fill[g.lvl[k]]++;
}

// The ops whose rows are copies (of a recv's single bit, or of the row of the node the op collapses onto).
template <bool MIXED>
static std::vector<int32_t> copied_rows(const Condensed &g)
{
    const int32_t n = (int32_t)g.val.size();
    std::vector<int32_t> copied(2 * (size_t)(n - g.M) + 2);         // (two more: MIXED writes every op, a node's is written over)
    size_t at = 0;
    for (int32_t v = 0; v < n; ++v) {
        const int32_t x = g.val[v], from = x < 0 ? x : g.op[x];
        if (MIXED || from != v) {
            copied[at] = v;
            copied[at + 1] = from;
            at += from != v ? 2 : 0;
        }
    }
    copied.resize(at);
    return copied;
}

// The level-major records of the kernel with 64-byte slices (see internal.h).  With such slices the ring holds few levels,
// and a row that a later level needs is handed on by copy nodes (op = -2: one input, the row goes to the ring only) in free
// slots of the levels between, each within reach of the one before; the copies of a row form one chain, which the
// consumers, taken level by level, extend.
struct QuadTables {
    std::vector<Dag::QuadRec> qrecs;
    std::vector<int32_t> lists, left;       // inputs of the nodes that fit no record; copied rows that found no slot
    int32_t far = 0;                        // inputs on the lists that have left the ring
};
static QuadTables make_quad_tables(const Condensed &g, const std::vector<int32_t> &copied, int32_t P, int32_t ring)
{
    const int32_t M = g.M, n_node_levels = g.n_levels;
    QuadTables out;
    std::vector<int32_t> &lists = out.lists, &left = out.left;
    std::vector<int32_t> slot_of(M), node_at(M);     // of a node; the nodes by position
    for (int32_t k = 0; k < M; ++k) {
        slot_of[k] = g.lvl[k] * P + (g.pos[k] - g.lvl_ptr[g.lvl[k]]);
        node_at[g.pos[k]] = k;
    }
    const uint32_t none = (uint32_t)ring, zero2 = none | none << 16;
    std::vector<Dag::QuadRec> &qrecs = out.qrecs;
    qrecs.assign((size_t)n_node_levels * P, Dag::QuadRec{zero2, zero2, 0xffffffffu, -1});
    const int32_t reach = ring / P - 1;        // a row of level x is in the ring up to level x + reach
    std::vector<int32_t> used(n_node_levels);
    for (int32_t l = 0; l < n_node_levels; ++l) used[l] = g.lvl_ptr[l + 1] - g.lvl_ptr[l];
    // the copies of node k's row, from the first to the last: copy q at level copy_lvl[q], followed by copy_next[q]
    std::vector<int32_t> first_copy(M, -1), last_copy(M, -1), copy_slot, copy_lvl, copy_next;
    auto within_reach = [&](int32_t k, int32_t l) -> int32_t {      // the slot to read the row of node k from at level l, or -1
        if (g.lvl[k] + reach >= l || slot_of[k] >= (l + 1) * P - ring) return slot_of[k];
        if (reach < 1 || l - g.lvl[k] > 8 * reach) return -1;
        int32_t q = last_copy[k], cur = q < 0 ? slot_of[k] : copy_slot[q], at = q < 0 ? g.lvl[k] : copy_lvl[q];
        while (l - at > reach) {
            int32_t t = at + reach;
            while (t > at && used[t] >= P) --t;
            if (t == at) return -1;
            const int32_t c = t * P + used[t]++;
            qrecs[c].in01 = (uint32_t)(cur & (ring - 1)) | none << 16;
            qrecs[c].op = -2;
            const int32_t made = (int32_t)copy_slot.size();
            copy_slot.push_back(c); copy_lvl.push_back(t); copy_next.push_back(-1);
            (q < 0 ? first_copy[k] : copy_next[q]) = made;
            q = last_copy[k] = made;
            cur = c;
            at = t;
        }
        return cur;
    };
    for (int32_t p = 0; p < M; ++p) {
        const int32_t k = node_at[p], l = g.lvl[k];
        Dag::QuadRec &f = qrecs[slot_of[k]];
        f.op = g.op[k];
        // (most nodes: one to four inputs, no recv, all in the ring; the last input again in place of those that are missing)
        if (const int32_t n_in = g.ptr[k + 1] - g.ptr[k]; (uint32_t)(n_in - 1) < 4u) {
            const int32_t *x = g.begin(k), x0 = x[0], x1 = x[std::min(1, n_in - 1)], x2 = x[std::min(2, n_in - 1)], x3 = x[n_in - 1];
            if ((x0 | x1 | x2 | x3) >= 0) {
                const int32_t s0 = slot_of[x0], s1 = slot_of[x1], s2 = slot_of[x2], s3 = slot_of[x3];
                if (std::min(std::min(s0, s1), std::min(s2, s3)) >= (l + 1) * P - ring) {
                    const int32_t m = ring - 1;
                    f.in01 = (uint32_t)(s0 & m) | (n_in > 1 ? (uint32_t)(s1 & m) : none) << 16;
                    f.in23 = (n_in > 2 ? (uint32_t)(s2 & m) : none) | (n_in > 3 ? (uint32_t)(s3 & m) : none) << 16;
                    continue;
                }
            }
        }
        int nn = 0, nr = 0;
        for (const int32_t *x = g.begin(k); x != g.end(k); ++x) (*x < 0 ? nr : nn) += 1;
        // (copies are made only for a node that then fits a record)
        bool resident = nn <= 4 && nr <= 2;
        uint32_t in[4] = {none, none, none, none}, rc[2] = {0xffffu, 0xffffu};
        int a = 0, b = 0;
        if (resident)
            for (const int32_t *x = g.begin(k); x != g.end(k); ++x) {
                if (*x < 0) { rc[b++] = (uint32_t)~*x; continue; }
                const int32_t c = within_reach(*x, l);
                if (c < 0) { resident = false; break; }
                in[a++] = (uint32_t)(c & (ring - 1));
            }
        if (resident) {
            f.in01 = in[0] | in[1] << 16;
            f.in23 = in[2] | in[3] << 16;
            f.rcv01 = rc[0] | rc[1] << 16;
            continue;
        }
        f.in01 = 0xffffffffu;
        f.in23 = (uint32_t)lists.size();
        lists.push_back(nn + nr);
        for (const int32_t *x = g.begin(k); x != g.end(k); ++x) {
            lists.push_back(*x < 0 ? *x : slot_of[*x]);
            out.far += *x >= 0 && slot_of[*x] < (l + 1) * P - ring;
        }
    }
    // The copied rows ride along in slots that are still free: a recv's row anywhere (no input, one recv
    // bit), the copy of a node's row at a level within reach of the node or of one of its copy nodes, as
    // a node with that one input and the op's own id.  What finds no slot stays on the list `left`.
    int32_t cursor = 0;
    for (size_t e = 0; e + 1 < copied.size(); e += 2) {
        const int32_t v = copied[e], sv = copied[e + 1];
        int32_t c = -1;
        if (sv < 0) {
            while (cursor < n_node_levels && used[cursor] >= P) ++cursor;
            if (cursor < n_node_levels) {
                c = cursor * P + used[cursor]++;
                qrecs[c] = Dag::QuadRec{zero2, zero2, (uint32_t)~sv | 0xffff0000u, v};
            }
        } else if (reach >= 1) {
            const int32_t k = g.val[sv];
            int32_t from = slot_of[k], at = g.lvl[k], q = first_copy[k];
            for (;;) {
                const int32_t end = std::min(at + reach + 1, n_node_levels);
                int32_t t = at + 1;
                while (t < end && used[t] >= P) ++t;
                if (t < end) {
                    c = t * P + used[t]++;
                    qrecs[c] = Dag::QuadRec{(uint32_t)(from & (ring - 1)) | none << 16, zero2, 0xffffffffu, v};
                }
                if (c >= 0 || q < 0) break;
                from = copy_slot[q]; at = copy_lvl[q]; q = copy_next[q];
            }
        }
        if (c < 0) { left.push_back(v); left.push_back(sv); }
    }
    return out;
}

// The tables of the propagation kernels on the host, and where they go on the device.
struct PropTables {
    Condensed g;
    std::vector<int32_t> copied;
    std::vector<Dag::NodeRec> nodes;
    std::vector<Dag::FastRec> lrecs, frecs;
    std::vector<int32_t> ovf_idx, chunk_end, lfovf, fovf;
    std::vector<int32_t> slot;              // level-major records: the slot of every node
    QuadTables quads;
    std::future<void> quads_made;           // (waited for before the rest goes: a thread of their own makes them)

    void add_to(Packer &p, Dag *d)
    {
        p.add(&d->d_frecs, frecs);
        p.add(&d->d_fovf, fovf);
        d->fovf_len = (int32_t)fovf.size();
        if (d->k1_lring == 0) {
            // the kernels that go by positions; the one for wide levels reads NodeRecs
            p.add(&d->d_nodes, nodes);
            p.add(&d->d_ovf_idx, ovf_idx);
            p.add(&d->d_nlvl_ptr, g.lvl_ptr);
            p.add(&d->d_chunk_end, chunk_end);
        } else {
            if (lrecs.empty()) {            // (launch_level_records makes them)
                p.add(&d->d_nlvl_ptr, g.lvl_ptr);
                p.add(&d->d_node_ptr, g.ptr.data(), (size_t)g.M + 1);
                p.add(&d->d_node_in, g.in.data(), (size_t)g.ptr[g.M]);
                p.add(&d->d_node_op, g.op.data(), (size_t)g.M);
                p.add(&d->d_node_slot, slot);
                // (a level's records, 8 KB for 256 slots, on as few pages as there are: 500 x 200 layered ops, 1 300 recvs 146 us;
                // 154 at a multiple of 4 KB or less)
                p.reserve(&d->d_lrecs, (size_t)d->n_node_levels * (d->k1_threads / d->k1_wc) * sizeof(Dag::FastRec), 65536);
                p.reserve(&d->d_lfovf, (size_t)d->lfovf_room * 4);
                p.reserve(&d->d_lfovf_used, ((size_t)g.M + 127) / 64 * 4);
            } else {
                p.add(&d->d_lrecs, lrecs);
                p.add(&d->d_lfovf, lfovf);
            }
            p.reserve(&d->d_k1_sink, (size_t)((d->W + d->k1_wc - 1) / d->k1_wc) * d->k1_threads * 8);
        }
        p.add(&d->d_copied, copied);
    }
    void add_quads_to(Packer &p, Dag *d)
    {
        if (!quads_made.valid()) return;
        quads_made.get();
        p.add(&d->d_qrecs, quads.qrecs);
        p.add(&d->d_qfovf, quads.lists);
        p.add(&d->d_q_copied, quads.left);
        d->qfovf_len = (int32_t)quads.lists.size();
        d->q_far = quads.far;
        d->n_q_copied = (int32_t)(quads.left.size() / 2);
        p.reserve(&d->d_k1_q_sink, (size_t)(d->W / 8) * d->k1_q_threads * 16);
    }
};

// Makes them.  order: the ops in topological order (empty: by id); level: longest path from a root.  The tables for several
// graphs are made by a thread of their own meanwhile.  by_kernel: the level-major records are left to
// launch_level_records, which pays for graphs whose rows the device forms (on smaller ones the launch and the wait for it cost 3
// to 50 us more than the records).
static void make_propagate_tables(Dag *d, const int32_t *row_ptr, const int32_t *col_idx, const std::vector<int32_t> &recv_of_op,
                                  const std::vector<int32_t> &level, const std::vector<int32_t> &order, const bool by_kernel, PropTables &t)
{
    Condensed &g = t.g;
    const bool mixed = mixed_degrees(d->n, row_ptr);
    (mixed ? condense<true> : condense<false>)(*d, row_ptr, col_idx, recv_of_op, level, order, g);
    const int32_t M = g.M, n_node_levels = g.n_levels, max_width = g.max_width;
    const std::vector<int32_t> &nlvl_ptr = g.lvl_ptr;
    d->M = M; d->n_node_levels = n_node_levels;
    t.copied = (mixed ? copied_rows<true> : copied_rows<false>)(g);
    d->n_copied = (int32_t)(t.copied.size() / 2);
    // words per workgroup slice, threads, and the chunks of levels of the node kernel
    // a workgroup's LDS traffic per level grows with its slice, so wide bitsets get many narrow slices
    d->k1_wc = d->W <= 1 ? 1 : (d->W <= 2 ? 2 : (d->W >= 16 ? 1 : 4));
    // Graphs with narrow levels take a level per LDS round trip when one wave holds every row of its slice,
    // every record and the input lists of the nodes that fit no record in LDS (propagate_nodes_wave); the
    // slice is narrowed until that fits.
    const size_t list_entries = g.list_entries;
    d->k1_wave = false;
    for (int wc = d->k1_wc; wc >= 1 && max_width <= 64 && list_entries <= 4096 && M > 0; wc >>= 1) {
        if (max_width * wc <= 64 &&
            ((size_t)(M + 2) * wc + 1) * 8 + (size_t)M * 32 + (size_t)(n_node_levels + 1) * 4 + list_entries * 4 <= 150 * 1024) {
            d->k1_wc = wc;
            d->k1_wave = true;
            break;
        }
    }
    int threads = max_width * d->k1_wc;
    threads = threads < 64 ? 64 : (threads > 1024 ? 1024 : (threads + 63) / 64 * 64);
    d->k1_threads = threads;
    const int32_t per_pass = threads / d->k1_wc;
    t.chunk_end.assign(n_node_levels, 0);
    for (int32_t l0 = 0; l0 < n_node_levels;) {
        int32_t l1 = l0 + 1;
        while (l1 < n_node_levels && l1 - l0 < 64 && nlvl_ptr[l1 + 1] - nlvl_ptr[l0] <= 4 * per_pass) ++l1;
        t.chunk_end[l0] = l1;
        l0 = l1;
    }
    // the LDS ring: a power of two of positions, at least two chunks (or all nodes), at most 64 KB beyond that
    int32_t ring = 64;
    while (ring < M && (ring < 2 * kK1Rpt * per_pass || (size_t)ring * 2 * d->k1_wc * 8 <= 64 * 1024)) ring *= 2;
    if (d->k1_wave) ring = M;                   // every row stays: no ring, positions are used as they are
    d->k1_ring = ring;
    // level-major records (see internal.h): when a workgroup has more than one wave, the padding at
    // most quadruples the records, and sixteen levels of slots fit the ring: at most 64 KB, and 32 KB for
    // one-word slices (many narrow workgroups: four of them then share a compute unit when several
    // graphs are propagated by one launch)
    int32_t lring = 0;
    if (max_width <= per_pass && threads > 64 && (int64_t)n_node_levels * per_pass <= (int64_t)4 * M + 8192 &&
        (int64_t)M + g.ptr[M] <= INT32_MAX) {
        const size_t ring_cap = d->k1_wc == 1 ? 32 * 1024 : 64 * 1024;
        lring = 64;
        while ((size_t)lring * 2 * d->k1_wc * 8 <= ring_cap && lring < n_node_levels * per_pass) lring *= 2;
        if (lring < 16 * per_pass && lring < n_node_levels * per_pass) lring = 0;
    }
    d->k1_lring = lring;
    // (the records of the chunked kernel take 256 bytes per node of a pass: beside the ring there is no room for those of levels
    // of more than 256 nodes with one-word slices, 288 with two-word slices)
    d->k1_wide = max_width > per_pass || (lring == 0 && !d->k1_wave && k1_nodes_lds(ring, d->k1_wc, per_pass) > kK1LdsMax);
    // Rows of a multiple of eight words, levels of at most 256 nodes: the kernel with 64-byte slices (four lanes per
    // slot, or two with 32-byte slices; P slots per level, a multiple of 32 so that the slots of a wave are whole; 2048
    // slots in the ring), which the propagation of several graphs by one launch takes (make_quad_tables).
    int32_t q_slots = (max_width + 31) / 32 * 32, q_ring = 0;
    if (q_slots < 32) q_slots = 32;
    if (d->k1_wc == 1 && d->W % 8 == 0 && d->W <= 1016 && max_width <= 256 && M > 0 &&
        (int64_t)n_node_levels * q_slots <= (int64_t)4 * M + 8192) {
        q_ring = 2048;
        while (q_ring > 64 && q_ring / 2 >= n_node_levels * q_slots) q_ring /= 2;
        // (eight levels: a list reads a row that has left the ring from memory, and stores are waited for seven levels on)
        if (q_ring < 8 * q_slots && q_ring < n_node_levels * q_slots) q_ring = 0;
    }
    d->k1_q_ring = q_ring;
    d->k1_q_threads = q_ring > 0 ? 4 * q_slots : 0;
    if (q_ring > 0) t.quads_made = std::async([&t, q_slots, q_ring] { t.quads = make_quad_tables(t.g, t.copied, q_slots, q_ring); });

    // FastRec of node k at level l: place(x) the byte offset of input node x in the ring, or -1 when it has left it
    auto fast = [&](Dag::FastRec &f, int32_t k, int32_t zero_row, std::vector<int32_t> &lists, auto &&place, auto &&name) {
        for (int j = 0; j < 4; ++j) f.in[j] = zero_row;
        f.rcv[0] = f.rcv[1] = -1;
        f.op = g.op[k];
        f.ovf = -1;
        int a = 0, b = 0;
        bool fits = true;
        for (const int32_t *x = g.begin(k); x != g.end(k) && fits; ++x) {
            if (*x < 0) {
                if ((fits = b < 2)) f.rcv[b++] = ~*x;
            } else {
                const int32_t q = a < 4 ? place(*x) : -1;
                if ((fits = q >= 0)) f.in[a++] = q;
            }
        }
        if (fits) return;
        for (int j = 0; j < 4; ++j) f.in[j] = zero_row;
        f.rcv[0] = f.rcv[1] = -1;
        f.ovf = (int32_t)lists.size();
        lists.push_back((int32_t)(g.end(k) - g.begin(k)));
        for (const int32_t *x = g.begin(k); x != g.end(k); ++x) lists.push_back(*x < 0 ? *x : name(*x));
    };
    if (lring > 0) {
        const int32_t P = per_pass;
        t.slot.resize(M);
        for (int32_t k = 0; k < M; ++k) t.slot[k] = g.lvl[k] * P + (g.pos[k] - nlvl_ptr[g.lvl[k]]);
        if (by_kernel) {
            d->lfovf_room = M + g.ptr[M];
        } else {
            // While level l is computed the ring holds the slots from (l + 1) * P - ring on.
            const int32_t row_bytes = d->k1_wc * 8, zero_row = lring * row_bytes;
            t.lrecs.assign((size_t)n_node_levels * P, Dag::FastRec{{zero_row, zero_row, zero_row, zero_row}, {-1, -1}, -1, -1});
            for (int32_t k = 0; k < M; ++k) {
                const int32_t oldest = (g.lvl[k] + 1) * P - lring;
                fast(t.lrecs[t.slot[k]], k, zero_row, t.lfovf,
                     [&](int32_t x) { return t.slot[x] >= oldest ? (t.slot[x] & (lring - 1)) * row_bytes : -1; },
                     [&](int32_t x) { return t.slot[x]; });
            }
            d->lfovf_len = (int32_t)t.lfovf.size();
        }
    } else if (!d->k1_wide) {
        const int32_t row_bytes = d->k1_wc * 8, zero_row = ring * row_bytes;
        t.frecs.resize(M);
        for (int32_t k = 0; k < M; ++k) {
            const int32_t oldest = nlvl_ptr[g.lvl[k] + 1] - ring;
            fast(t.frecs[g.pos[k]], k, zero_row, t.fovf,
                 [&](int32_t x) { const int32_t q = g.pos[x]; return q >= oldest ? (d->k1_wave ? q : (q & (ring - 1))) * row_bytes : -1; },
                 [&](int32_t x) { return g.pos[x]; });
        }
    } else {
        t.nodes.resize(M);
        for (int32_t k = 0; k < M; ++k) {
            Dag::NodeRec &r = t.nodes[g.pos[k]];
            r.op = g.op[k];
            r.ovf_beg = -1;
            for (int j = 0; j < 6; ++j) r.in[j] = INT32_MIN;
            int j = 0;
            for (const int32_t *x = g.begin(k); x != g.end(k); ++x, ++j) {
                const int32_t y = *x < 0 ? *x : g.pos[*x];
                if (j < 6) { r.in[j] = y; continue; }
                if (r.ovf_beg < 0) { r.ovf_beg = (int32_t)t.ovf_idx.size(); t.ovf_idx.push_back(0); }
                t.ovf_idx.push_back(y);
                t.ovf_idx[r.ovf_beg]++;
            }
        }
    }
}

// The line between the rows formed on the host and by the kernels: on layered graphs of 11 000 ops and 16 words (0.6 million
// words) the host part of a build takes 2.1 ms one way and 3.7 ms the other, at 21 000 ops (1.2 million) 3.7 and 6.8, at 22 000
// ops of 32 words (2.6 million) 12.2 and 11.3, without the kernels' own time.
constexpr int64_t kHostRowWords = (int64_t)1 << 21;
// From so many ops and predecessors on, the tables of the propagation kernels are made by a thread of their own while the
// rows and classes are formed.  Starting it costs what it saves on small graphs (a build of inception3, 15 984, takes 136 us
// without it and 175 with it; 7 061 ops with 17 300 predecessors 281 and 130, 10 512 with 26 900 661 and 643).  The tables are
// a tenth of a small graph's build (resnet50 41 us, 37 without them) and up to two fifths where sets and classes are quick
// to form (3 236 ops, 8 122 predecessors, two words: 163 us, 93 without), and are made nevertheless: a first
// tictac_dag_recompute_deps would otherwise make them, wait for the stream twice and take 1.1 ms instead of 0.1 at 20 512
// ops, a first batch of 32 such handles 31 ms instead of 2.8.
constexpr int64_t kPropThread = 16384;

// Checks the predecessors; levels, as long as every predecessor has a lower id (topological).
template <bool MIXED>
static int levels_by_id(int32_t n, const int32_t *row_ptr, const int32_t *col_idx, std::vector<int32_t> &level, int32_t &n_levels,
                        bool &topological)
{
    for (int32_t v = 0; v < n; ++v) {
        int32_t l = 0, e0 = row_ptr[v];
        const int32_t e1 = row_ptr[v + 1];
        // (one to four predecessors, as most ops have: the last one again in place of those that are missing, so that no
        // branch depends on how many there are)
        if (MIXED && (uint32_t)(e1 - e0 - 1) < 4u) {
            const int32_t a = col_idx[e0], b = col_idx[std::min(e0 + 1, e1 - 1)], c = col_idx[std::min(e0 + 2, e1 - 1)], f = col_idx[e1 - 1];
            const uint32_t most = std::max(std::max((uint32_t)a, (uint32_t)b), std::max((uint32_t)c, (uint32_t)f));
            if (most < (uint32_t)n) {
                topological &= most < (uint32_t)v;
                l = std::max(std::max(level[a], level[b]), std::max(level[c], level[f])) + 1;
                e0 = e1;
            }
        }
        for (int32_t e = e0; e < e1; ++e) {
            const int32_t u = col_idx[e];
            if (u < 0 || u >= n) { set_error("pred_col_idx[%d]=%d out of range", e, u); return TICTAC_ERR_BAD_CSR; }
            topological &= u < v;
            l = std::max(l, level[u] + 1);
        }
        level[v] = l;
        n_levels = std::max(n_levels, l + 1);
    }
    return TICTAC_OK;
}

static int build(int32_t n, const int32_t *row_ptr, const int32_t *col_idx, int32_t R, const int32_t *recv_ids,
                 hipStream_t s, Dag *d)
{
    // ---- validation (host) ----
    if (n < 0 || R < 0 || R > n) { set_error("bad sizes: n_ops=%d n_recv=%d", n, R); return TICTAC_ERR_BAD_CSR; }
    if (!row_ptr) { set_error("pred_row_ptr is NULL"); return TICTAC_ERR_NULL; }
    if (R > 0 && !recv_ids) { set_error("recv_ids is NULL"); return TICTAC_ERR_NULL; }
    if (row_ptr[0] != 0) { set_error("pred_row_ptr[0] != 0"); return TICTAC_ERR_BAD_CSR; }
    for (int32_t v = 0; v < n; ++v)
        if (row_ptr[v + 1] < row_ptr[v]) { set_error("pred_row_ptr decreases at op %d", v); return TICTAC_ERR_BAD_CSR; }
    const int32_t E = row_ptr[n];
    if (E > 0 && !col_idx) { set_error("pred_col_idx is NULL"); return TICTAC_ERR_NULL; }
    // (levels along the way, as long as every predecessor has a lower id)
    bool topological = true;
    std::vector<int32_t> level(n, 0);
    int32_t n_levels = 0;
    const int status = (mixed_degrees(n, row_ptr) ? levels_by_id<true> : levels_by_id<false>)(n, row_ptr, col_idx, level, n_levels, topological);
    if (status != TICTAC_OK) return status;
    std::vector<int32_t> recv_of_op(n, -1);
    for (int32_t i = 0; i < R; ++i) {
        int32_t v = recv_ids[i];
        if (v < 0 || v >= n) { set_error("recv_ids[%d]=%d out of range", i, v); return TICTAC_ERR_BAD_CSR; }
        if (recv_of_op[v] >= 0) { set_error("op %d listed twice in recv_ids", v); return TICTAC_ERR_DUP_RECV; }
        recv_of_op[v] = i;
    }
    for (int32_t i = 0; i < R; ++i) {
        int32_t v = recv_ids[i];
        if (row_ptr[v + 1] != row_ptr[v]) { set_error("recv %d (op %d) has predecessors", i, v); return TICTAC_ERR_RECV_NOT_ROOT; }
    }
    d->n = n; d->R = R; d->W = (R + 63) / 64; d->N = n - R; d->E = E;
    // Small graphs (few words in the rows of all ops and predecessors) need no trip to the device and back before their ops
    // can be grouped: the rows are formed here, and the device gets op.dep from those of the sets.  Larger graphs are
    // propagated by the kernels of k1_propagate.hip.
    const bool on_host = ((int64_t)n + E) * std::max(d->W, 1) <= kHostRowWords && !getenv("TICTAC_GROUP_ON_HOST");
    std::vector<int32_t> order;
    if (topological) {
        d->n_levels = n_levels;
    } else if (!find_levels(n, row_ptr, col_idx, level, order, d->n_levels)) {
        set_error("the graph has a cycle");
        return TICTAC_ERR_CYCLE;
    }
    d->h_row_ptr.assign(row_ptr, row_ptr + n + 1);
    d->h_col_idx.assign(col_idx, col_idx + E);
    d->h_recv_ids.assign(recv_ids, recv_ids + R);
    HIP_TRY(hipGetDevice(&d->device));

    HostSets sets;
    PropTables prop;
    std::future<void> prop_made;            // (after what its thread works on: it ends first)
    if ((size_t)n * d->W) {
        auto make = [&] { make_propagate_tables(d, row_ptr, col_idx, recv_of_op, level, order, !on_host, prop); };
        if (on_host && (int64_t)n + E > kPropThread) prop_made = std::async(make);
        else make();
    }
    std::vector<int32_t> op_of_col;
    if (on_host) {
        host_sets(n, d->W, row_ptr, col_idx, recv_of_op, order, sets);
    } else {
        const std::vector<int32_t> zeros(64, 0);
        Packer graph;
        prop.add_to(graph, d);
        graph.add(&d->d_recv_of_op, recv_of_op);
        op_of_col.resize((size_t)d->N + 1);
        for (int32_t v = 0, j = 0; v < n; ++v) {
            op_of_col[j] = v;
            j += recv_of_op[v] < 0;
        }
        op_of_col.pop_back();
        graph.add(&d->d_op_of_col, op_of_col);
        graph.add(&d->d_bad_order, zeros);
        graph.reserve(&d->d_dep, (size_t)n * d->W * 8);
        HIP_TRY(graph.commit(d->graph_block, d->device, s));
        HIP_TRY(launch_level_records(*d, s));
        // (how many entries the lists have: the wait is for this as well)
        if (d->d_lfovf_used)
            HIP_TRY(hipMemcpyAsync(&d->lfovf_len, d->d_lfovf_used, sizeof(int32_t), hipMemcpyDeviceToHost, s));
        HIP_TRY(graph.finish());
        if ((size_t)n * d->W) HIP_TRY(launch_propagate(*d, s));
    }
    const size_t dep_words = (size_t)n * d->W;

    // ---- classes of identical rows among the compute ops (a lambda: done again on the host when the device's
    // grouping cannot be used; returns a status, or 1 for "again, from the rows") ----
    auto classes = [&](const bool on_device) -> int {
    const bool from_sets = on_host;
    // Large graphs (8 MB of rows or more) are grouped without bringing the rows to the host: the device hashes
    // every row (128 bits, with the number of set bits and the lowest one) and finds the ops of equal hashes through a
    // table, the host numbers the sets, and the device forms the class rows and checks every op's row against its class (on a mismatch, which two
    // different rows with one hash would cause, everything below is done again from the rows themselves).
    std::vector<uint64_t> rows, cls_dep, depT;
    std::vector<int32_t> cls_ptr, cls_cols, cnt0, first_op, lowest, cls_of_set, op_src, col_cls;
    const std::vector<int32_t> zeros(64, 0);
    // only classes far larger than a lane's fair share of the ops are split
    const int32_t max_members = std::min(256, std::max(16, (d->N + 63) / 64));
    if (on_device) {
        HIP_TRY(ensure_workspace(d, group_workspace_bytes(d->N)));
        HIP_TRY(launch_group_rows(*d, d->d_op_of_col, d->d_work, s));
        std::vector<int32_t> pageable;
        Stage staging;
        int32_t *rep = static_cast<int32_t *>(staging.take((size_t)d->N * 12));
        if (!rep) {
            pageable.resize((size_t)d->N * 3);
            rep = pageable.data();
        }
        HIP_TRY(hipMemcpyAsync(rep, d->d_work, (size_t)d->N * 12, hipMemcpyDeviceToHost, s));
        HIP_TRY(hipStreamSynchronize(s));
        std::vector<int32_t> first_col;
        group_reps(rep, d->N, max_members, cls_ptr, cls_cols, first_col, col_cls, d->C_distinct);
        d->C = (int32_t)cls_ptr.size() - 1;
        d->Cpad = (d->C + 63) / 64 * 64;
        if (d->R <= 1024 && d->C <= 1024) return 1;      // the small-graph kernels want tables made from the rows
        cnt0.resize(d->C); first_op.resize(d->C); lowest.resize(d->C);
        for (int32_t c = 0; c < d->C; ++c) {
            cnt0[c] = rep[(size_t)d->N + first_col[c]];
            lowest[c] = rep[(size_t)2 * d->N + first_col[c]];
            first_op[c] = op_of_col[first_col[c]];
        }
    } else if (!from_sets) {
        rows.resize((size_t)d->N * d->W);
        if (!rows.empty()) {
            std::vector<uint64_t> pageable;
            Stage staging;
            uint64_t *all = static_cast<uint64_t *>(staging.take(dep_words * 8));
            if (!all) {
                pageable.resize(dep_words);
                all = pageable.data();
            }
            HIP_TRY(hipMemcpyAsync(all, d->d_dep, dep_words * 8, hipMemcpyDeviceToHost, s));
            HIP_TRY(hipStreamSynchronize(s));
            for (int32_t v = 0, j = 0; v < n; ++v)
                if (recv_of_op[v] < 0) memcpy(&rows[(size_t)j++ * d->W], &all[(size_t)v * d->W], (size_t)d->W * 8);
        }
        group_classes(rows, d->N, d->W, max_members, cls_dep, cls_ptr, cls_cols, d->C_distinct);
    } else {
        group_sets(sets, recv_of_op, d->N, d->W, max_members, cls_dep, cls_ptr, cls_cols, d->C_distinct, cls_of_set);
    }
    if (!on_device) {
        d->C = (int32_t)cls_ptr.size() - 1;
        d->Cpad = (d->C + 63) / 64 * 64;
        cnt0.assign(d->C, 0);
        depT.assign((size_t)d->W * d->Cpad, 0);
        // (the transpose in blocks of 16 classes: the block of rows stays in cache and every word row
        // of depT receives 128 consecutive bytes at a time)
        for (int32_t c0 = 0; c0 < d->C; c0 += 16) {
            const int32_t c1 = std::min(d->C, c0 + 16);
            for (int32_t w = 0; w < d->W; ++w) {
                uint64_t *dst = &depT[(size_t)w * d->Cpad];
                for (int32_t c = c0; c < c1; ++c) {
                    const uint64_t x = cls_dep[(size_t)c * d->W + w];
                    cnt0[c] += __builtin_popcountll(x);
                    dst[c] = x;
                }
            }
        }
    }
    d->cls_nnz = 0;
    for (int32_t c = 0; c < d->C; ++c) d->cls_nnz += cnt0[c];
    // runs [lo, hi) of consecutive recv indices of every class row, and the sum of its indices
    // (only the kernels for graphs with at most 1 024 recvs and 512 classes use the runs, with up to 1 024 classes the sums)
    const bool want_runs = !on_device && d->R <= 1024 && d->C <= 512;
    const bool want_isum = !on_device && d->R <= 1024 && d->C <= 1024;
    std::vector<int32_t> run_ptr, run_lo, run_hi, isum;
    if (want_runs) {
        run_ptr.assign(1, 0);
        isum.assign(d->C, 0);
    }
    if (want_isum && !want_runs) {
        isum.assign(d->C, 0);
        for (int32_t c = 0; c < d->C; ++c)
            for (int32_t w = 0; w < d->W; ++w)
                for (uint64_t x = cls_dep[(size_t)c * d->W + w]; x; x &= x - 1) isum[c] += w * 64 + __builtin_ctzll(x);
    }
    for (int32_t c = 0; want_runs && c < d->C; ++c) {
        const uint64_t *row = &cls_dep[(size_t)c * d->W];
        int32_t i = 0;
        int64_t sum = 0;
        while (i < d->R) {
            // next set bit at or after i
            int32_t w = i >> 6;
            uint64_t x = row[w] & (~0ull << (i & 63));
            while (!x && ++w < d->W) x = row[w];
            if (!x) break;
            const int32_t lo = w * 64 + __builtin_ctzll(x);
            // next clear bit after lo
            w = lo >> 6;
            uint64_t y = ~row[w] & (~0ull << (lo & 63));
            while (!y && ++w < d->W) y = ~row[w];
            const int32_t hi = y ? std::min(d->R, w * 64 + __builtin_ctzll(y)) : d->R;
            run_lo.push_back(lo);
            run_hi.push_back(hi);
            sum += (int64_t)(lo + hi - 1) * (hi - lo) / 2;
            i = hi;
        }
        run_ptr.push_back((int32_t)run_lo.size());
        isum[c] = (int32_t)sum;
    }
    Packer cls;
    cls.add(&d->d_cls_isum, isum);      // index sums stay below 2^20
    d->max_members = 0;
    for (int32_t c = 0; c < d->C; ++c) d->max_members = std::max(d->max_members, cls_ptr[c + 1] - cls_ptr[c]);
    d->n_runs = (int32_t)run_lo.size();
    cls.add(&d->d_run_ptr, run_ptr);
    cls.add(&d->d_run_lo, run_lo);
    cls.add(&d->d_run_hi, run_hi);
    if (!on_device) {
        cls.add(&d->d_cls_dep, cls_dep);
        cls.add(&d->d_cls_depT, depT);
    } else {
        cls.add(&d->d_cls_first_op, first_op);
    }
    cls.add(&d->d_cls_cnt0, cnt0);
    cls.add(&d->d_cls_ptr, cls_ptr);
    cls.add(&d->d_cls_cols, cls_cols);
    if (col_cls.empty()) {
        col_cls.assign(d->N, 0);
        for (int32_t c = 0; c < d->C; ++c)
            for (int32_t m = cls_ptr[c]; m < cls_ptr[c + 1]; ++m) col_cls[cls_cols[m]] = c;
    }
    cls.add(&d->d_col_cls, col_cls);
    if (!on_device && d->C <= 512 + kChainMaxGates) d->h_cls_dep = cls_dep;

    // what the tables of the bit-sliced TAC kernel are made from, when it is first run
    d->h_cls_lowest = std::move(lowest);
    if (!on_device) {
        d->h_cls_lowest.assign(d->C, -1);
        for (int32_t c = 0; c < d->C; ++c)
            for (int32_t w = 0; w < d->W; ++w)
                if (const uint64_t x = cls_dep[(size_t)c * d->W + w]) { d->h_cls_lowest[c] = w * 64 + __builtin_ctzll(x); break; }
    }
    if (from_sets) {
        // where op.dep of every op comes from: a class, or (~i) the bit of recv i
        op_src.resize(n);
        for (int32_t v = 0; v < n; ++v) op_src[v] = recv_of_op[v] >= 0 ? ~recv_of_op[v] : cls_of_set[sets.of_op[v]];
        cls.add(&d->d_op_src, op_src);
        if (R > 1024 || d->C > 8192) cls.add(&d->d_recv_of_op, recv_of_op);        // (TIC from the rows of the ops)
        cls.add(&d->d_bad_order, zeros);
        cls.reserve(&d->d_dep, dep_words * 8);
        // the tables of the propagation kernels, which recompute_deps runs
        if (prop_made.valid()) prop_made.get();
        if (dep_words) {
            prop.add_to(cls, d);
            prop.add_quads_to(cls, d);
        }
    }
    if (on_device) {
        cls.reserve(&d->d_cls_dep, (size_t)d->C * d->W * 8);
        cls.reserve(&d->d_cls_depT, (size_t)d->W * d->Cpad * 8);
    }
    HIP_TRY(cls.commit(d->class_block, d->device, s));
    if (from_sets && dep_words) HIP_TRY(launch_expand_sets(*d, s));
    int32_t *mismatch = d->d_bad_order + 1;         // (a second word of the zeroed flag block)
    if (on_device) HIP_TRY(launch_class_rows(*d, d->d_op_of_col, d->d_cls_first_op, mismatch, s));
    int32_t differs = 0;
    if (on_device) HIP_TRY(hipMemcpyAsync(&differs, mismatch, sizeof(int32_t), hipMemcpyDeviceToHost, s));
    HIP_TRY(cls.finish());              // (waits for `differs` as well; the handle is complete)
    d->long_runs = !on_device && std::max(d->C, d->R) > 256 && std::max(d->C, d->R) <= 512 && long_class_runs(col_cls);
    d->h_col_cls = std::move(col_cls);
    d->h_cls_cnt0 = std::move(cnt0);
    if (differs) {
        HIP_TRY(hipMemsetAsync(mismatch, 0, sizeof(int32_t), s));
        return 1;
    }
    return TICTAC_OK;
    };
    int rc = classes(dep_words * 8 >= ((size_t)8 << 20) && d->N > 0 && group_on_device(d->N, d->W) && !on_host && !getenv("TICTAC_GROUP_ON_HOST"));
    if (rc == 1) rc = classes(false);
    if (rc != TICTAC_OK || on_host) return rc;
    Packer quads;
    prop.add_quads_to(quads, d);
    HIP_TRY(quads.commit(d->quad_block, d->device, s));
    HIP_TRY(quads.finish());
    return TICTAC_OK;
}

// The tables of a handle's first TAC call go to the device on a stream of the library's own, one per device: the call waits
// for that copy and not for what is queued on the caller's stream, which may also be one that is being captured.
constexpr int kMaxDevices = 64;
static hipError_t table_stream(int device, hipStream_t *out)
{
    static std::mutex mutex;
    static hipStream_t streams[kMaxDevices];
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mutex);
    if (!streams[device]) {
        const hipError_t e = hipStreamCreateWithFlags(&streams[device], hipStreamNonBlocking);
        if (e != hipSuccess) return e;
    }
    *out = streams[device];
    return hipSuccess;
}

bool being_captured(hipStream_t s)
{
    hipStreamCaptureStatus c = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &c) == hipSuccess) return c != hipStreamCaptureStatusNone;
    (void)hipGetLastError();            // (the null stream while another stream is captured; the next launch would report it)
    return false;
}

static std::vector<int32_t> classes_of_ops(const Dag *d)
{
    std::vector<int32_t> cls_of_op(d->n, 0);
    for (int32_t r : d->h_recv_ids) cls_of_op[r] = -1;
    for (int32_t v = 0, j = 0; v < d->n; ++v)
        if (cls_of_op[v] >= 0) cls_of_op[v] = d->h_col_cls[j++];
    return cls_of_op;
}

static hipError_t make_sliced_tables(Dag *d)
{
    const int32_t CW = (d->C + 63) / 64;
    if (d->R < 1 || d->W > 64 || CW > 15 * 64 * 4) {
        d->sliced_made = true;
        return hipSuccess;
    }
    const std::vector<int32_t> cls_of_op = classes_of_ops(d), &cnt0 = d->h_cls_cnt0;
    Packer cls;
    d->CW = CW;
    d->CWpad = (CW + 15) / 16 * 16;
    // parents: among the classes of the compute predecessors of an op, those with a strictly smaller dep
    // that holds two recvs or more; the two largest are kept
    std::vector<int32_t> par((size_t)d->C * 2, -1);
    for (int32_t v = 0; v < d->n; ++v) {
        if (cls_of_op[v] < 0) continue;
        const int32_t cv = cls_of_op[v];
        for (int32_t e = d->h_row_ptr[v]; e < d->h_row_ptr[v + 1]; ++e) {
            const int32_t u = d->h_col_idx[e];
            if (cls_of_op[u] < 0) continue;
            const int32_t cu = cls_of_op[u];
            if (cnt0[cu] < 2 || cnt0[cu] >= cnt0[cv]) continue;
            int32_t *pv = &par[(size_t)cv * 2];
            if (pv[0] == cu || pv[1] == cu) continue;
            if (pv[0] < 0 || cnt0[cu] > cnt0[pv[0]]) { pv[1] = pv[0]; pv[0] = cu; }
            else if (pv[1] < 0 || cnt0[cu] > cnt0[pv[1]]) pv[1] = cu;
        }
    }
    std::vector<uint64_t> ndom0((size_t)d->CWpad * 2, 0);
    std::vector<int32_t> nchild(d->C, 0);
    for (int32_t c = 0; c < d->C; ++c)
        for (int j = 0; j < 2; ++j) {
            const int32_t u = par[(size_t)c * 2 + j];
            if (u < 0) continue;
            ndom0[(size_t)c >> 5] += 1ull << ((c & 31) * 2);
            ++nchild[u];
        }
    std::vector<int32_t> cptr(d->C + 1, 0);
    for (int32_t c = 0; c < d->C; ++c) cptr[c + 1] = cptr[c] + nchild[c];
    std::vector<int32_t> cidx(cptr[d->C]), cfill(cptr.begin(), cptr.end() - 1);
    for (int32_t c = 0; c < d->C; ++c)
        for (int j = 0; j < 2; ++j) {
            const int32_t u = par[(size_t)c * 2 + j];
            if (u >= 0) cidx[cfill[u]++] = c;
        }
    std::vector<int4> crec(d->C);
    std::vector<int32_t> child_ovf;
    for (int32_t c = 0; c < d->C; ++c) {
        const int32_t nc = nchild[c], *ch = cidx.data() + cptr[c];
        int4 r = make_int4(nc, -1, -1, -1);
        if (nc >= 1) r.y = ch[0];
        if (nc >= 2) r.z = ch[1];
        if (nc == 3) r.w = ch[2];
        if (nc > 3) {
            r.w = (int32_t)child_ovf.size();
            child_ovf.insert(child_ovf.end(), ch + 2, ch + nc);
        }
        crec[c] = r;
    }
    // classes that depend on one recv (by recv, ascending class) and on none
    std::vector<int32_t> single_ptr(d->R + 1, 0), single_cls, empty_cls, first_recv(d->C, -1);
    for (int32_t c = 0; c < d->C; ++c) {
        if (cnt0[c] == 0) empty_cls.push_back(c);
        if (cnt0[c] != 1) continue;
        first_recv[c] = d->h_cls_lowest[c];
        single_ptr[first_recv[c] + 1]++;
    }
    for (int32_t r = 0; r < d->R; ++r) single_ptr[r + 1] += single_ptr[r];
    single_cls.resize(single_ptr[d->R]);
    {
        std::vector<int32_t> fill(single_ptr.begin(), single_ptr.end() - 1);
        for (int32_t c = 0; c < d->C; ++c)
            if (cnt0[c] == 1) single_cls[fill[first_recv[c]]++] = c;
    }
    d->n_empty_cls = (int32_t)empty_cls.size();
    cls.add(&d->d_ndom0, ndom0);
    cls.add(&d->d_cls_par, par);
    cls.add(&d->d_crec, crec);
    cls.add(&d->d_child_ovf, child_ovf);
    cls.add(&d->d_single_ptr, single_ptr);
    cls.add(&d->d_single_cls, single_cls);
    cls.add(&d->d_empty_cls, empty_cls);
    cls.reserve(&d->d_colbits, (size_t)d->R * d->CWpad * 8);
    cls.reserve(&d->d_planes0, (size_t)13 * d->CWpad * 8);
    cls.reserve(&d->d_live0, (size_t)d->CWpad * 8);
    hipStream_t s;
    hipError_t e = table_stream(d->device, &s);
    if (e == hipSuccess) e = cls.commit(d->sliced_block, d->device, s);
    if (e == hipSuccess) e = launch_sliced_tables(*d, s);
    if (e == hipSuccess) e = cls.finish();
    d->sliced_made = e == hipSuccess;
    return e;
}

// What the frontier form's tables hold, from the graph as given (host work only).
static void plan_frontier(const Dag *d, FrontierPlan &p, FrontierTable &table)
{
    const std::vector<int32_t> cls_of_op = classes_of_ops(d);
    std::vector<int32_t> recv_of_op(d->n, -1), level(d->n, 0), order;
    for (int32_t i = 0; i < d->R; ++i) recv_of_op[d->h_recv_ids[i]] = i;
    const int32_t *row_ptr = d->h_row_ptr.data(), *col_idx = d->h_col_idx.data();
    bool topological = true;
    for (int32_t v = 0; v < d->n; ++v)
        for (int32_t e = row_ptr[v]; e < row_ptr[v + 1]; ++e) {
            topological &= col_idx[e] < v;
            level[v] = std::max(level[v], level[col_idx[e]] + 1);
        }
    int32_t n_levels = 0;
    if (topological || find_levels(d->n, row_ptr, col_idx, level, order, n_levels))
        make_frontier_plan(d->n, d->R, d->C, row_ptr, col_idx, level.data(), cls_of_op.data(), recv_of_op.data(), d->h_cls_cnt0, d->h_col_cls, p);
    if (p.ok) make_frontier_table(p, table);
}

static hipError_t commit_frontier(Dag *d, const FrontierPlan &p, const FrontierTable &table)
{
    FrontierTables &f = d->frontier;
    if (!p.ok) {
        f.made = true;
        return hipSuccess;
    }
    Packer t;
    t.add(&f.d_table, table.words);
    t.add(&f.d_inputs, table.inputs);
    t.add(&f.d_counters, p.counters);
    t.add(&f.d_wide, p.wide);
    t.add(&f.d_roots, p.roots);
    t.add(&f.d_free_cols, p.free_cols);
    t.add(&f.d_own_ptr, p.own_ptr);
    t.add(&f.d_own, p.own);
    if (p.numbered) {
        t.add(&f.d_cls_of, p.cls_of);
        t.reserve(&f.d_cls_dep, (size_t)d->C * d->W * 8);
    }
    hipStream_t s;
    hipError_t e = table_stream(d->device, &s);
    if (e == hipSuccess) e = t.commit(f.block, d->device, s);
    if (e == hipSuccess && p.numbered) e = launch_frontier_rows(*d, s);
    if (e == hipSuccess) e = t.finish();
    if (e != hipSuccess) return e;
    f.n_counters = (int32_t)p.counters.size();
    f.n_roots = (int32_t)p.roots.size();
    f.n_free = (int32_t)p.free_cols.size();
    f.ok = f.made = true;
    return hipSuccess;
}

hipError_t ensure_large_tables(Dag *d, bool frontier)
{
    std::lock_guard<std::mutex> lock(d->tables_mutex);
    frontier = frontier && !d->frontier.made;
    if (!frontier) return d->sliced_made ? hipSuccess : make_sliced_tables(d);
    FrontierPlan plan;
    FrontierTable table;
    std::future<void> planned;              // (after what its thread works on: it ends first)
    auto make = [&] { plan_frontier(d, plan, table); };
    hipError_t e = hipSuccess, ef = hipSuccess;
    if (!d->sliced_made) {
        if ((int64_t)d->n + d->E > kPropThread) {
            try {
                planned = std::async(std::launch::async, make);
            } catch (const std::system_error &) {           // (no thread to be had)
            }
        }
        e = make_sliced_tables(d);
    }
    try {
        if (planned.valid()) planned.get();
        else make();
        ef = commit_frontier(d, plan, table);
    } catch (const std::bad_alloc &) {
        ef = hipErrorOutOfMemory;
    }
    return e != hipSuccess || ef == hipErrorOutOfMemory ? e : ef;
}

struct ChainUpload {
    const ChainPlan &p;
    ChainRec *rec = nullptr;
    ChainGate *gate = nullptr;

    explicit ChainUpload(const ChainPlan &plan) : p(plan) {}
    void add(Packer &t, ChainTables &c)
    {
        static_assert(sizeof(ChainRec) == 16 && sizeof(ChainGate) == 16, "records are read as 16 bytes");
        t.add(&rec, p.rec);
        t.add(&gate, p.gate);
        t.add(&c.d_list, p.list);
        t.add(&c.d_place, p.place);
        t.add(&c.d_extra, p.extra);
        t.add(&c.d_head, p.head);
        t.add(&c.d_cand_ptr, p.cand_ptr);
        t.add(&c.d_cand, p.cand);
    }
    void done(ChainTables &c) const         // (they are on the device)
    {
        c.d_rec = reinterpret_cast<int4 *>(rec);
        c.d_gate = reinterpret_cast<int4 *>(gate);
        c.n_chains = p.n_slots; c.n_gates = (int32_t)p.gate.size();
        c.start = p.start; c.n_start = p.n_start; c.empty = p.empty;
        c.second_gates = p.second_gates; c.n_extra = p.n_extra; c.n_head = (int32_t)p.head.size();
        c.ok = c.made = true;
    }
};

// The tables of class_totals_kernel first, for which a call launches it; those of tac_chain_kernel (ensure_chain_tables) are made while it
// runs: the first call on inception3 (5 912 ops), 8 192 samples, takes 383 us and not 427, on resnet50 (1 260 ops) 139 and not 149.  Of small
// graphs (vgg16, 90 ops) all tables are made at once: a second copy and its wait take 6 us more than there is to plan.
// Whether the graph has the form is known here, before a call takes memory or launches anything for it (hipErrorNotSupported: it has not), and
// so is the room that its other tables take: a workspace that left none for them would be of no use.
constexpr int64_t kChainAtOnce = 1000;      // ops and predecessors
hipError_t ensure_chain_columns(Dag *d)
try {
    std::lock_guard<std::mutex> lock(d->tables_mutex);
    ChainTables &c = d->chain;
    if (c.made) return c.ok ? hipSuccess : hipErrorNotSupported;
    if (c.cols_made) return hipSuccess;
    const size_t W = (size_t)d->W;
    auto sets = std::make_shared<ChainSets>();
    auto form = std::make_shared<ChainForm>();
    ChainColumns p;
    // pieces of one set (classes with equal rows) are one set again: they follow each other
    std::vector<int32_t> set_of_cls(d->C), set_of_col(d->N), set_of_op(d->n, 0);
    bool may_be = !d->h_cls_dep.empty();
    for (int32_t k = 0; k < d->C && may_be; ++k) {
        const uint64_t *row = &d->h_cls_dep[k * W];
        if (sets->rows.empty() || memcmp(sets->rows.back(), row, W * 8) != 0) {
            sets->rows.push_back(row);
            sets->row_of_set.push_back(k);
        }
        set_of_cls[k] = (int32_t)sets->rows.size() - 1;
    }
    may_be = may_be && chain_may_be(d->R, (int)sets->rows.size());
    if (may_be) {
        for (int32_t r : d->h_recv_ids) set_of_op[r] = -1;
        for (int32_t v = 0, j = 0; v < d->n; ++v)
            if (set_of_op[v] >= 0) {
                set_of_op[v] = set_of_col[j] = set_of_cls[d->h_col_cls[j]];
                ++j;
            }
        may_be = chain_owners(d->R, d->W, d->n, d->h_row_ptr.data(), d->h_col_idx.data(), set_of_op.data(), *sets) &&
                 chain_form(d->R, d->W, *sets, *form) && make_chain_columns(d->N, (int)sets->rows.size(), set_of_col.data(), p);
    }
    if (!may_be) {
        c.made = true;
        return hipErrorNotSupported;
    }
    const bool at_once = (int64_t)d->n + d->E <= kChainAtOnce;
    ChainPlan plan;
    if (at_once) make_chain_plan(d->R, *sets, *form, p.first, plan);
    ChainUpload up(plan);
    Packer t;
    t.add(&c.d_several, p.several);
    t.add(&c.d_flush, p.flush);
    t.add(&c.d_flush_row, p.flush_row);
    t.add(&c.d_block_first, p.block_first);
    if (at_once) up.add(t, c);
    else t.reserve(&c.room, chain_plan_bytes(d->R, *form));
    hipStream_t s;
    hipError_t e = table_stream(d->device, &s);
    if (e == hipSuccess) e = t.commit(c.block, d->device, s);
    if (e == hipSuccess) e = t.finish();
    if (e != hipSuccess) return e;
    c.first_total = std::move(p.first);
    c.n_totals = c.first_total.back(); c.n_several = (int32_t)p.several.size(); c.n_pairs = p.n_pairs;
    c.cols_made = true;
    if (at_once) {
        up.done(c);
    } else {
        c.sets = std::move(sets);
        c.form = std::move(form);
    }
    return hipSuccess;
} catch (const std::bad_alloc &) {
    return hipErrorOutOfMemory;
}

// (after ensure_chain_columns has found that the graph has the form)
hipError_t ensure_chain_tables(Dag *d)
try {
    std::lock_guard<std::mutex> lock(d->tables_mutex);
    ChainTables &c = d->chain;
    if (c.made) return hipSuccess;
    ChainPlan p;
    make_chain_plan(d->R, *c.sets, *c.form, c.first_total, p);
    ChainUpload up(p);
    Packer t;
    t.by_kernel = false;                    // (class_totals_kernel runs meanwhile)
    up.add(t, c);
    hipStream_t s;
    hipError_t e = table_stream(d->device, &s);
    if (e == hipSuccess) e = t.commit_at(c.room, chain_plan_bytes(d->R, *c.form), s);
    if (e == hipSuccess) e = t.finish();
    if (e != hipSuccess) return e;          // (the next call plans again)
    up.done(c);
    c.sets.reset();
    c.form.reset();
    return hipSuccess;
} catch (const std::bad_alloc &) {
    return hipErrorOutOfMemory;
}

}  // namespace tictac

using namespace tictac;

extern "C" {

int tictac_build_deps(int32_t n_ops, const int32_t *pred_row_ptr, const int32_t *pred_col_idx, int32_t n_recv,
                      const int32_t *recv_ids, tictac_stream stream, tictac_dag **out)
try {
    if (!out) { set_error("out is NULL"); return TICTAC_ERR_NULL; }
    Dag *d = new (std::nothrow) Dag();
    if (!d) { set_error("out of host memory"); return TICTAC_ERR_NO_MEM; }
    int rc;
    try {
        rc = build(n_ops, pred_row_ptr, pred_col_idx, n_recv, recv_ids, (hipStream_t)stream, d);
    } catch (...) {
        rc = caught();
    }
    if (rc != TICTAC_OK) { free_dag(d); return rc; }
    *out = reinterpret_cast<tictac_dag *>(d);
    return TICTAC_OK;
} TT_CATCH

int tictac_dag_info(const tictac_dag *dag, int32_t *n_ops, int32_t *n_recv, int32_t *words, int32_t *n_levels,
                    int32_t *n_classes)
try {
    if (!dag) { set_error("dag is NULL"); return TICTAC_ERR_NULL; }
    const Dag *d = reinterpret_cast<const Dag *>(dag);
    if (n_ops) *n_ops = d->n;
    if (n_recv) *n_recv = d->R;
    if (words) *words = d->W;
    if (n_levels) *n_levels = d->n_levels;
    if (n_classes) *n_classes = d->C_distinct;
    return TICTAC_OK;
} TT_CATCH

int tictac_dag_deps(const tictac_dag *dag, const uint64_t **dep_device)
try {
    if (!dag || !dep_device) { set_error("NULL argument"); return TICTAC_ERR_NULL; }
    *dep_device = reinterpret_cast<const Dag *>(dag)->d_dep;
    return TICTAC_OK;
} TT_CATCH

int tictac_dag_copy_deps(const tictac_dag *dag, uint64_t *dst_device, tictac_stream stream)
try {
    if (!dag) { set_error("dag is NULL"); return TICTAC_ERR_NULL; }
    const Dag *d = reinterpret_cast<const Dag *>(dag);
    const size_t bytes = (size_t)d->n * d->W * 8;
    if (bytes == 0) return TICTAC_OK;
    if (!dst_device) { set_error("dst_device is NULL"); return TICTAC_ERR_NULL; }
    HIP_TRY(hipMemcpyAsync(dst_device, d->d_dep, bytes, hipMemcpyDeviceToDevice, (hipStream_t)stream));
    return TICTAC_OK;
} TT_CATCH

int tictac_dag_recompute_deps(tictac_dag *dag, tictac_stream stream)
try {
    if (!dag) { set_error("dag is NULL"); return TICTAC_ERR_NULL; }
    HIP_TRY(launch_propagate(*reinterpret_cast<Dag *>(dag), (hipStream_t)stream));
    return TICTAC_OK;
} TT_CATCH

int tictac_dag_recompute_deps_batch(tictac_dag *const *dags, int32_t n_dags, tictac_stream stream)
try {
    if (n_dags < 0) { set_error("n_dags = %d is negative", n_dags); return TICTAC_ERR_UNSUPPORTED; }
    if (n_dags == 0) return TICTAC_OK;
    if (!dags) { set_error("dags is NULL"); return TICTAC_ERR_NULL; }
    for (int32_t g = 0; g < n_dags; ++g)
        if (!dags[g]) { set_error("dags[%d] is NULL", g); return TICTAC_ERR_NULL; }
    Dag *const *ds = reinterpret_cast<Dag *const *>(dags);
    hipStream_t s = (hipStream_t)stream;
    HIP_TRY(ensure_workspace(ds[0], propagate_batch_staging_bytes(n_dags)));
    const hipError_t e = launch_propagate_batch(ds, n_dags, ds[0]->d_work, s);
    if (e == hipErrorNotSupported) {
        // graphs of different shapes, or graphs that take another propagation kernel: one after the other
        for (int32_t g = 0; g < n_dags; ++g) HIP_TRY(launch_propagate(*ds[g], s));
        return TICTAC_OK;
    }
    HIP_TRY(e);
    return TICTAC_OK;
} TT_CATCH

int tictac_dag_free(tictac_dag *dag)
try {
    if (!dag) return TICTAC_OK;
    free_dag(reinterpret_cast<Dag *>(dag));
    return TICTAC_OK;
} TT_CATCH

int tictac_trim_memory(void)
try {
    HIP_TRY(trim_memory());
    return TICTAC_OK;
} TT_CATCH

int tictac_tic_priority(const tictac_dag *dag, int32_t *prio, int32_t *order, int32_t *rank, tictac_stream stream)
try {
    if (!dag) { set_error("dag is NULL"); return TICTAC_ERR_NULL; }
    const Dag *d = reinterpret_cast<const Dag *>(dag);
    if (d->R == 0) return TICTAC_OK;
    if (!prio) { set_error("prio is NULL"); return TICTAC_ERR_NULL; }
    HIP_TRY(launch_tic(*d, prio, order, rank, nullptr, (hipStream_t)stream));
    return TICTAC_OK;
} TT_CATCH

static int check_batch(const Dag *d, int32_t B, const void *op_time, const void *recv_time)
{
    if (B < 0) { set_error("B = %d", B); return TICTAC_ERR_BAD_CSR; }
    if (B > 0 && d->N > 0 && !op_time) { set_error("op_time is NULL"); return TICTAC_ERR_NULL; }
    if (B > 0 && d->R > 0 && !recv_time) { set_error("recv_time is NULL"); return TICTAC_ERR_NULL; }
    return TICTAC_OK;
}

int tictac_tac_priority(const tictac_dag *dag, int32_t B, const double *op_time, const double *recv_time,
                        int32_t *order, int32_t *rank, double *sel_P, double *sel_Mplus, tictac_stream stream)
try {
    if (!dag) { set_error("dag is NULL"); return TICTAC_ERR_NULL; }
    Dag *d = const_cast<Dag *>(reinterpret_cast<const Dag *>(dag));
    int rc = check_batch(d, B, op_time, recv_time);
    if (rc != TICTAC_OK) return rc;
    if (B == 0 || d->R == 0) return TICTAC_OK;
    if (!order) { set_error("order is NULL"); return TICTAC_ERR_NULL; }
    TacArgs a{B, op_time, recv_time, order, rank, sel_P, sel_Mplus, false, nullptr, nullptr, nullptr, nullptr, nullptr};
    HIP_TRY(launch_tac(*d, a, (hipStream_t)stream));
    return TICTAC_OK;
} TT_CATCH

static int tac_simulate_any(const tictac_dag *dag, int32_t B, const void *op_time, const void *recv_time, bool f32,
                            int32_t *order, int32_t *rank, double *sel_P, double *sel_Mplus, double *makespan,
                            double *eff, double *U, double *L, double *S, tictac_stream stream)
{
    if (!dag) { set_error("dag is NULL"); return TICTAC_ERR_NULL; }
    Dag *d = const_cast<Dag *>(reinterpret_cast<const Dag *>(dag));
    int rc = check_batch(d, B, op_time, recv_time);
    if (rc != TICTAC_OK) return rc;
    if (B == 0) return TICTAC_OK;
    if (d->R > 0 && !order) { set_error("order is NULL"); return TICTAC_ERR_NULL; }
    TacArgs a{B, op_time, recv_time, order, rank, sel_P, sel_Mplus, true, makespan, eff, U, L, S};
    a.f32 = f32;
    HIP_TRY(launch_tac(*d, a, (hipStream_t)stream));
    return TICTAC_OK;
}

// ---- the entry point that allocates nothing ----
// Per-call memory of tictac_tac_simulate_noalloc: one flag per sample ("left to the general kernel").  The
// array exists once per GPU for as long as the library is loaded; every call on a GPU uses it.
constexpr int32_t kNoallocMaxB = 1 << 20;
static __device__ __align__(256) int32_t scratch[kNoallocMaxB];
static void *g_scratch_ptr[kMaxDevices];         // device address of `scratch` on every device, 0 = not asked yet
static std::mutex g_scratch_mutex;

// the device address of the array on the current device (asked of the runtime once per device)
static hipError_t scratch_address(int32_t **out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *q = nullptr;
        e = hipGetSymbolAddress(&q, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[dev] = q;
    }
    *out = static_cast<int32_t *>(g_scratch_ptr[dev]);
    return hipSuccess;
}

int tictac_tac_simulate_noalloc(const tictac_dag *dag, int32_t B, const double *op_time, const double *recv_time,
                                int32_t *order, int32_t *rank, double *makespan, double *eff, double *U, double *L,
                                double *S, tictac_stream stream)
try {
    if (!dag) { set_error("dag is NULL"); return TICTAC_ERR_NULL; }
    Dag *d = const_cast<Dag *>(reinterpret_cast<const Dag *>(dag));
    int rc = check_batch(d, B, op_time, recv_time);
    if (rc != TICTAC_OK) return rc;
    if (B > kNoallocMaxB) {
        set_error("B = %d: tictac_tac_simulate_noalloc takes at most %d samples per call", B, kNoallocMaxB);
        return TICTAC_ERR_UNSUPPORTED;
    }
    if (B == 0) return TICTAC_OK;
    if (d->R > 0 && !order) { set_error("order is NULL"); return TICTAC_ERR_NULL; }
    int32_t *flags = nullptr;
    HIP_TRY(scratch_address(&flags));
    TacArgs a{B, op_time, recv_time, order, rank, nullptr, nullptr, true, makespan, eff, U, L, S};
    a.ext_flags = flags;
    const hipError_t e = launch_tac(*d, a, (hipStream_t)stream);
    if (e == hipErrorNotSupported) {
        set_error("%d recvs, %d classes: tictac_tac_simulate_noalloc serves graphs with at most 512 classes of compute ops, "
                  "384 recvs and per-sample state that fits the local memory of a compute unit", d->R, d->C);
        return TICTAC_ERR_UNSUPPORTED;
    }
    HIP_TRY(e);
    return TICTAC_OK;
} TT_CATCH

int tictac_tac_simulate(const tictac_dag *dag, int32_t B, const double *op_time, const double *recv_time,
                        int32_t *order, int32_t *rank, double *sel_P, double *sel_Mplus, double *makespan,
                        double *eff, double *U, double *L, double *S, tictac_stream stream)
try {
    return tac_simulate_any(dag, B, op_time, recv_time, false, order, rank, sel_P, sel_Mplus, makespan, eff, U, L, S,
                            stream);
} TT_CATCH

int tictac_tac_simulate_f32(const tictac_dag *dag, int32_t B, const float *op_time, const float *recv_time,
                            int32_t *order, int32_t *rank, double *sel_P, double *sel_Mplus, double *makespan,
                            double *eff, double *U, double *L, double *S, tictac_stream stream)
try {
    return tac_simulate_any(dag, B, op_time, recv_time, true, order, rank, sel_P, sel_Mplus, makespan, eff, U, L, S,
                            stream);
} TT_CATCH

static int simulate_any(const tictac_dag *dag, int32_t B, const int32_t *order, int32_t order_stride,
                        const void *op_time, const void *recv_time, bool f32, double *makespan, double *eff, double *U,
                        double *L, double *S, tictac_stream stream)
{
    if (!dag) { set_error("dag is NULL"); return TICTAC_ERR_NULL; }
    Dag *d = const_cast<Dag *>(reinterpret_cast<const Dag *>(dag));
    int rc = check_batch(d, B, op_time, recv_time);
    if (rc != TICTAC_OK) return rc;
    if (order_stride != 0 && order_stride != d->R) {
        set_error("order_stride = %d, expected 0 or n_recv = %d", order_stride, d->R);
        return TICTAC_ERR_BAD_ORDER;
    }
    if (B == 0) return TICTAC_OK;
    if (d->R > 0 && !order) { set_error("order is NULL"); return TICTAC_ERR_NULL; }
    if (!makespan || !eff) { set_error("makespan or eff is NULL"); return TICTAC_ERR_NULL; }
    SimArgs a{B, order, order_stride, op_time, recv_time, makespan, eff, U, L, S};
    a.f32 = f32;
    HIP_TRY(launch_simulate(*d, a, (hipStream_t)stream));
    return TICTAC_OK;
}

int tictac_simulate(const tictac_dag *dag, int32_t B, const int32_t *order, int32_t order_stride,
                    const double *op_time, const double *recv_time, double *makespan, double *eff, double *U,
                    double *L, double *S, tictac_stream stream)
try {
    return simulate_any(dag, B, order, order_stride, op_time, recv_time, false, makespan, eff, U, L, S, stream);
} TT_CATCH

int tictac_simulate_f32(const tictac_dag *dag, int32_t B, const int32_t *order, int32_t order_stride,
                        const float *op_time, const float *recv_time, double *makespan, double *eff, double *U,
                        double *L, double *S, tictac_stream stream)
try {
    return simulate_any(dag, B, order, order_stride, op_time, recv_time, true, makespan, eff, U, L, S, stream);
} TT_CATCH

int tictac_simulate_channels(const tictac_dag *dag, int32_t B, int32_t n_channels, const int32_t *channel_of_recv,
                             const int32_t *order, int32_t order_stride, const double *op_time,
                             const double *recv_time, double *makespan, double *eff, double *U, double *L,
                             double *S, tictac_stream stream)
try {
    if (!dag) { set_error("dag is NULL"); return TICTAC_ERR_NULL; }
    Dag *d = const_cast<Dag *>(reinterpret_cast<const Dag *>(dag));
    int rc = check_batch(d, B, op_time, recv_time);
    if (rc != TICTAC_OK) return rc;
    if (n_channels < 1 || n_channels > 64) {
        set_error("n_channels = %d, expected 1 .. 64", n_channels);
        return TICTAC_ERR_UNSUPPORTED;
    }
    if (order_stride != 0 && order_stride != d->R) {
        set_error("order_stride = %d, expected 0 or n_recv = %d", order_stride, d->R);
        return TICTAC_ERR_BAD_ORDER;
    }
    if (d->R > 0 && !channel_of_recv) { set_error("channel_of_recv is NULL"); return TICTAC_ERR_NULL; }
    for (int32_t i = 0; i < d->R; ++i)
        if (channel_of_recv[i] < 0 || channel_of_recv[i] >= n_channels) {
            set_error("channel_of_recv[%d] = %d is outside 0 .. %d", i, channel_of_recv[i], n_channels - 1);
            return TICTAC_ERR_BAD_ORDER;
        }
    if (B == 0) return TICTAC_OK;
    if (d->R > 0 && !order) { set_error("order is NULL"); return TICTAC_ERR_NULL; }
    if (!makespan || !eff) { set_error("makespan or eff is NULL"); return TICTAC_ERR_NULL; }
    SimArgs a{B, order, order_stride, op_time, recv_time, makespan, eff, U, L, S};
    hipStream_t s = (hipStream_t)stream;
    if (d->R == 0) {                      // no transfers: the channels play no role
        HIP_TRY(launch_simulate(*d, a, s));
        return TICTAC_OK;
    }
    if (d->R > 512 || d->C > 512) {
        set_error("%d recvs and %d classes: the several-channel simulation handles at most 512 of each", d->R, d->C);
        return TICTAC_ERR_UNSUPPORTED;
    }
    // the channel table goes to the device through a staging block of the handle
    HIP_TRY(ensure_chan_table(d, channel_of_recv, s));
    const hipError_t e = launch_simulate_channels(*d, a, n_channels, d->d_chan, s);
    if (e == hipErrorNotSupported) {
        set_error("graph outside what the several-channel simulation handles");
        return TICTAC_ERR_UNSUPPORTED;
    }
    HIP_TRY(e);
    return TICTAC_OK;
} TT_CATCH

int tictac_dag_check_orders(tictac_dag *dag, tictac_stream stream)
try {
    if (!dag) { set_error("dag is NULL"); return TICTAC_ERR_NULL; }
    Dag *d = reinterpret_cast<Dag *>(dag);
    if (!d->d_bad_order) return TICTAC_OK;
    hipStream_t s = (hipStream_t)stream;
    int32_t raised = 0;
    HIP_TRY(hipMemcpyAsync(&raised, d->d_bad_order, sizeof(int32_t), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    if (raised == 0) return TICTAC_OK;
    HIP_TRY(hipMemsetAsync(d->d_bad_order, 0, sizeof(int32_t), s));
    set_error("an order given since the last check was no permutation of 0 .. n_recv-1");
    return TICTAC_ERR_BAD_ORDER;
} TT_CATCH

// Tables of the iteration with send ops for the given send set (kept until another set is given).
// TICTAC_OK, or the status to return (the error text is set).
static int ensure_send_tables(Dag *d, int32_t n_send, const int32_t *send_ids, hipStream_t s)
{
    if (d->send_tables_built && d->h_send_ids.size() == (size_t)n_send &&
        (n_send == 0 || memcmp(d->h_send_ids.data(), send_ids, (size_t)n_send * sizeof(int32_t)) == 0))
        return TICTAC_OK;
    const int32_t n = d->n, E = d->E;
    std::vector<int32_t> recv_of_op(n, -1), col_of_op(n, -1), n_succ(n, 0);
    for (int32_t i = 0; i < d->R; ++i) recv_of_op[d->h_recv_ids[i]] = i;
    for (int32_t v = 0, j = 0; v < n; ++v)
        if (recv_of_op[v] < 0) col_of_op[v] = j++;
    for (int32_t e = 0; e < E; ++e) n_succ[d->h_col_idx[e]]++;
    std::vector<uint8_t> is_send(n, 0);
    for (int32_t i = 0; i < n_send; ++i) {
        const int32_t v = send_ids[i];
        if (v < 0 || v >= n) { set_error("send_ids[%d] = %d is no op id", i, v); return TICTAC_ERR_BAD_CSR; }
        if (recv_of_op[v] >= 0) { set_error("send_ids[%d] = %d is a recv op", i, v); return TICTAC_ERR_BAD_CSR; }
        if (is_send[v]) { set_error("send_ids holds op %d twice", v); return TICTAC_ERR_BAD_CSR; }
        if (n_succ[v] != 0) {
            set_error("send op %d has successors (Sec. 2.2: the send ops are leaves)", v);
            return TICTAC_ERR_BAD_CSR;
        }
        is_send[v] = 1;
    }
    // rec[v]: where the successors of v start in succ (-1: none), the column of its time (-1: a recv), 1 for a send.
    // succ[e]: a successor (the top bit marks the last one of its list), and what running that successor needs, so
    // that an op released by the op before it is run without a read of rec: its column, where its own successors
    // start, 1 for a send.  64 entries of padding: a wave reads 64 entries at a time.
    std::vector<int4> rec(n), succ((size_t)E + 64, make_int4(0, 0, 0, 0));
    std::vector<int32_t> fill(n), send_free;
    std::vector<uint16_t> indeg(n);
    std::vector<uint32_t> ready0(((size_t)n + 31) / 32, 0u);
    std::vector<uint8_t> col_kind(d->N > 0 ? d->N : 1, 0);
    int32_t at = 0;
    for (int32_t v = 0; v < n; ++v) {
        rec[v] = make_int4(n_succ[v] > 0 ? at : -1, 0, col_of_op[v], is_send[v]);
        fill[v] = at;
        at += n_succ[v];
        const int32_t deg = d->h_row_ptr[v + 1] - d->h_row_ptr[v];
        if (deg > 65535) { set_error("op %d has %d predecessors, more than 65535", v, deg); return TICTAC_ERR_UNSUPPORTED; }
        indeg[v] = (uint16_t)deg;
        if (recv_of_op[v] < 0 && deg == 0) {
            if (is_send[v]) send_free.push_back(col_of_op[v]);
            else ready0[v >> 5] |= 1u << (v & 31);
        }
        if (is_send[v]) col_kind[col_of_op[v]] = 1;
    }
    for (int32_t v = 0; v < n; ++v)
        for (int32_t e = d->h_row_ptr[v]; e < d->h_row_ptr[v + 1]; ++e) {
            const int32_t u = d->h_col_idx[e], at_u = fill[u]++;
            const bool last = at_u + 1 == rec[u].x + n_succ[u];
            succ[at_u] = make_int4(last ? (int32_t)((uint32_t)v | 0x80000000u) : v, rec[v].z, rec[v].x, rec[v].w);
        }

    // The form with one lane per sample: columns of 13 bits, lists short on average (a lane goes through its successors one
    // by one), and counters of half a byte, or of a byte, for the ops of several predecessors.
    std::vector<uint2> lane_rec, lane_recv_rec;
    std::vector<uint32_t> lane_succ;
    std::vector<uint8_t> lane_cnt0;
    std::vector<uint64_t> lane_ready0;
    const uint16_t most = n > 0 ? *std::max_element(indeg.begin(), indeg.end()) : (uint16_t)0;
    if (d->N <= 8128 && most <= 255 && (int64_t)E <= 4 * (int64_t)n) {
        d->lane_half = most <= 15;
        std::vector<uint32_t> entry(n, 0);
        lane_ready0.assign(((size_t)d->N + 63) / 64, 0);
        uint32_t counters = 0;
        for (int32_t v = 0; v < n; ++v) {
            const int32_t j = col_of_op[v];
            if (j < 0) continue;
            uint32_t c = 0;
            if (indeg[v] > 1) {
                c = ++counters;
                if (!d->lane_half || (c & 1)) lane_cnt0.push_back((uint8_t)indeg[v]);
                else lane_cnt0.back() |= (uint8_t)(indeg[v] << 4);
            }
            entry[v] = (uint32_t)j | (is_send[v] ? 1u << 13 : 0u) | c << 14;
            if (indeg[v] == 0 && !is_send[v]) lane_ready0[j >> 6] |= 1ull << (j & 63);
        }
        lane_rec.resize(d->N);
        lane_recv_rec.resize(d->R);
        for (int32_t v = 0; v < n; ++v) {
            uint2 &r = recv_of_op[v] >= 0 ? lane_recv_rec[recv_of_op[v]] : lane_rec[col_of_op[v]];
            r = make_uint2(1u << 30, 0u);
            if (n_succ[v] == 0) continue;
            // (the sends last: the first successor is the op that is expected to run next)
            const int4 *list = &succ[rec[v].x];
            const size_t first = lane_succ.size();
            for (int pass = 0; pass < 2; ++pass)
                for (int32_t e = 0; e < n_succ[v]; ++e)
                    if (list[e].w == pass) lane_succ.push_back(entry[list[e].x & 0x7fffffff]);
            r.x = lane_succ[first];
            lane_succ.erase(lane_succ.begin() + first);
            if (n_succ[v] == 1) continue;
            lane_succ.back() |= 0x80000000u;
            r.y = (uint32_t)first + 1u;
        }
    }
    lane_cnt0.resize((lane_cnt0.size() + 3) / 8 * 8 + 4, 0);       // (an odd number of words of 4 bytes: see SendLaneParams::words)
    d->n_lane_succ = (int32_t)lane_succ.size();

    // The straight form: ids in topological order, sends behind compute ops only, at most a tile's worth of recvs per op.
    // A graph that starts with several ops waiting side by side would give up nearly every sample at once (the transfers
    // have no lead yet): none of the first ops may wait for a recv unless it is alone.
    std::vector<uint32_t> st_code;
    std::vector<int32_t> st_chk, st_req(send_free);
    std::vector<int4> st_tiles;
    {
        bool ok = d->N > 1;
        std::vector<int32_t> last_pred(d->N, -1), n_chk(d->N, 0), n_req(d->N, 0), others(d->N + 1, 0);
        std::vector<std::vector<int32_t>> sends_after(d->N);
        for (int32_t v = 0; v < n && ok; ++v) {
            const int32_t j = col_of_op[v];
            for (int32_t e = d->h_row_ptr[v]; e < d->h_row_ptr[v + 1]; ++e) {
                const int32_t u = d->h_col_idx[e];
                ok = ok && u < v && !(is_send[v] && recv_of_op[u] >= 0);
                if (recv_of_op[u] >= 0) ++n_chk[j];
                else last_pred[j] = std::max(last_pred[j], col_of_op[u]);
            }
            ok = ok && (j < 0 || n_chk[j] <= 32);
            if (j < 0 || !ok) continue;
            if (is_send[v]) {
                if (last_pred[j] >= 0) sends_after[last_pred[j]].push_back(j);
            } else if (last_pred[j] + 1 < j) {
                // between its last predecessor and itself the op could run in place of one that waits
                ++others[last_pred[j] + 1];
                --others[j];
            }
        }
        for (int32_t v = 0, open = 0; v < n && ok; ++v) {
            const int32_t j = col_of_op[v];
            if (j < 0) continue;
            open += others[j];
            if (st_tiles.empty() || st_tiles[st_tiles.size() - 2].y == 64 || st_tiles[st_tiles.size() - 2].w + n_chk[j] > 32) {
                st_tiles.push_back(make_int4(j, 0, (int32_t)st_chk.size(), 0));
                st_tiles.push_back(make_int4(0, 0, 0, 0));
                st_code.resize(st_tiles.size() * 32, 0u);
            }
            int4 &tile = st_tiles[st_tiles.size() - 2], &mask = st_tiles.back();
            const int32_t at = tile.y++;
            uint32_t &code = st_code[st_tiles.size() * 32 - 64 + at];
            if (is_send[v]) continue;
            ok = sends_after[j].size() <= 0xffffu;
            code = 1u | (uint32_t)n_chk[j] << 1 | (open == 0 ? 0x100u : 0u) | (uint32_t)sends_after[j].size() << 16;
            st_req.insert(st_req.end(), sends_after[j].begin(), sends_after[j].end());
            if (j < 16 && n_chk[j] > 0 && open != 0) ok = false;
            (at < 32 ? mask.x : mask.y) |= (int32_t)(1u << (at & 31));
            if (n_chk[j] > 0 || !sends_after[j].empty()) (at < 32 ? mask.z : mask.w) |= (int32_t)(1u << (at & 31));
            tile.w += n_chk[j];
            for (int32_t e = d->h_row_ptr[v]; e < d->h_row_ptr[v + 1]; ++e)
                if (recv_of_op[d->h_col_idx[e]] >= 0) st_chk.push_back(recv_of_op[d->h_col_idx[e]]);
        }
        if (!ok) { st_tiles.clear(); st_code.clear(); st_chk.clear(); }
        // (sends alone at the end: nothing runs there)
        while (st_tiles.size() > 2 && !(st_tiles.back().x | st_tiles.back().y | st_tiles.back().z | st_tiles.back().w)) {
            st_tiles.resize(st_tiles.size() - 2);
            st_code.resize(st_tiles.size() * 32);
        }
        d->straight_req_lo = d->straight_req_span = 0;
        if (!st_req.empty()) {
            const auto ends = std::minmax_element(st_req.begin(), st_req.end());
            d->straight_req_lo = *ends.first;
            d->straight_req_span = *ends.second - *ends.first + 1;
        }
    }
    st_chk.resize(st_chk.size() + 32, 0);
    d->n_straight_tiles = (int32_t)st_tiles.size() / 2;
    if (d->n_straight_tiles > 0) st_tiles.resize(st_tiles.size() + 2, make_int4(0, 0, 0, 0));      // (read, not used)
    d->lane_cnt_bytes = (int32_t)lane_cnt0.size();

    Packer tables;
    tables.add(&d->d_straight_code, st_code);
    tables.add(&d->d_straight_chk, st_chk);
    tables.add(&d->d_straight_req, st_req);
    tables.add(&d->d_straight_tiles, st_tiles);
    tables.add(&d->d_lane_rec, lane_rec);
    tables.add(&d->d_lane_recv_rec, lane_recv_rec);
    tables.add(&d->d_lane_succ, lane_succ);
    tables.add(&d->d_lane_cnt0, lane_cnt0);
    tables.add(&d->d_lane_ready0, lane_ready0);
    tables.add(&d->d_send_rec, rec);
    tables.add(&d->d_send_succ, succ);
    tables.add(&d->d_send_indeg, indeg);
    tables.add(&d->d_send_ready0, ready0);
    tables.add(&d->d_send_free, send_free);
    tables.add(&d->d_send_col_kind, col_kind);
    tables.add(&d->d_send_recv_ids, d->h_recv_ids);
    d->n_send_free = (int32_t)send_free.size();
    d->send_tables_built = false;
    HIP_TRY(tables.commit(d->send_block, d->device, s));
    HIP_TRY(tables.finish());
    d->h_send_ids.assign(send_ids, send_ids + n_send);
    d->send_tables_built = true;
    return TICTAC_OK;
}

int tictac_simulate_sends(const tictac_dag *dag, int32_t B, int32_t n_send, const int32_t *send_ids,
                          const int32_t *order, int32_t order_stride, const double *op_time,
                          const double *recv_time, double *makespan, double *eff, double *U, double *L, double *S,
                          tictac_stream stream)
try {
    if (!dag) { set_error("dag is NULL"); return TICTAC_ERR_NULL; }
    Dag *d = const_cast<Dag *>(reinterpret_cast<const Dag *>(dag));
    int rc = check_batch(d, B, op_time, recv_time);
    if (rc != TICTAC_OK) return rc;
    if (n_send < 0) { set_error("n_send = %d is negative", n_send); return TICTAC_ERR_BAD_CSR; }
    if (n_send > 0 && !send_ids) { set_error("send_ids is NULL"); return TICTAC_ERR_NULL; }
    if (order_stride != 0 && order_stride != d->R) {
        set_error("order_stride = %d, expected 0 or n_recv = %d", order_stride, d->R);
        return TICTAC_ERR_BAD_ORDER;
    }
    hipStream_t s = (hipStream_t)stream;
    rc = ensure_send_tables(d, n_send, send_ids, s);
    if (rc != TICTAC_OK) return rc;
    if (B == 0) return TICTAC_OK;
    if (d->R > 0 && !order) { set_error("order is NULL"); return TICTAC_ERR_NULL; }
    if (!makespan || !eff) { set_error("makespan or eff is NULL"); return TICTAC_ERR_NULL; }
    if (d->n == 0) {
        SimArgs a0{B, order, order_stride, op_time, recv_time, makespan, eff, U, L, S};
        HIP_TRY(launch_simulate(*d, a0, s));        // the empty graph: nothing to send
        return TICTAC_OK;
    }
    SimArgs a{B, order, order_stride, op_time, recv_time, makespan, eff, U, L, S};
    HIP_TRY(launch_check_orders(*d, B, order, order_stride, s));
    const hipError_t e = launch_simulate_sends(*d, a, s);
    if (e == hipErrorNotSupported) {
        set_error("%d ops and %d recvs: the per-sample state of the iteration with send ops does not fit LDS", d->n, d->R);
        return TICTAC_ERR_UNSUPPORTED;
    }
    HIP_TRY(e);
    return TICTAC_OK;
} TT_CATCH

int tictac_straggler_effect(int32_t B, int32_t w, const double *makespan, double *straggler, tictac_stream stream)
try {
    if (B < 0) { set_error("B = %d is negative", B); return TICTAC_ERR_UNSUPPORTED; }
    if (w < 1) { set_error("w = %d, expected at least 1", w); return TICTAC_ERR_UNSUPPORTED; }
    if (B / w == 0) return TICTAC_OK;
    if (!makespan || !straggler) { set_error("makespan or straggler is NULL"); return TICTAC_ERR_NULL; }
    HIP_TRY(launch_straggler(B, w, makespan, straggler, (hipStream_t)stream));
    return TICTAC_OK;
} TT_CATCH

int tictac_time_oracle_min(int32_t n_runs, int64_t n, const double *runs, double *time, tictac_stream stream)
try {
    if (n_runs < 1) { set_error("n_runs = %d, expected at least 1", n_runs); return TICTAC_ERR_UNSUPPORTED; }
    if (n < 0) { set_error("n is negative"); return TICTAC_ERR_UNSUPPORTED; }
    if (n == 0) return TICTAC_OK;
    if (!runs || !time) { set_error("runs or time is NULL"); return TICTAC_ERR_NULL; }
    HIP_TRY(launch_time_oracle_min(n_runs, n, runs, time, (hipStream_t)stream));
    return TICTAC_OK;
} TT_CATCH

int tictac_order_search(const tictac_dag *dag, int32_t B, const int32_t *order, int32_t order_stride,
                        int32_t n_moves, const int32_t *moves, const double *op_time, const double *recv_time,
                        int32_t *best_order, double *best_makespan, double *start_makespan, int32_t *n_accepted,
                        tictac_stream stream)
try {
    if (!dag) { set_error("dag is NULL"); return TICTAC_ERR_NULL; }
    Dag *d = const_cast<Dag *>(reinterpret_cast<const Dag *>(dag));
    int rc = check_batch(d, B, op_time, recv_time);
    if (rc != TICTAC_OK) return rc;
    if (n_moves < 0) { set_error("n_moves = %d is negative", n_moves); return TICTAC_ERR_UNSUPPORTED; }
    if (order_stride != 0 && order_stride != d->R) {
        set_error("order_stride = %d, expected 0 or n_recv = %d", order_stride, d->R);
        return TICTAC_ERR_BAD_ORDER;
    }
    if (d->R == 0) { set_error("the graph has no recv: there is nothing to order"); return TICTAC_ERR_UNSUPPORTED; }
    if (d->R > 512 || d->C > 512) {
        set_error("%d recvs and %d classes: the order search handles at most 512 of each", d->R, d->C);
        return TICTAC_ERR_UNSUPPORTED;
    }
    if (B == 0) return TICTAC_OK;
    if (!order) { set_error("order is NULL"); return TICTAC_ERR_NULL; }
    if (n_moves > 0 && !moves) { set_error("moves is NULL"); return TICTAC_ERR_NULL; }
    if (!best_order || !best_makespan) { set_error("best_order or best_makespan is NULL"); return TICTAC_ERR_NULL; }
    SearchArgs a{B, order, order_stride, n_moves, moves, op_time, recv_time, best_order, best_makespan,
                 start_makespan, n_accepted};
    HIP_TRY(launch_check_orders(*d, B, order, order_stride, (hipStream_t)stream));
    const hipError_t e = launch_order_search(*d, a, (hipStream_t)stream);
    if (e == hipErrorNotSupported) {
        set_error("graph outside what the order search handles");
        return TICTAC_ERR_UNSUPPORTED;
    }
    HIP_TRY(e);
    return TICTAC_OK;
} TT_CATCH

const char *tictac_last_error(void) { return g_err; }

const char *tictac_version(void) { return "0.1"; }

}  // extern "C"
