// What the builders on the device share (internal): their working memory and the upload of A.
#ifndef SPMM_UPLOAD_H
#define SPMM_UPLOAD_H

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <condition_variable>
#include <cstring>
#include <mutex>
#include <thread>
#include <vector>

namespace builder {

typedef uint32_t upload_unit __attribute__((ext_vector_type(4)));

// A builder's working memory, in one piece (an allocation and its release cost 10 to 100 us each), and the
// stream it works on.  The memory is ordered by that stream: hipFree would wait for the work of all streams
// (4096 x 4096, 80 % pruned, with 100 ms of matrix products on another stream: created after 100 ms, now
// after 43, its kernels between theirs).  The calling thread's own stream waits for the null stream as every
// copy does, and there is none to create: a new one costs 0.15 ms of 1.3.
struct workshop {
    const hipStream_t stream = hipStreamPerThread;
    char *base = nullptr;
    size_t bytes = 0;
    ~workshop()
    {
        if (base && give_back() == hipSuccess) (void)hipStreamSynchronize(stream);
    }
    size_t reserve(size_t n)
    {
        const size_t at = bytes;
        bytes += (n + 255) & ~(size_t)255;
        return at;
    }
    hipError_t take() { return hipMallocAsync(reinterpret_cast<void **>(&base), bytes, stream); }
    // The device has the memory back after the stream's next synchronisation.
    hipError_t give_back()
    {
        char *p = base;
        base = nullptr;
        return hipFreeAsync(p, stream);
    }
    template <typename T> T *at(size_t offset) const { return reinterpret_cast<T *>(base + offset); }
};

// Pinned memory through which a builder uploads large matrices: the device reads it at 54 GB/s, ordinary memory at 28
// to 35.  Its first pages cost 0.1 ms per MiB once, and giving it back may wait for
// all streams, which a creation must not.  So there is one piece of it for the process, lent to one creation at
// a time (another one that runs meanwhile uploads from ordinary memory), and it goes back when the last plan on tiles or strips
// is released.  4096 x 4096, 80 % pruned (20 MB), plan on tiles and product in ms:
//                                 each plan released before the next   one lives    the first of a process (after a small plan)
//   three pieces of 2 MiB           0.90 (0.84 if the memory stayed)     0.80        1.95
//   three of 4                      0.88                                 0.77        2.35    (8192 x 4096, 30 %: 1.9 instead of 2.0)
//   four of 1                       0.96                                 0.85        1.7
//   from ordinary memory            1.26                                             2.2
struct staging_memory {
    static constexpr size_t PIECE = 2u << 20, PIECES = 3, WORDS = 256u << 10;  // pieces of the entries; what else a builder sends
    std::mutex lock;
    char *memory = nullptr;
    bool lent = false;
    int64_t plans = 0;  // on tiles and strips, alive
    char *lend()
    {
        const std::lock_guard<std::mutex> hold(lock);
        if (lent) return nullptr;
        if (!memory && hipHostMalloc(reinterpret_cast<void **>(&memory), PIECE * PIECES + WORDS, hipHostMallocPortable) != hipSuccess) {
            (void)hipGetLastError();
            memory = nullptr;
        }
        lent = memory != nullptr;
        return memory;
    }
    void take_back()  // (a creation that made a plan has counted it)
    {
        const std::lock_guard<std::mutex> hold(lock);
        lent = false;
        release_unused();
    }
    void count_plan(int64_t by)
    {
        const std::lock_guard<std::mutex> hold(lock);
        plans += by;
        release_unused();
    }

private:
    void release_unused()
    {
        if (plans > 0 || lent || !memory) return;
        (void)hipHostFree(memory);
        memory = nullptr;
    }
};
inline staging_memory staging;

// A copy from pinned memory that a kernel makes beside its own work (n = 0: none).
struct pull {
    const upload_unit *from = nullptr;
    upload_unit *to = nullptr;
    uint32_t n = 0;
};
constexpr unsigned PULL_BLOCKS = 128;  // of 256 threads
__device__ inline void run_pull(const pull &p, uint32_t block)
{
    for (uint32_t i = block * 256u + threadIdx.x; i < p.n; i += PULL_BLOCKS * 256u) p.to[i] = p.from[i];
}

// Copies from pinned memory, between a builder's kernels.  (With hipMemcpyAsync, whose engines and the kernels wait for each other,
// the creation below takes 0.2 ms longer.)
static __global__ __launch_bounds__(256) void pull_kernel(const upload_unit *from, upload_unit *to, uint32_t n)
{
    for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i < n; i += gridDim.x * 256u) to[i] = from[i];
}

// The columns and values on their way to the device.  Four threads and the caller fill the pinned memory, columns as 16-bit
// numbers where those hold them, and check the columns; each piece is copied when it is full, while the next ones
// are filled.  (4096 x 4096, 80 % pruned: 20 MB; the plan is made in 0.7 ms, with 27 MB from ordinary memory in 1.1.)
class uploader {
public:
    bool begin(int64_t K, const int32_t *col_idx, const float *vals, int64_t nnz, hipStream_t s)
    {
        stream = s;
        if (nnz < (1 << 19)) return false;  // 4 MB: nothing to gain
        size_t n_pieces = 0;
        narrow = K <= 65536;
        entry_bytes[0] = narrow ? 2 : 4;
        for (int kind = 0; kind < 2; ++kind) {
            const size_t most = staging_memory::PIECE / entry_bytes[kind];
            for (size_t at = 0; at < (size_t)nnz; at += most) pieces.push_back(piece{kind, at, std::min(most, (size_t)nnz - at)});
            if (kind == 0) column_pieces = pieces.size();
        }
        n_pieces = pieces.size();
        left = std::vector<std::atomic<int>>(n_pieces);
        for (size_t i = 0; i < n_pieces; ++i) left[i] = (int)parts(pieces[i]);
        for (hipEvent_t &e : copied)
            if (hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) {
                (void)hipGetLastError();
                e = nullptr;
                return false;
            }
        pinned = staging.lend();
        if (!pinned) return false;
        std::memset(flags(), 0, 64);
        columns = reinterpret_cast<const uint32_t *>(col_idx);
        values = vals;
        limit = (uint32_t)K;
        // (a thread takes 15 us to start: the first one starts the others)
        auto start = [this](int t, auto job) {
            try {
                helpers[t] = std::thread(job);
            } catch (...) {  // the others and the caller fill what is left
            }
        };
        start(0, [this, start] {
            for (int t = 1; t < HELPERS; ++t) start(t, [this] { help(); });
            help();
        });
        return true;
    }
    bool narrow_columns() const { return narrow; }
    // Copies the columns (kind 0) or the values (1) to `to`, whose size is a multiple of 16 bytes.
    hipError_t copy(int kind, char *to)
    {
        for (; next < (kind == 0 ? column_pieces : pieces.size()); ++next) {
            const piece &p = pieces[next];
            hipError_t e = await_next();
            if (e != hipSuccess) return e;
            hipLaunchKernelGGL(pull_kernel, dim3(128), dim3(256), 0, stream, reinterpret_cast<const upload_unit *>(place(next)),
                               reinterpret_cast<upload_unit *>(to + p.first * entry_bytes[kind]), (uint32_t)((p.count * entry_bytes[kind] + 15) / 16));
            e = hipEventRecord(copied[next % staging_memory::PIECES], stream);
            launched_pieces = next + 1;
            if (e == hipSuccess) e = look();
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    // The next piece of the values, when it is full, as a pull of the caller's, who says when that has been launched (none: n = 0).
    hipError_t next_values(char *to, pull &out)
    {
        out = pull();
        if (!pinned || next >= pieces.size() || pieces[next].kind != 1) return hipSuccess;
        const hipError_t e = await_next();
        if (e != hipSuccess) return e;
        const piece &p = pieces[next];
        out = pull{reinterpret_cast<const upload_unit *>(place(next)), reinterpret_cast<upload_unit *>(to + p.first * 4), (uint32_t)((p.count * 4 + 15) / 16)};
        ++next;
        return hipSuccess;
    }
    hipError_t launched()
    {
        for (; launched_pieces < next; ++launched_pieces) {
            const hipError_t e = hipEventRecord(copied[launched_pieces % staging_memory::PIECES], stream);
            if (e != hipSuccess) return e;
        }
        return look();
    }
    // Lets the helpers go on where copies have left room.
    hipError_t look()
    {
        while (pinned && usable.load() < pieces.size()) {
            const size_t oldest = usable.load() - staging_memory::PIECES;  // piece in the place that is wanted next
            if (oldest >= launched_pieces) break;
            const hipError_t e = hipEventQuery(copied[oldest % staging_memory::PIECES]);
            if (e == hipErrorNotReady) {
                (void)hipGetLastError();
                break;
            }
            if (e != hipSuccess) return e;
            one_more_usable();
        }
        return hipSuccess;
    }
    // Copies some words beside them, to memory of a multiple of 16 bytes.
    hipError_t copy_words(const std::vector<uint32_t> &words, uint32_t *to)
    {
        const size_t bytes = (words.size() * 4 + 15) / 16 * 16;
        if (!pinned || sent + bytes > staging_memory::WORDS - 64) return hipMemcpyWithStream(to, words.data(), words.size() * 4, hipMemcpyHostToDevice, stream);
        char *from = pinned + staging_memory::PIECE * staging_memory::PIECES + sent;
        sent += bytes;
        std::copy(words.begin(), words.end(), reinterpret_cast<uint32_t *>(from));
        hipLaunchKernelGGL(pull_kernel, dim3(16), dim3(256), 0, stream, reinterpret_cast<const upload_unit *>(from), reinterpret_cast<upload_unit *>(to), (uint32_t)(bytes / 16));
        return hipGetLastError();
    }
    // Words of pinned memory that a kernel may write, zero before; to be read when the stream has been waited for.
    uint32_t *flags() { return reinterpret_cast<uint32_t *>(pinned + staging_memory::PIECE * staging_memory::PIECES + staging_memory::WORDS - 64); }
    bool column_outside() const { return outside.load(); }  // after the columns' copies
    void arrived()  // the stream has been waited for
    {
        next = 0;
        sent = 0;
    }
    ~uploader()
    {
        {
            const std::lock_guard<std::mutex> hold(lock);
            stop.store(true);
        }
        changed.notify_all();
        for (std::thread &t : helpers)  // (the first one first)
            if (t.joinable()) t.join();
        if (pinned) {
            if (next > 0 || sent > 0) (void)hipStreamSynchronize(stream);
            staging.take_back();
        }
        for (hipEvent_t e : copied)
            if (e) (void)hipEventDestroy(e);
    }

private:
    struct piece {
        int kind;
        size_t first, count;  // entries
    };
    static constexpr size_t PART = 32u << 10;  // entries that a thread takes at a time
    static size_t parts(const piece &p) { return (p.count + PART - 1) / PART; }
    char *place(size_t i) const { return pinned + i % staging_memory::PIECES * staging_memory::PIECE; }
    void help()
    {
        while (!stop.load()) {
            if (fill_part()) continue;
            // Room comes every 45 us while the device copies, and a thread that sleeps may wake 100 us late.
            const auto until = std::chrono::steady_clock::now() + std::chrono::microseconds(300);
            auto nothing = [this] { return !stop.load() && fill_piece.load() < pieces.size() && fill_piece.load() >= usable.load(); };
            while (nothing() && std::chrono::steady_clock::now() < until) std::this_thread::yield();
            if (!nothing()) {
                if (fill_piece.load() == pieces.size()) return;
                continue;
            }
            std::unique_lock<std::mutex> hold(lock);
            changed.wait(hold, [this] { return stop.load() || fill_piece.load() == pieces.size() || fill_piece.load() < usable.load(); });
            if (fill_piece.load() == pieces.size()) return;
        }
    }
    void one_more_usable()
    {
        {
            const std::lock_guard<std::mutex> hold(lock);
            usable.fetch_add(1);
        }
        changed.notify_all();
    }
    // Fills with the others until the next piece is full.
    hipError_t await_next()
    {
        while (left[next].load(std::memory_order_acquire) > 0) {
            const hipError_t e = look();
            if (e != hipSuccess) return e;
            if (!fill_part()) std::this_thread::yield();
        }
        return hipSuccess;
    }
    // Fills one part; false if there is none, or no place for it yet.
    bool fill_part()
    {
        size_t i, k;
        {
            const std::lock_guard<std::mutex> hold(lock);
            i = fill_piece.load();
            if (i == pieces.size() || i >= usable.load()) return false;
            k = next_part++;
            if (next_part == parts(pieces[i])) {
                next_part = 0;
                fill_piece.store(i + 1);
                if (i + 1 == pieces.size()) changed.notify_all();
            }
        }
        const piece &p = pieces[i];
        const size_t at = k * PART, n = std::min(PART, p.count - at);
        char *to = place(i) + at * entry_bytes[p.kind];
        if (p.kind == 1) {
            std::memcpy(to, values + p.first + at, n * 4);
        } else {
            const uint32_t *from = columns + p.first + at;
            uint32_t beyond = 0;
            if (narrow) {
                uint16_t *out = reinterpret_cast<uint16_t *>(to);
                for (size_t x = 0; x < n; ++x) {
                    out[x] = (uint16_t)from[x];
                    beyond |= (uint32_t)(from[x] >= limit);
                }
            } else {
                uint32_t *out = reinterpret_cast<uint32_t *>(to);
                for (size_t x = 0; x < n; ++x) {
                    out[x] = from[x];
                    beyond |= (uint32_t)(from[x] >= limit);
                }
            }
            if (beyond) outside.store(true);
        }
        left[i].fetch_sub(1, std::memory_order_release);
        return true;
    }

    char *pinned = nullptr;
    size_t sent = 0;  // bytes of words
    hipStream_t stream = nullptr;
    hipEvent_t copied[staging_memory::PIECES] = {};  // the copy from each place
    const uint32_t *columns = nullptr;
    const float *values = nullptr;
    uint32_t limit = 0;
    bool narrow = false;
    size_t entry_bytes[2] = {4, 4};
    std::vector<piece> pieces;
    std::vector<std::atomic<int>> left;  // parts of each piece that are still to be filled
    size_t column_pieces = 0, next = 0, next_part = 0, launched_pieces = 0;  // launched_pieces: whose event is recorded
    std::mutex lock;
    std::condition_variable changed;  // fill_piece, usable or stop, for helpers that have nothing to fill
    std::atomic<size_t> fill_piece{0}, usable{staging_memory::PIECES};  // pieces below have a place in the memory
    std::atomic<bool> outside{false}, stop{false};
    static constexpr int HELPERS = 4;
    std::thread helpers[HELPERS];
};

}  // namespace builder

#endif
