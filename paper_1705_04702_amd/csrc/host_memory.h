// host_memory.h -- device blocks that a context keeps for its next call, and
// pinned host memory through which results are copied to and from a caller's
// ordinary arrays.
//
// What this replaces: a hipMalloc and a hipFree on each call, and pageable copies,
// which the runtime stages piece by piece.  The copy through pinned slots is left
// with the caller's array itself (its fresh pages, one pass of stores): 50 MB of
// FP32 pixels to 100 MB of FP64 take 5.5 ms against 10.4.  The calling thread alone
// does it: helper threads halved that again in an idle process, but lost all of it
// where a program's other threads (a numerical library's, still spinning after their
// own work) had the CPUs.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <cstring>
#include <memory>
#include <mutex>
#include <vector>

namespace mcrt {

// Device blocks of one context that are free to be used again.  All work of a
// context runs on its one stream, so a block's next user is ordered behind its
// last.  Kept up to kIdleBytes; freed with the context, or when any allocation of
// the library finds no memory left on the device.
class DevicePool {
  public:
    static std::shared_ptr<DevicePool> make(int device)
    {
        auto pool = std::make_shared<DevicePool>(device);
        All &all = every();
        std::lock_guard<std::mutex> lock(all.mu);
        all.pools.erase(std::remove_if(all.pools.begin(), all.pools.end(),
                                       [](const std::weak_ptr<DevicePool> &w) { return w.expired(); }),
                        all.pools.end());
        all.pools.push_back(pool);
        return pool;
    }

    // Memory of the current device, `device`: where it has none left, the idle
    // blocks of all contexts on it are freed first.
    static hipError_t allocate(int device, void **p, size_t bytes)
    {
        hipError_t e = hipMalloc(p, bytes);
        if (e != hipSuccess && drain_all(device)) {
            (void)hipGetLastError();
            e = hipMalloc(p, bytes);
        }
        if (e != hipSuccess) *p = nullptr;
        return e;
    }

    explicit DevicePool(int device) : device_(device) { idle_.reserve(kIdleBlocks); }
    ~DevicePool() { close(); }
    DevicePool(const DevicePool &) = delete;
    DevicePool &operator=(const DevicePool &) = delete;

    int device() const { return device_; }

    // A block of at least `bytes` bytes; *cap is its size.
    hipError_t get(size_t bytes, void **p, size_t *cap)
    {
        bytes = (std::max<size_t>(bytes, 1) + 4095) / 4096 * 4096;
        {
            std::lock_guard<std::mutex> lock(mu_);
            size_t best = idle_.size();
            for (size_t i = 0; i < idle_.size(); ++i)
                if (idle_[i].cap >= bytes && idle_[i].cap <= 2 * bytes + (64u << 10) &&
                    (best == idle_.size() || idle_[i].cap < idle_[best].cap))
                    best = i;
            if (best < idle_.size()) {
                *p = idle_[best].p;
                *cap = idle_[best].cap;
                idle_bytes_ -= idle_[best].cap;
                idle_[best] = idle_.back();
                idle_.pop_back();
                return hipSuccess;
            }
        }
        *cap = bytes;
        return allocate(device_, p, bytes);
    }

    void put(void *p, size_t cap)
    {
        {
            std::lock_guard<std::mutex> lock(mu_);
            if (!closed_ && idle_.size() < kIdleBlocks && idle_bytes_ + cap <= kIdleBytes) {
                idle_.push_back({p, cap}); // within the reserve
                idle_bytes_ += cap;
                return;
            }
        }
        (void)hipFree(p);
    }

    // The context is gone: blocks still in use are freed when they come back.
    void close()
    {
        {
            std::lock_guard<std::mutex> lock(mu_);
            closed_ = true;
        }
        (void)drain();
    }

  private:
    struct Block {
        void *p;
        size_t cap;
    };
    static constexpr size_t kIdleBlocks = 32, kIdleBytes = size_t(1) << 30;

    struct All {
        std::mutex mu;
        std::vector<std::weak_ptr<DevicePool>> pools;
    };
    static All &every()
    {
        static All *all = new All; // outlives any context
        return *all;
    }

    static bool drain_all(int device)
    {
        std::vector<std::shared_ptr<DevicePool>> pools;
        {
            All &all = every();
            std::lock_guard<std::mutex> lock(all.mu);
            for (const std::weak_ptr<DevicePool> &w : all.pools)
                if (std::shared_ptr<DevicePool> pool = w.lock())
                    if (pool->device_ == device) pools.push_back(std::move(pool));
        }
        bool any = false;
        for (const std::shared_ptr<DevicePool> &pool : pools) any = pool->drain() || any;
        return any;
    }

    bool drain()
    {
        std::lock_guard<std::mutex> lock(mu_);
        if (idle_.empty()) return false;
        (void)hipSetDevice(device_);
        for (const Block &b : idle_) (void)hipFree(b.p);
        idle_.clear();
        idle_bytes_ = 0;
        return true;
    }

    const int device_;
    std::mutex mu_;
    std::vector<Block> idle_;
    size_t idle_bytes_ = 0;
    bool closed_ = false;
};

// Pinned host memory of a device, shared by its contexts and freed with the
// last of them: cells for small results, which kernels write directly, and
// slots for the chunks of large copies (one copy at a time; a second caller
// takes the runtime's own way).
class Staging {
  public:
    static constexpr size_t kCellBytes = size_t(64) << 10, kSlotBytes = size_t(512) << 10;
    static constexpr int kCells = 4, kSlots = 8;

    static std::shared_ptr<Staging> of(int device)
    {
        static std::mutex mu;
        static std::vector<std::weak_ptr<Staging>> all;
        std::lock_guard<std::mutex> lock(mu);
        if ((size_t)device >= all.size()) all.resize((size_t)device + 1);
        std::shared_ptr<Staging> s = all[(size_t)device].lock();
        if (!s) {
            s = std::make_shared<Staging>(device);
            all[(size_t)device] = s;
        }
        return s;
    }

    explicit Staging(int device) : device_(device) {}
    ~Staging()
    {
        (void)hipSetDevice(device_);
        for (hipEvent_t ev : events_)
            if (ev) (void)hipEventDestroy(ev);
        if (cells_) (void)hipHostFree(cells_);
        if (slots_) (void)hipHostFree(slots_);
    }
    Staging(const Staging &) = delete;
    Staging &operator=(const Staging &) = delete;

    // A small piece of pinned memory (kCellBytes), or none.
    class Cell {
      public:
        explicit Cell(Staging *s) : s_(s)
        {
            if (!s_) return;
            std::lock_guard<std::mutex> lock(s_->mu_);
            if (!s_->cells_ && !s_->no_cells_) {
                if (hipHostMalloc((void **)&s_->cells_, kCells * kCellBytes, hipHostMallocDefault) != hipSuccess) {
                    (void)hipGetLastError();
                    s_->cells_ = nullptr;
                    s_->no_cells_ = true;
                }
            }
            if (!s_->cells_) return;
            for (int i = 0; i < kCells && at_ < 0; ++i)
                if (!(s_->used_ >> i & 1u)) {
                    s_->used_ |= 1u << i;
                    at_ = i;
                }
        }
        ~Cell()
        {
            if (at_ < 0) return;
            std::lock_guard<std::mutex> lock(s_->mu_);
            s_->used_ &= ~(1u << at_);
        }
        Cell(const Cell &) = delete;
        Cell &operator=(const Cell &) = delete;
        explicit operator bool() const { return at_ >= 0; }
        void *data() const { return s_->cells_ + (size_t)at_ * kCellBytes; }

      private:
        Staging *s_;
        int at_ = -1;
    };

    // Copies `bytes` bytes of device memory to the host in chunks: use(chunk,
    // offset, length) takes each while the next ones arrive.  `done` tells
    // whether it was done (else nothing was: no pinned memory, or another copy
    // under way).
    template <typename Use>
    hipError_t download(const void *src, size_t bytes, hipStream_t st, bool &done, Use use)
    {
        std::unique_lock<std::mutex> lock(copy_, std::try_to_lock);
        done = lock.owns_lock() && ready();
        if (!done) return hipSuccess;
        const size_t n = (bytes + kSlotBytes - 1) / kSlotBytes;
        auto length = [&](size_t c) { return std::min(kSlotBytes, bytes - c * kSlotBytes); };
        hipError_t e = hipSuccess;
        size_t sent = 0;
        for (size_t c = 0; c < n && e == hipSuccess; ++c) {
            for (; sent < n && sent < c + kSlots && e == hipSuccess; ++sent) {
                e = hipMemcpyAsync(slot(sent), (const char *)src + sent * kSlotBytes, length(sent),
                                   hipMemcpyDeviceToHost, st);
                if (e == hipSuccess) e = hipEventRecord(events_[sent % kSlots], st);
            }
            if (e == hipSuccess) e = hipEventSynchronize(events_[c % kSlots]);
            if (e == hipSuccess) use((const void *)slot(c), c * kSlotBytes, length(c));
        }
        if (e != hipSuccess) (void)hipStreamSynchronize(st); // no copy into a slot outlives this call
        return e;
    }

    // The other direction, from ordinary host memory.
    hipError_t upload(void *dst, const void *src, size_t bytes, hipStream_t st, bool &done)
    {
        std::unique_lock<std::mutex> lock(copy_, std::try_to_lock);
        done = lock.owns_lock() && ready();
        if (!done) return hipSuccess;
        const size_t n = (bytes + kSlotBytes - 1) / kSlotBytes;
        hipError_t e = hipSuccess;
        for (size_t c = 0; c < n && e == hipSuccess; ++c) {
            const size_t len = std::min(kSlotBytes, bytes - c * kSlotBytes);
            if (c >= kSlots) e = hipEventSynchronize(events_[c % kSlots]);
            if (e != hipSuccess) break;
            std::memcpy(slot(c), (const char *)src + c * kSlotBytes, len);
            e = hipMemcpyAsync((char *)dst + c * kSlotBytes, slot(c), len, hipMemcpyHostToDevice, st);
            if (e == hipSuccess) e = hipEventRecord(events_[c % kSlots], st);
        }
        const hipError_t idle = hipStreamSynchronize(st); // no copy out of a slot outlives this call
        return e == hipSuccess ? idle : e;
    }

  private:
    char *slot(size_t c) const { return slots_ + c % kSlots * kSlotBytes; }

    bool ready()
    {
        if (slots_) return true;
        if (no_slots_) return false;
        no_slots_ = true; // one attempt
        for (hipEvent_t &ev : events_)
            if (hipEventCreateWithFlags(&ev, hipEventDisableTiming) != hipSuccess) {
                (void)hipGetLastError();
                ev = nullptr;
                return false;
            }
        if (hipHostMalloc((void **)&slots_, kSlots * kSlotBytes, hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            slots_ = nullptr;
            return false;
        }
        return true;
    }

    const int device_;
    std::mutex mu_, copy_;
    char *cells_ = nullptr, *slots_ = nullptr;
    bool no_cells_ = false, no_slots_ = false;
    unsigned used_ = 0;
    hipEvent_t events_[kSlots] = {};
};

// Whether p is ordinary host memory, which the runtime does not know.  Memory that
// it allocated for the host may still be the target of a copy on a stream, so a
// copy from it has its place on the stream, and the host does not read it before;
// and one copy fills it at the link's rate, where chunks through other pinned memory
// and the calling thread take twice as long (32 MB: 0.62 against 1.49 ms).
inline bool ordinary(const void *p)
{
    hipPointerAttribute_t a{};
    if (hipPointerGetAttributes(&a, p) != hipSuccess) {
        (void)hipGetLastError();
        return true;
    }
    return a.type == hipMemoryTypeUnregistered;
}

// Whether p is memory that only the host uses (the runtime does not know it)
// or that was allocated as host memory.
inline bool on_host(const void *p)
{
    hipPointerAttribute_t a{};
    if (hipPointerGetAttributes(&a, p) != hipSuccess) {
        (void)hipGetLastError();
        return true;
    }
    return a.type == hipMemoryTypeHost || a.type == hipMemoryTypeUnregistered;
}

} // namespace mcrt
