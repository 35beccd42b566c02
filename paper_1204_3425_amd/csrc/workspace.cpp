// Device and pinned host memory: the buffers that handles keep between their
// calls, and the allocations that may take them back.
#include <algorithm>
#include <atomic>
#include <exception>
#include <mutex>
#include <vector>

#include "internal.h"

namespace hub {

// bytes kept by all handles of the process, and blocks given back so far
static std::atomic<size_t> g_kept{0};
static std::atomic<uint64_t> g_given{0};

// Every workspace alive.  Taken before a workspace's own lock, never inside it.
struct Registry {
    std::mutex mu;
    std::vector<Workspace *> all;
};
static Registry &registry()
{
    static Registry *r = new Registry;  // outlives handles freed at exit
    return *r;
}

Workspace::Workspace()
{
    Registry &r = registry();
    std::lock_guard<std::mutex> lk(r.mu);
    r.all.push_back(this);
}

Workspace::~Workspace()
{
    {
        Registry &r = registry();
        std::lock_guard<std::mutex> lk(r.mu);
        r.all.erase(std::remove(r.all.begin(), r.all.end(), this), r.all.end());
    }
    release();
}

void release_kept()
{
    Registry &r = registry();
    std::lock_guard<std::mutex> lk(r.mu);
    for (Workspace *w : r.all)
        w->release();
}

static bool out_of_memory(hipError_t e) { return e == hipErrorOutOfMemory || e == hipErrorMemoryAllocation; }

void *device_alloc(size_t bytes)
{
    void *p = nullptr;
    hipError_t e = hipMalloc(&p, bytes);
    if (out_of_memory(e)) {
        (void)hipGetLastError();
        release_kept();
        e = hipMalloc(&p, bytes);
    }
    hip_check(e, "hipMalloc");
    return p;
}

void *host_alloc(size_t bytes)
{
    const unsigned flags = hipHostMallocMapped | hipHostMallocCoherent;
    void *p = nullptr;
    hipError_t e = hipHostMalloc(&p, bytes, flags);
    if (out_of_memory(e)) {
        (void)hipGetLastError();
        release_kept();
        e = hipHostMalloc(&p, bytes, flags);
    }
    hip_check(e, "hipHostMalloc");
    return p;
}

static size_t rounded(size_t bytes) { return (std::max<size_t>(bytes, 16) + 65535) / 65536 * 65536; }

void *Workspace::take_kept(size_t bytes, size_t *got)
{
    bytes = rounded(bytes);
    const size_t most = bytes < ((size_t)64 << 20) ? 2 * bytes : bytes + bytes / 4;
    if (void *p = take_own(bytes, most, got))
        return p;
    // small blocks are not worth a walk over the handles
    if (bytes < ((size_t)1 << 20) || g_kept.load() < bytes)
        return nullptr;
    Registry &r = registry();
    std::lock_guard<std::mutex> lk(r.mu);
    for (Workspace *w : r.all)
        if (w != this && w->device == device)
            if (void *p = w->take_own(bytes, most, got))
                return p;
    return nullptr;
}

void *Workspace::take_own(size_t bytes, size_t most, size_t *got)
{
    std::lock_guard<std::mutex> lk(mu_);
    size_t best = dev_.size();
    for (size_t k = 0; k < dev_.size(); k++)
        if (dev_[k].bytes >= bytes && dev_[k].bytes <= most &&
            (best == dev_.size() || dev_[k].bytes < dev_[best].bytes))
            best = k;
    if (best == dev_.size())
        return nullptr;
    const Block b = dev_[best];
    drop(best);
    *got = b.bytes;
    return b.p;
}

void *Workspace::take(size_t bytes, size_t *got)
{
    if (void *p = take_kept(bytes, got))
        return p;
    *got = rounded(bytes);
    return device_alloc(*got);
}

void Workspace::drop(size_t k)
{
    held_ -= dev_[k].bytes;
    g_kept -= dev_[k].bytes;
    dev_.erase(dev_.begin() + (std::ptrdiff_t)k);
}

void Workspace::give(void *p, size_t bytes)
{
    if (bytes > kKeepAll) {
        (void)hipFree(p);
        return;
    }
    {
        std::lock_guard<std::mutex> lk(mu_);
        dev_.push_back(Block{p, bytes, ++g_given});
        held_ += bytes;
        g_kept += bytes;
    }
    if (g_kept.load() <= kKeepAll)
        return;
    Registry &r = registry();
    std::lock_guard<std::mutex> lk(r.mu);
    while (g_kept.load() > kKeepAll) {
        Workspace *w = nullptr;
        uint64_t first = 0;
        for (Workspace *x : r.all) {
            const uint64_t age = x->oldest();
            if (age && (!w || age < first)) {
                w = x;
                first = age;
            }
        }
        if (!w)
            break;
        w->drop_oldest();
    }
}

uint64_t Workspace::oldest()
{
    std::lock_guard<std::mutex> lk(mu_);
    return dev_.empty() ? 0 : dev_.front().age;
}

void Workspace::drop_oldest()
{
    std::lock_guard<std::mutex> lk(mu_);
    if (dev_.empty())
        return;
    (void)hipFree(dev_.front().p);
    drop(0);
}

void *Workspace::take_host(size_t bytes, size_t *got)
{
    bytes = (bytes + 16383) / 16384 * 16384;
    {
        std::lock_guard<std::mutex> lk(mu_);
        for (size_t k = 0; k < host_.size(); k++)
            if (host_[k].bytes >= bytes) {
                void *p = host_[k].p;
                *got = host_[k].bytes;
                host_.erase(host_.begin() + (std::ptrdiff_t)k);
                return p;
            }
    }
    *got = bytes;
    return host_alloc(bytes);
}

void Workspace::give_host(void *p, size_t bytes)
{
    {
        std::lock_guard<std::mutex> lk(mu_);
        // one or two small blocks serve every call
        if (host_.size() < 2 && bytes <= (1 << 20)) {
            host_.push_back(Block{p, bytes, 0});
            return;
        }
    }
    (void)hipHostFree(p);
}

void Workspace::release()
{
    std::lock_guard<std::mutex> lk(mu_);
    for (const Block &b : dev_)
        (void)hipFree(b.p);
    for (const Block &b : host_)
        (void)hipHostFree(b.p);
    g_kept -= held_;
    dev_.clear();
    host_.clear();
    held_ = 0;
}

DevBuf::DevBuf(size_t n, Workspace *w) : ws(w)
{
    if (!n)
        return;
    bytes = n;
    if (ws)
        p = ws->take(n, &bytes);
    else
        p = device_alloc(n);
}

std::unique_ptr<DevBuf> DevBuf::kept(size_t n, Workspace *w)
{
    std::unique_ptr<DevBuf> b(new DevBuf());
    b->ws = w;
    if (w)
        b->p = w->take_kept(n, &b->bytes);
    if (!b->p)
        b.reset();
    return b;
}

DevBuf::~DevBuf()
{
    if (!p)
        return;
    if (!ws) {
        (void)hipFree(p);
        return;
    }
    // a call that ends in an error may have left work in flight
    if (std::uncaught_exceptions() > 0)
        (void)hipDeviceSynchronize();
    ws->give(p, bytes);
}

PinnedBuf::PinnedBuf(size_t n, Workspace *w) : bytes(n), ws(w)
{
    if (ws)
        p = ws->take_host(n, &bytes);
    else
        p = host_alloc(n);
    HUB_HIP(hipHostGetDevicePointer(&dev, p, 0));
}

PinnedBuf::~PinnedBuf()
{
    if (!p)
        return;
    if (!ws) {
        (void)hipHostFree(p);
        return;
    }
    if (std::uncaught_exceptions() > 0)
        (void)hipDeviceSynchronize();
    ws->give_host(p, bytes);
}

bool BasisPool::reserve(size_t j, size_t limit, hipStream_t s)
{
    const size_t cb = kBasisChunk * vb, spare = (size_t)2 << 30;
    auto read_free = [&] {
        size_t fr = 0, tot = 0;
        HUB_HIP(hipMemGetInfo(&fr, &tot));
        seen_free = true;
        free_left = fr;
        return fr >= cb + spare;
    };
    while (j >= capacity()) {
        if ((chunks.size() + 1) * cb > limit)
            return false;
        std::unique_ptr<DevBuf> c = DevBuf::kept(cb, ws);
        if (!c) {
            // (re)read the free memory; chunks of up to 1 GiB go by the last reading
            if ((cb > ((size_t)1 << 30) || !seen_free || free_left < cb + spare) && !read_free()) {
                release_kept();
                if (!read_free())
                    return false;
            }
            free_left -= cb;
            try {
                c.reset(new DevBuf(cb, ws));
            } catch (const Error &) {
                (void)hipGetLastError();
                return false;
            }
        }
        chunks.push_back(std::move(c));
        if (pitch > pad_off)
            HUB_HIP(hipMemset2DAsync(static_cast<char *>(chunks.back()->p) + pad_off, pitch, 0, pitch - pad_off,
                                     (size_t)rows * kBasisChunk, s));
    }
    return true;
}

}  // namespace hub
