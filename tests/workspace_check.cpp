// The library's device memory (workspace.cpp) against a device of a few MiB that
// exists only here: each check is a function named on the command line.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <thread>

#include "internal.h"

namespace {
std::mutex mu;
std::map<void *, size_t> live;
size_t used = 0, capacity = 0;
int mallocs = 0;
}  // namespace

extern "C" {
hipError_t hipMalloc(void **p, size_t n)
{
    std::lock_guard<std::mutex> lk(mu);
    mallocs++;
    if (used + n > capacity)
        return hipErrorOutOfMemory;
    *p = std::malloc(16);
    live[*p] = n;
    used += n;
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    std::lock_guard<std::mutex> lk(mu);
    used -= live.at(p);
    live.erase(p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void *p) { return hipFree(p); }
hipError_t hipHostGetDevicePointer(void **d, void *p, unsigned)
{
    *d = p;
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipMemGetInfo(size_t *f, size_t *t)
{
    std::lock_guard<std::mutex> lk(mu);
    *f = capacity - used;
    *t = capacity;
    return hipSuccess;
}
hipError_t hipMemset2DAsync(void *, size_t, int, size_t, size_t, hipStream_t) { return hipSuccess; }
}

namespace hub {
[[noreturn]] void fail(int code, const std::string &msg) { throw Error{code, msg}; }
void hip_check(hipError_t e, const char *what)
{
    if (e != hipSuccess)
        fail(HUBBARD_ENOMEM, what);
}
}  // namespace hub

using namespace hub;

static void need(bool ok, const char *what)
{
    if (!ok) {
        std::printf("failed: %s\n", what);
        std::exit(1);
    }
}

constexpr size_t M = 1 << 20;

// what idle handles keep makes room for any allocation of the library
static void others_make_room()
{
    capacity = 64 * M;
    Workspace a, b;
    { DevBuf x(24 * M, &a), y(24 * M, &b); }
    need(used == 48 * M, "both blocks are kept");
    { DevBuf x(40 * M, &a); }  // neither fits nor is there room beside them
    need(used == 40 * M, "the other handle's block went");
    { DevBuf plain(60 * M); }
    need(used == 0, "a buffer of no handle frees every kept block");
    { PinnedBuf h(M, &b); }
    { DevBuf x(30 * M, &a); }
    need(used == 31 * M, "kept again");
    { PinnedBuf h(60 * M); }
    need(used == 0, "pinned memory too");
    { DevBuf x(24 * M, &a); }
    (void)hipFree(device_alloc(50 * M));
    need(used == 0, "tables and work rows too");
    int code = 0;
    try {
        DevBuf x(65 * M, &a);
    } catch (const Error &e) {
        code = e.code;
    }
    need(code == HUBBARD_ENOMEM, "more than the device has is still refused");
}

// a handle freed leaves no trace, and blocks in use are never taken
static void lifetimes()
{
    capacity = 64 * M;
    auto a = std::make_unique<Workspace>();
    Workspace b;
    { DevBuf x(16 * M, a.get()); }
    DevBuf held(16 * M, &b);
    a.reset();
    need(used == 16 * M, "freed with its handle");
    int code = 0;
    try {
        DevBuf x(60 * M, &b);
    } catch (const Error &e) {
        code = e.code;
    }
    need(code == HUBBARD_ENOMEM && used == 16 * M && live.count(held.p), "a buffer in use stays");
}

// what all handles keep is bounded, and the oldest block goes first, whosever it is
static void bound()
{
    constexpr size_t G = (size_t)1 << 30;
    capacity = 64 * G;
    Workspace a, b;
    { DevBuf x(3 * G, &a); }
    { DevBuf x(2 * G, &b); }
    { DevBuf x(G, &a); }
    need(used == 6 * G, "one handle may keep most of it");
    const int before = mallocs;
    { DevBuf x(3 * G, &a), y(2 * G, &b), z(G, &a); }
    need(mallocs == before && used == 6 * G, "a repeated call allocates nothing");
    // the order of giving back is now z, y, x
    { DevBuf x(4 * G, &b); }
    need(used == 4 * G + 3 * G, "the oldest two went: a's gigabyte and b's two");
    { DevBuf x(9 * G, &b); }
    need(used == 7 * G, "more than the bound is not kept");
    { DevBuf x(3 * G, &a); }
    need(used == 7 * G, "a's three are still there");
}

// handles that take turns share what they keep, on one device
static void turns()
{
    capacity = 64 * 1024 * M;
    std::vector<std::unique_ptr<Workspace>> w;
    for (int k = 0; k < 24; k++)
        w.emplace_back(new Workspace);
    for (int round = 0; round < 3; round++)
        for (auto &x : w)
            DevBuf a(900 * M, x.get()), b(800 * M, x.get()), c(3 * M, x.get());
    need(mallocs == 3, "one call's blocks serve all of them");
    w[0]->device = w[1]->device = 1;  // (they keep nothing)
    { DevBuf a(900 * M, w[0].get()); }
    need(mallocs == 4, "a block of the other device does not");
    { DevBuf a(900 * M, w[1].get()); }
    need(mallocs == 4, "its own does");
    w.clear();
    need(used == 0, "freed with the handles");
}

// several threads whose handles take, give and run out at once
static void threads()
{
    capacity = 40 * M;
    std::vector<std::thread> t;
    for (int k = 0; k < 8; k++)
        t.emplace_back([k] {
            for (int i = 0; i < 400; i++) {
                Workspace w;
                for (size_t n = 1; n <= 4; n++) {
                    try {
                        DevBuf x((size_t)(1 + (k + i) % 5) * n * M, &w), y(M, &w);
                        PinnedBuf h(64 << 10, &w);
                    } catch (const Error &e) {
                        need(e.code == HUBBARD_ENOMEM, "only out of memory");
                    }
                }
            }
        });
    for (auto &x : t)
        x.join();
    need(used == 0 && live.empty(), "everything is freed");
}

// a resident basis grows on what its handle keeps, and on what others do, where
// the device itself has less than a chunk and the 2 GiB left free
static void basis()
{
    constexpr size_t G = (size_t)1 << 30;
    capacity = 3 * G;
    Workspace a, b;
    auto grow = [&](size_t vectors, size_t vb, size_t limit) {
        BasisPool p;
        p.ws = &a;
        p.vb = vb;
        p.pitch = p.pad_off = vb;
        p.rows = 1;
        for (size_t j = 0; j < vectors; j++)
            if (!p.reserve(j, limit, nullptr))
                return j;
        return vectors;
    };
    const size_t vb = 16 * M, chunk = kBasisChunk * vb;  // chunks of 512 MiB: two fit
    need(grow(200, vb, 10 * G) == 64, "two chunks, then less than 2 GiB would be left");
    need(used == 2 * chunk, "both are kept");
    void *outside = device_alloc(G + 3 * G / 4);  // another program's memory: 256 MiB left
    need(grow(200, vb, 10 * G) == 64, "the kept chunks serve the next run");
    need(grow(200, vb, chunk + 1) == 32, "within the handle's limit");
    (void)hipFree(outside);
    a.release();
    { DevBuf x(G, &b); }  // another handle's kept gigabyte
    need(grow(200, vb, 10 * G) == 64, "counts as free");
    a.release();
    outside = device_alloc(G);
    need(grow(200, vb, 10 * G) == 0, "no kept chunk, less than 2 GiB beside one");
    (void)hipFree(outside);
}

int main(int argc, char **argv)
{
    const std::map<std::string, void (*)()> all = {
        {"others_make_room", others_make_room}, {"lifetimes", lifetimes}, {"threads", threads},
        {"basis", basis},
        {"bound", bound},
        {"turns", turns}};
    need(argc == 2 && all.count(argv[1]), "a check's name");
    all.at(argv[1])();
    std::printf("ok\n");
    return 0;
}
