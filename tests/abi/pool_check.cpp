// The pool of device blocks on a device of the host (stub/hip/hip_runtime.h): prints "ok" or the first thing that is wrong.
#include "../../paper_1802_02422_amd/csrc/pool.hpp"

#include <cstdio>
#include <new>

static bool no_new = false;
void *operator new(size_t n)
{
    if (no_new) {
        std::puts("operator new");
        std::exit(1);
    }
    return std::malloc(n);
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }

using namespace ivf;

#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)

// a block through the pool and back
static int once(DevPool &pool, size_t bytes)
{
    void *p = nullptr;
    size_t got = 0;
    int dev = -1;
    if (pool.take(&p, &got, &dev, bytes) != hipSuccess) return 1;
    pool.give(p, got, dev);
    return 0;
}

// an allocation that has no room beside the idle blocks gets theirs, one that has none at all fails and leaves NULL
static int idle_blocks_make_room()
{
    DevPool pool;
    FakeDevice &d = fake();
    d.room = 1 << 20;
    CHECK(!once(pool, 600000));
    CHECK(d.used == 600000);
    void *p = nullptr;
    CHECK(pool.fresh(&p, 900000) == hipSuccess && p && d.used == 900000);
    void *q = &d;
    CHECK(pool.fresh(&q, 900000) == hipErrorOutOfMemory && !q);
    hipFree(p);
    CHECK(!once(pool, 600000) && pool.fresh(&p, 500000) == hipSuccess && d.used == 500000);
    hipFree(p);
    CHECK(d.used == 0);
    return 0;
}

// a block larger than the pool may hold is freed, and the ones that are held stay
static int large_blocks_leave_the_others()
{
    DevPool pool;
    FakeDevice &d = fake();
    d.room = (size_t)8 << 30;
    CHECK(!once(pool, 1000000) && !once(pool, 5000000));
    const int frees = d.frees;
    CHECK(!once(pool, POOL_BYTES + 1) && d.frees == frees + 1 && d.used == 6000000);
    const int mallocs = d.mallocs;
    CHECK(!once(pool, 1000000) && !once(pool, 5000000) && d.mallocs == mallocs);
    // more than fits: the oldest go
    CHECK(!once(pool, POOL_BYTES - 5500000) && d.used == POOL_BYTES - 500000);
    pool.trim(0);
    CHECK(d.used == 0);
    return 0;
}

// no memory of the host is asked for (a container that grows throws where there is none, out of a destructor), however many
// blocks come back; devices do not share them
static int many_blocks_and_devices()
{
    DevPool pool;
    FakeDevice &d = fake();
    void *p[200];
    size_t got[200];
    int dev[200];
    for (int i = 0; i < 200; ++i) CHECK(pool.take(&p[i], &got[i], &dev[i], 4096) == hipSuccess);
    no_new = true;
    for (int i = 0; i < 200; ++i) pool.give(p[i], got[i], dev[i]);
    no_new = false;
    CHECK(d.live.size() > 0 && d.live.size() < 200);
    const int mallocs = d.mallocs;
    d.current = 1;
    CHECK(!once(pool, 4096) && d.mallocs == mallocs + 1);
    pool.trim(0);
    CHECK(d.live.size() == 1);
    pool.trim(1);
    CHECK(d.used == 0);
    d.current = 0;
    return 0;
}

int main()
{
    if (idle_blocks_make_room() || large_blocks_leave_the_others() || many_blocks_and_devices()) return 1;
    std::puts("ok");
    return 0;
}
