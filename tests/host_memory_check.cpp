// CPU check of host_memory.h on the stub device (hipstub): prints the line that failed.
#include "host_memory.h"

#include <cstdio>

using mcrt::DevicePool;

#define CHECK(x)                                             \
    do {                                                     \
        if (!(x)) return std::printf("%d: %s\n", __LINE__, #x), 1; \
    } while (0)

int main()
{
    const size_t MB = size_t(1) << 20;
    auto a = DevicePool::make(0), b = DevicePool::make(0), other = DevicePool::make(1);
    void *p = nullptr, *q = nullptr, *r = nullptr;
    size_t cp = 0, cq = 0, cr = 0;
    CHECK(a->get(MB, &p, &cp) == hipSuccess && b->get(MB, &q, &cq) == hipSuccess && other->get(MB, &r, &cr) == hipSuccess);
    a->put(p, cp);
    other->put(r, cr);
    CHECK(stub().used == 3 * MB); // idle blocks stay

    // an allocation outside the pools gets the idle blocks of its device, and no others
    void *x = nullptr;
    CHECK(DevicePool::allocate(0, &x, 2 * MB) == hipSuccess && x);
    CHECK(stub().used == 4 * MB && stub().blocks.count(q) && stub().blocks.count(r) && !stub().blocks.count(p));
    // nothing idle on the device any more: the error stays an error
    void *y = &cp;
    CHECK(DevicePool::allocate(0, &y, MB) == hipErrorOutOfMemory && !y);
    CHECK(DevicePool::allocate(1, &y, MB) == hipSuccess && !stub().blocks.count(r)); // device 1 had one
    CHECK(hipFree(y) == hipSuccess);

    // a pool gets another pool's idle blocks too
    b->put(q, cq);
    CHECK(hipFree(x) == hipSuccess && stub().used == MB);
    CHECK(a->get(4 * MB, &p, &cp) == hipSuccess && cp == 4 * MB && stub().used == 4 * MB);
    // a pool that is closed keeps nothing; one that is gone is not asked
    a->close();
    a->put(p, cp);
    CHECK(stub().used == 0);
    CHECK(b->get(3 * MB, &q, &cq) == hipSuccess);
    b->put(q, cq);
    b.reset();
    CHECK(stub().used == 0 && DevicePool::allocate(0, &x, 4 * MB) == hipSuccess && hipFree(x) == hipSuccess);
    std::puts("ok");
    return 0;
}
