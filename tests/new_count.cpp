// operator new that counts the allocations whose call lies in libhr.so while
// counting is on, for a process that loads this library first.
#include <dlfcn.h>

#include <atomic>
#include <cstdlib>
#include <cstring>
#include <new>

static std::atomic<bool> on{false};
static std::atomic<long> hits{0};
extern "C" long new_count(int count)
{
    on = count != 0;
    return hits.load();
}

void* operator new(std::size_t n)
{
    Dl_info at;
    if (on && dladdr(__builtin_return_address(0), &at) && at.dli_fname &&
        std::strstr(at.dli_fname, "libhr.so"))
        ++hits;
    void* p = std::malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
