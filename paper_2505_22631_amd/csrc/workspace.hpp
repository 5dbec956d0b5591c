// workspace.hpp -- growth of a cached workspace with a part that a call can do
// without.  Host code without HIP calls; the allocator is the caller's.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace oim {

struct Workspace {
    void* ptr = nullptr;
    size_t bytes = 0;
    size_t refused = SIZE_MAX;  // smallest size that could not be had
};

// Room for `base` bytes in w and for `extra` more if they can be had (kept:
// whether they are there; extra = 0 asks for none).  A size that was refused
// is not asked for again, nor a larger one, and a workspace that covers `base`
// is given up only for a larger one that is there: a call that has to do
// without the extra part then neither frees nor allocates, which would make
// it wait for the device.  alloc(size, &ptr): 0, kRefused (out of memory) or
// another error, which is returned; release(ptr) waits for the work that uses
// it.
constexpr int kRefused = 1;

template <class Alloc, class Release>
int grow_workspace(Workspace& w, size_t base, size_t extra, bool& kept, Alloc alloc,
                   Release release) {
    const size_t full = base + extra;
    kept = extra > 0;
    if (w.bytes >= full) return 0;
    if (w.bytes < base && w.ptr) {
        release(w.ptr);
        w.ptr = nullptr;
        w.bytes = 0;
    }
    if (kept && full < w.refused) {
        void* p = nullptr;
        const int st = alloc(full, &p);
        if (st == 0) {
            if (w.ptr) release(w.ptr);
            w.ptr = p;
            w.bytes = full;
            return 0;
        }
        if (st != kRefused) return st;
        w.refused = full;
    }
    kept = false;
    if (w.bytes >= base) return 0;
    const int st = alloc(base, &w.ptr);
    if (st == 0) w.bytes = base;
    else w.ptr = nullptr;
    return st;
}

}  // namespace oim
