// Workspace growth (csrc/workspace.hpp) against an allocator of limited size:
// prints "ok", or the line that failed.
#include <cstdio>
#include <cstdlib>
#include <map>

#include "workspace.hpp"

using oim::grow_workspace;
using oim::kRefused;
using oim::Workspace;

static size_t g_room = 0, g_used = 0;
static int g_allocs = 0, g_frees = 0, g_error = 0;
static std::map<void*, size_t> g_live;

static int take(size_t n, void** p) {
    ++g_allocs;
    if (g_error) return g_error;
    if (g_used + n > g_room) return kRefused;
    *p = malloc(n ? n : 1);
    g_live[*p] = n;
    g_used += n;
    return 0;
}

static void give(void* p) {
    ++g_frees;
    g_used -= g_live.at(p);
    g_live.erase(p);
    free(p);
}

#define CHECK(c)                                                   \
    do {                                                           \
        if (!(c)) {                                                \
            std::printf("line %d: %s\n", __LINE__, #c);            \
            return 1;                                              \
        }                                                          \
    } while (0)

int main() {
    bool kept = false;
    auto grow = [&](Workspace& w, size_t base, size_t extra) {
        g_allocs = g_frees = 0;
        return grow_workspace(w, base, extra, kept, take, give);
    };
    {   // room for all: one allocation, then none
        Workspace w;
        g_room = 1000;
        CHECK(grow(w, 100, 300) == 0 && kept && w.bytes == 400 && g_allocs == 1);
        CHECK(grow(w, 100, 300) == 0 && kept && g_allocs == 0 && g_frees == 0);
        CHECK(grow(w, 350, 0) == 0 && !kept && g_allocs == 0);
        CHECK(grow(w, 500, 100) == 0 && kept && w.bytes == 600 && g_frees == 1);
        give(w.ptr);
    }
    {   // the extra part is refused once: later calls neither free nor allocate
        Workspace w;
        g_room = 350;
        CHECK(grow(w, 100, 300) == 0 && !kept && w.bytes == 100 && g_allocs == 2);
        void* held = w.ptr;
        for (int k = 0; k < 3; ++k)
            CHECK(grow(w, 100, 300) == 0 && !kept && w.ptr == held && g_allocs == 0 && g_frees == 0);
        CHECK(grow(w, 90, 320) == 0 && !kept && w.ptr == held && g_allocs == 0);  // larger than refused
        // smaller than what was refused: asked for, beside the workspace
        CHECK(grow(w, 100, 200) == 0 && !kept && w.ptr == held && g_allocs == 1 && g_frees == 0);
        CHECK(grow(w, 100, 100) == 0 && kept && w.bytes == 200 && g_allocs == 1 && g_frees == 1);
        give(w.ptr);
    }
    {   // a workspace too small for base is given up first
        Workspace w;
        g_room = 500;
        CHECK(grow(w, 300, 0) == 0 && w.bytes == 300);
        CHECK(grow(w, 400, 90) == 0 && kept && w.bytes == 490 && g_frees == 1 && g_allocs == 1);
        CHECK(grow(w, 495, 90) == 0 && !kept && w.bytes == 495 && g_frees == 1 && g_allocs == 2);
        CHECK(grow(w, 600, 0) == kRefused && w.ptr == nullptr && w.bytes == 0);
        CHECK(grow(w, 200, 0) == 0 && w.bytes == 200);
        give(w.ptr);
    }
    {   // any other error comes back, with the workspace as it was
        Workspace w;
        g_room = 500;
        CHECK(grow(w, 100, 0) == 0);
        g_error = -1;
        CHECK(grow(w, 100, 100) == -1 && w.ptr && w.bytes == 100);
        g_error = 0;
        CHECK(grow(w, 100, 100) == 0 && kept);
        give(w.ptr);
    }
    CHECK(g_live.empty() && g_used == 0);
    std::printf("ok\n");
    return 0;
}
