// The handles' pinned buffers on the CPU: the library's host source with the HIP calls
// that make and free them replaced by counting ones.
//
//   pinned
//       prints "NAME made M freed F live L" after each of a few sequences of handles
//       made and released, by one thread and by several
#include "fdtd_host.cpp"

#include <cstdlib>
#include <thread>

namespace fdtd {
int field_step_occupancy(int, int, bool) { return 1; }
int field_step2_occupancy(int, bool) { return 1; }
int field_step2_material_occupancy(int, int, bool) { return 1; }
}  // namespace fdtd

static std::atomic<int> g_made{0}, g_freed{0};
static bool g_refuse = false;

extern "C" {
hipError_t hipHostMalloc(void** p, size_t n, unsigned)
{
    if (g_refuse) return hipErrorOutOfMemory;
    *p = malloc(n);
    ++g_made;
    return hipSuccess;
}
hipError_t hipHostFree(void* p)
{
    free(p);
    ++g_freed;
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t*, unsigned) { return hipSuccess; }
}

static void* some_alloc(size_t, void*) { return nullptr; }
static void some_free(void*, void*) {}

static fdtd_grid* make(int nx, int ny, bool callers)
{
    fdtd_grid* g = new fdtd_grid();
    g->d.nx = nx;
    g->d.ny = ny;
    g->pitch = row_pitch(nx);
    if (callers) {
        g->d.dev_alloc = some_alloc;
        g->d.dev_free = some_free;
    }
    if (make_pin(g) != hipSuccess) {
        delete g;
        return nullptr;
    }
    // the whole buffer is the handle's: a shared one would be overwritten by another
    memset(g->pin, (int)(uintptr_t)g & 0xff, kPinHead + 2 * g->pin_room);
    return g;
}

static bool release(fdtd_grid* g)
{
    bool own = g->pin_half <= g->pin_room;
    for (size_t q = 0; q < kPinHead + 2 * g->pin_half; ++q) own &= (uint8_t)g->pin[q] == ((uintptr_t)g & 0xff);
    give_pin(g->device, g->pin_room, g->pin, !g->d.dev_free);
    delete g;
    return own;
}

static void report(const char* name)
{
    printf("%s made %d freed %d live %d\n", name, g_made.load(), g_freed.load(), g_made - g_freed);
    fflush(stdout);
    g_made = g_freed = 0;
}

int main()
{
    // one after another, memory from the caller's allocator: one buffer, never freed
    for (int q = 0; q < 10; ++q)
        if (!release(make(48, 43, true))) return 3;
    report("in_turn_callers");
    // the last of several handles, its own memory from hipMalloc: all freed
    {
        fdtd_grid* a = make(48, 43, true);
        fdtd_grid* b = make(300, 420, false);      // a plane of 539 KB: halves of 1 MiB, as below
        fdtd_grid* c = make(310, 420, false);
        bool ok = release(c);
        fdtd_grid* d = make(320, 500, false);
        ok &= release(a) && release(d) && release(b);
        if (!ok) return 3;
    }
    report("several_sizes");
    // more than are kept
    {
        std::vector<fdtd_grid*> gs;
        for (int q = 0; q < 150; ++q) gs.push_back(make(1048, 792, true));   // 4 MiB each
        for (fdtd_grid* g : gs)
            if (!release(g)) return 3;
    }
    report("many_large");
    if (!release(make(48, 43, false))) return 3;
    report("given_back");
    // no memory: refused, and counted out again
    g_refuse = true;
    if (make(48, 43, false)) return 4;
    g_refuse = false;
    if (!release(make(48, 43, false))) return 3;
    report("refused");
    // several threads
    {
        std::vector<std::thread> ts;
        std::atomic<bool> ok{true};
        for (int t = 0; t < 8; ++t)
            ts.emplace_back([&ok, t] {
                for (int q = 0; q < 50; ++q) {
                    fdtd_grid* a = make(48 + 100 * (t % 3), 43, (q + t) & 1);
                    fdtd_grid* b = make(900, 43 + 20 * t, q & 1);
                    if (!release(a) || !release(b)) ok = false;
                }
            });
        for (std::thread& t : ts) t.join();
        if (!ok) return 3;
    }
    if (!release(make(48, 43, false))) return 3;
    report("threads");
    return 0;
}
