// Bringing results to the host (read_out) on the CPU: the library's host source with
// a stream whose work runs only when it is waited for.
//
//   readout
//       random results through halves of random sizes: each comes back as stored,
//       the watchdog flag is the one of its time, and nothing is allocated on the way;
//       prints "trials T turns N wrong W allocations A"
#include "fdtd_host.cpp"

#include <cstdlib>
#include <memory>
#include <random>

static long g_allocs = 0;
static bool g_count = false;
void* operator new(size_t n)
{
    if (g_count) ++g_allocs;
    void* p = malloc(n ? n : 1);
    if (!p) abort();
    return p;
}
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }

struct Op {
    const void* src;
    int elem;
    int64_t pitch;
    uint32_t len, col, n;
    double scale;
    void* out;
    const int32_t* bad;
    int32_t* bad_out;
    hipEvent_t ev;   // a recorded event, nothing else
};
static Op g_ops[4096];
static int g_begin = 0, g_end = 0;
static long g_turns = 0;

static void run_op(const Op& o)
{
    if (o.ev) return;
    if (o.bad_out) *o.bad_out = *o.bad;
    for (uint32_t t = 0; t < o.n; ++t) {
        const int64_t at = (int64_t)((o.col + t) / o.len) * o.pitch + (o.col + t) % o.len;
        if (o.elem == 8)
            ((uint64_t*)o.out)[t] = ((const uint64_t*)o.src)[at];
        else if (o.scale == 1.0)
            ((uint32_t*)o.out)[t] = ((const uint32_t*)o.src)[at];
        else
            ((float*)o.out)[t] = (float)((double)((const float*)o.src)[at] * o.scale);
    }
}
static void push(const Op& o)
{
    if (g_begin == g_end) g_begin = g_end = 0;
    if (g_end == 4096) abort();
    g_ops[g_end++] = o;
}

namespace fdtd {
int field_step_occupancy(int, int, bool) { return 1; }
int field_step2_occupancy(int, bool) { return 1; }
int field_step2_material_occupancy(int, int, bool) { return 1; }
hipError_t launch_pack(const void* src, int elem, int64_t pitch, uint32_t len, uint32_t col, uint32_t n,
                       double scale, void* out, const int32_t* bad, int32_t* bad_out, hipStream_t)
{
    push(Op{src, elem, pitch, len, col, n, scale, out, bad, bad_out, nullptr});
    return hipSuccess;
}
}  // namespace fdtd

extern "C" {
hipError_t hipEventRecord(hipEvent_t e, hipStream_t)
{
    ++g_turns;
    push(Op{nullptr, 0, 0, 0, 0, 0, 0, nullptr, nullptr, nullptr, e});
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e)
{
    int last = -1;
    for (int q = g_begin; q < g_end; ++q)
        if (g_ops[q].ev == e) last = q;
    for (; g_begin <= last; ++g_begin) run_op(g_ops[g_begin]);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t)
{
    for (; g_begin < g_end; ++g_begin) run_op(g_ops[g_begin]);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind, hipStream_t)
{
    if (n != 4) abort();
    push(Op{src, 4, 1, 1, 0, 1, 1.0, dst, nullptr, nullptr, nullptr});
    return hipSuccess;
}
}

int main()
{
    std::mt19937 rng(5);
    auto upto = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
    long wrong = 0;
    const int trials = 3000;
    for (int t = 0; t < trials; ++t) {
        auto g = std::make_unique<fdtd_grid>();
        g->pin_half = 256u * upto(1, 12);
        std::vector<char> pin(kPinHead + 2 * g->pin_half, (char)0x5a);
        g->pin = pin.data();
        g->pin_ev[0] = (hipEvent_t)1;
        g->pin_ev[1] = (hipEvent_t)2;
        int32_t flag = upto(0, 1) ? upto(1, 9) : 0;
        g->bad_dev = &flag;
        const int npc = upto(0, 6);
        std::vector<Piece> pc(npc);
        std::vector<std::vector<char>> src(npc), got(npc), want(npc);
        for (int q = 0; q < npc; ++q) {
            Piece& p = pc[q];
            p.elem = upto(0, 1) ? 4 : 8;
            p.rows = upto(0, 9) ? upto(1, 40) : 0;
            p.len = upto(1, upto(0, 3) ? 40 : 700);
            p.pitch = p.len + (upto(0, 2) ? upto(0, 33) : 0);
            p.scale = p.elem == 4 && upto(0, 1) ? 1.0 / 376.73 : 1.0;
            const int64_t n = p.rows * p.len;
            src[q].resize((size_t)std::max<int64_t>(1, p.rows * p.pitch * p.elem));
            for (size_t b = 0; b + 4 <= src[q].size(); b += 4) {
                const float v = (float)((int)(rng() % 20001) - 10000) / 37.0f;
                memcpy(&src[q][b], &v, 4);
            }
            got[q].assign((size_t)n * p.elem + 8, (char)0x33);
            want[q] = got[q];
            p.src = src[q].data();
            p.out = got[q].data();
            for (int64_t e = 0; e < n; ++e) {
                const char* x = &src[q][(size_t)(e / p.len * p.pitch + e % p.len) * p.elem];
                if (p.scale == 1.0) {
                    memcpy(&want[q][(size_t)e * p.elem], x, (size_t)p.elem);
                } else {
                    float v;
                    memcpy(&v, x, 4);
                    v = (float)((double)v * p.scale);
                    memcpy(&want[q][(size_t)e * 4], &v, 4);
                }
            }
        }
        const bool ask = npc == 0 || upto(0, 1);
        int32_t bad = -1;
        g_count = true;
        const int e = read_out(g.get(), pc.data(), npc, ask ? &bad : nullptr);
        g_count = false;
        wrong += e != FDTD_OK || g_begin != g_end || (ask && bad != flag) || got != want;
        hipStreamSynchronize(nullptr);
    }
    printf("trials %d turns %ld wrong %ld allocations %ld\n", trials, g_turns, wrong, g_allocs);
    return 0;
}
