// Which kernel fdtd_step_n launches, on the CPU: the library's host source and its
// choice of bricks, on a device of 256 compute units whose memory is host memory and
// whose launches are only counted.
//
//   routes
//       one line "NAME B|M ..." per sequence of calls: bricks or the marching kernel
#define launch_brick launch_brick_on_the_device
#include "fdtd_kernels_brick.hip"
#undef launch_brick
#include "fdtd_host.cpp"

#include <cstdlib>

static int g_bricks = 0, g_marches = 0, g_singles = 0, g_device = 0;
static bool g_recording = false;

namespace fdtd {
int num_shapes() { return 1; }
void shape_at(int, int* tx, int* ty) { *tx = 64; *ty = 15; }
int num_shapes2() { return 2; }
void shape2_at(int q, int* tx, int* ty) { *tx = 64; *ty = q ? 10 : 14; }
int field_step_occupancy(int, int, bool) { return 1; }
int field_step2_occupancy(int, bool) { return 1; }
int field_step2_material_occupancy(int, int, bool) { return 1; }
hipError_t noalloc_scratch(int, void** p) { *p = nullptr; return hipSuccess; }
hipError_t launch_fill_zero(float* p, int64_t n, hipStream_t) { memset(p, 0, (size_t)n * 4); return hipSuccess; }
hipError_t launch_advance_one(int64_t*, int64_t, int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_field_step(int, int, const BoardDev*, const TileRef*, int, int, int, bool, hipStream_t)
{
    ++g_singles;
    return hipSuccess;
}
hipError_t launch_field_step2(int, const BoardDev*, const TileRef*, int, int, int, bool, bool, bool, hipStream_t)
{
    ++g_marches;
    return hipSuccess;
}
hipError_t launch_brick(int, const BoardDev&, int, int, bool, bool, hipStream_t)
{
    ++g_bricks;
    return hipSuccess;
}
hipError_t launch_pack(const void*, int, int64_t, uint32_t, uint32_t, uint32_t, double, void*, const int32_t* bad,
                       int32_t* bad_out, hipStream_t)
{
    if (bad_out) *bad_out = *bad;
    return hipSuccess;
}
hipError_t launch_fft(const float*, int64_t, int, double2*, double*, double*, const int32_t* bad, int32_t* bad_out,
                      hipStream_t)
{
    if (bad_out) *bad_out = *bad;
    return hipSuccess;
}
}  // namespace fdtd

extern "C" {
hipError_t hipGetDevice(int* d) { *d = g_device; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) { *p = malloc(n); return hipSuccess; }
hipError_t hipFree(void* p) { free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = malloc(n); return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t)
{
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)1; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s)
{
    *s = g_recording ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)1; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t)1; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }
}

static void must(int e)
{
    if (e == FDTD_OK) return;
    printf("failed %d %s\n", e, fdtd_last_error());
    exit(3);
}

static fdtd_grid* board(int nx, int ny, int nz)
{
    fdtd_grid_desc d{};
    d.nx = nx;
    d.ny = ny;
    d.nz = nz;
    d.dx = d.dy = 1e-3;
    d.dz = 0.4e-3;
    d.max_steps = 1 << 16;
    fdtd_grid* g = nullptr;
    must(fdtd_create_grid(&d, &g));
    std::vector<float> eps((size_t)nx * ny * nz, 1.0f);
    must(fdtd_set_materials(g, eps.data(), nullptr));
    int id;
    must(fdtd_add_probe(g, nx / 2, ny / 2, nz / 2, &id));
    return g;
}

static void step(fdtd_grid* g, int64_t n = 2)
{
    g_bricks = g_marches = g_singles = 0;
    must(fdtd_step_n(g, n));
    const bool ok = g_bricks + g_marches == n / 2 && (g_bricks == 0 || g_marches == 0) && g_singles == n % 2;
    printf(" %s", !ok ? "?" : g_bricks ? "B" : "M");
}

int main()
{
    fdtd_grid* g[5];
    for (fdtd_grid*& h : g) h = board(48, 43, 30);
    auto name = [](const char* n) { printf("%s", n); };
    auto end = [] { printf("\n"); };

    name("alone");
    for (int64_t n : {2, 3, 100, 4097}) step(g[0], n);
    end();
    name("three_at_once");          // the third and all later ones while none is waited for
    for (int r = 0; r < 2; ++r)
        for (int q = 0; q < 3; ++q) step(g[q], r ? 64 : 7);
    end();
    name("waited_for");             // each of the calls that wait ends a handle's share
    float probe[8];
    std::vector<float> field((size_t)49 * 44 * 31);
    std::vector<double> re(65537), im(65537);
    std::vector<char> image((size_t)fdtd_state_bytes(g[1]));
    double ms;
    int64_t launches;
    for (int how = 0; how < 8; ++how) {
        step(g[0]);
        step(g[1]);
        step(g[2]);
        for (int q = 0; q < 2; ++q) {
            switch (how) {
                case 0: must(fdtd_synchronize(g[q])); break;
                case 1: must(fdtd_get_probe(g[q], 0, probe, 2)); break;
                case 2: must(fdtd_get_field(g[q], FDTD_EZ, field.data())); break;
                case 3: must(fdtd_get_plane(g[q], FDTD_EZ, 3, field.data())); break;
                case 4: must(fdtd_probe_fft(g[q], 0, 32768, re.data(), im.data())); break;
                case 5: must(fdtd_set_field(g[q], FDTD_EZ, field.data())); break;
                case 6: must(fdtd_get_timing(g[q], &ms, &launches)); break;
                default:
                    must(fdtd_save_state(g[q], image.data(), (int64_t)image.size()));
                    must(fdtd_load_state(g[q], image.data(), (int64_t)image.size()));
            }
        }
        step(g[2]);                 // alone with steps enqueued: bricks
        must(fdtd_synchronize(g[2]));
    }
    end();
    name("recorded");               // marches, and counts for nothing
    g_recording = true;
    step(g[0]);
    step(g[1]);
    g_recording = false;
    step(g[2]);
    step(g[0]);
    end();
    name("other_device");
    g_device = 1;
    fdtd_grid* far[2] = {board(48, 43, 30), board(48, 43, 30)};
    g_device = 0;
    step(far[0]);
    step(far[1]);
    must(fdtd_synchronize(g[2]));
    step(g[0]);
    step(g[1]);
    end();
    name("released");               // a handle that goes takes its share along
    step(g[2]);
    must(fdtd_destroy_grid(g[1]));
    must(fdtd_destroy_grid(far[0]));
    must(fdtd_destroy_grid(far[1]));
    step(g[2]);
    must(fdtd_synchronize(g[0]));
    must(fdtd_synchronize(g[2]));
    end();
    // boards of every kind, the last of five stepping at once
    const int sizes[][3] = {{48, 43, 30}, {40, 30, 20}, {60, 60, 30}, {64, 40, 60}, {56, 24, 100}, {112, 40, 30},
                            {28, 100, 28}, {80, 72, 37}, {130, 60, 40}, {300, 300, 40}};
    for (const int* s : sizes) {
        printf("crowd_%dx%dx%d", s[0], s[1], s[2]);
        fdtd_grid* c = board(s[0], s[1], s[2]);
        step(c);
        must(fdtd_synchronize(c));
        step(g[0]);
        step(g[2]);
        step(c);
        must(fdtd_destroy_grid(c));
        must(fdtd_synchronize(g[0]));
        must(fdtd_synchronize(g[2]));
        end();
    }
    name("left");
    printf(" %d\n", g_stepping[0].load());
    return 0;
}
