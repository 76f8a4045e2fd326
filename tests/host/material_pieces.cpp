// Which kernels' pieces boards with rebuilt coefficients run, alone and in one batched
// call, on the CPU.
//
//   material_pieces CUS BOARDS NX NY NZ KB KE [NX NY NZ KB KE ...]
//       BOARDS copies of each board whose tiles all need the material arithmetic on node
//       planes KB..KE-1; per board "alone" lines and then "batch" lines, each
//       "alone|batch kernel board tx ty kb ke" (kernel: plain, conduct, tall or short)
#include "fdtd_host.cpp"

#include <cstdlib>

namespace fdtd {
int field_step_occupancy(int, int, bool) { return 1; }
int field_step2_occupancy(int, bool) { return 1; }
int field_step2_material_occupancy(int, int, bool) { return 1; }
}  // namespace fdtd

int main(int argc, char** argv)
{
    static const char* kKernel[5] = {"", "plain", "conduct", "tall", "short"};
    std::vector<std::unique_ptr<fdtd_grid>> hs;
    std::vector<fdtd_grid*> gs;
    for (int a = 3; a + 4 < argc; a += 5)
        for (int copy = 0; copy < atoi(argv[2]); ++copy) {
            auto g = std::make_unique<fdtd_grid>();
            g->d.nx = atoi(argv[a]);
            g->d.ny = atoi(argv[a + 1]);
            g->d.nz = atoi(argv[a + 2]);
            g->cus = atoi(argv[1]);
            g->mat = true;
            g->tile_x = 64;
            g->tile_y = kHybridTY;
            g->tile_steps = 2;
            int cx, cy;
            tile_counts(g->d.nx, g->d.ny, 64, owned_rows(kHybridTY, 2), &cx, &cy);
            const int stride = g->d.nz + 1;
            g->tile_need.assign((size_t)cx * cy * stride, 0);
            for (int t = 0; t < cx * cy; ++t)
                for (int k = atoi(argv[a + 3]); k < atoi(argv[a + 4]); ++k) g->tile_need[(size_t)t * stride + k] = 1;
            material_pieces(g.get());
            const int b = (int)hs.size();
            auto put = [&](const char* kernel, const std::vector<TileRef>& v) {
                for (const TileRef& t : v) printf("alone %s %d %d %d %d %d\n", kernel, b, t.tx, t.ty, t.kb, t.ke);
            };
            put("plain", g->pc_plain);
            put("conduct", g->pc_cd);
            put(g->mat_ty == kMatTY ? "short" : "tall", g->pc_rb);
            gs.push_back(g.get());
            hs.push_back(std::move(g));
        }
    const std::vector<int64_t> n(gs.size(), 2);
    RoundHost r;
    plan_round(gs.data(), (int)gs.size(), n.data(), r);
    for (const Span& sp : r.spans)
        for (int l = 0; l < sp.nl; ++l)
            for (int q = 0; q < sp.count[l]; ++q) {
                const TileRef& t = r.items[(size_t)sp.off[l] + q];
                if (t.board >= 0)
                    printf("batch %s %d %d %d %d %d\n", kKernel[sp.kind[l]], r.order[t.board], t.tx, t.ty, t.kb, t.ke);
            }
    return 0;
}
