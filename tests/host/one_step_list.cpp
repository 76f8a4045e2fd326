// The work list of a one-step shape (but 64 x 15), on the CPU.
//
//   one_step_list NX NY NZ TX ROWS SLOTS
//       one line "tx ty kb ke" per entry of each XCD's run in order ("idle" for padding)
#include "fdtd_host.cpp"

#include <cstdlib>

namespace fdtd {
int field_step_occupancy(int, int, bool) { return 1; }
int field_step2_occupancy(int, bool) { return 1; }
int field_step2_material_occupancy(int, int, bool) { return 1; }
}  // namespace fdtd

int main(int, char** argv)
{
    std::vector<TileRef> whole, out;
    board_tiles(0, atoi(argv[1]), atoi(argv[2]), atoi(argv[3]), atoi(argv[4]), atoi(argv[5]), whole);
    build_work(whole, atoi(argv[6]), out, true);
    for (const TileRef& t : out) {
        if (t.board < 0)
            printf("idle\n");
        else
            printf("%d %d %d %d\n", t.tx, t.ty, t.kb, t.ke);
    }
    return 0;
}
