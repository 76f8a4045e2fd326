// The small boards' kernel choice on the CPU: pick_brick of the library's brick source,
// compiled for the host alone.
//
//   brick_pick CUS NX NY NZ [NX NY NZ ...]
//       one line per board: "rows planes" that a brick owns, "0 0" for the marching kernel
#include "fdtd_kernels_brick.hip"

#include <cstdio>
#include <cstdlib>

int main(int argc, char** argv)
{
    for (int a = 2; a + 2 < argc; a += 3) {
        const int q = fdtd::pick_brick(atoi(argv[a]), atoi(argv[a + 1]), atoi(argv[a + 2]), atoi(argv[1]));
        int rows = 0, planes = 0;
        if (q >= 0) fdtd::brick_owned(q, &rows, &planes);
        printf("%d %d\n", rows, planes);
    }
    return 0;
}
