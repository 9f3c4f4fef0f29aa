// Prints whether launches multiply in halves: a line for each "cin cout kernel outputs positions" read, on 256 compute units.
#include "../paper_1704_04313_amd/csrc/kernels.h"

#include <cstdio>

using namespace cbk;

int main()
{
    int cin, cout, k, outputs, positions;
    while (scanf("%d %d %d %d %d", &cin, &cout, &k, &outputs, &positions) == 5) {
        GemmArgs a{};
        a.dtype = kF32;
        a.M = cout;
        const int bm = gemm_channel_tile(cout), step = gemm_k_multiple(kF32);
        a.Mpad = (cout + bm - 1) / bm * bm;
        a.Kpad = (k * k * ((cin + 3) / 4 * 4) + step - 1) / step * step;
        a.max_pixels = outputs;
        a.halves_range = gemm_halves_range(a.Kpad, k * k * cin);
        a.grid = gemm_grid(a, 256);
        printf("%d\n", (int)gemm_takes_halves(a, positions));
    }
    return 0;
}
