// Prints what the multiplication's host entry answers to arguments whose derived fields belong to other arguments.
#include "../paper_1704_04313_amd/csrc/kernels.h"

#include <cstdio>

using namespace cbk;

static char memory[64];

static GemmArgs layer(int streams, int height, int width, bool dilate)
{
    GemmArgs a{};
    a.dtype = kF32;
    a.x = a.wt = a.out = memory;
    a.bias = a.partial = reinterpret_cast<float *>(memory);
    a.tickets = reinterpret_cast<int *>(memory);
    a.sel_map = a.upd_out = reinterpret_cast<uint64_t *>(memory);
    a.kh = a.kw = 3;
    a.pad = a.stride = 1;
    a.S = streams;
    a.H = height; a.W = a.Wo = width; a.N = a.No = height * width;
    a.M = a.Mpad = a.Ms = a.pix_words = 64;
    a.Kpad = 9 * 64;
    a.max_pixels = streams * a.No;
    a.zero_word = a.max_pixels * a.pix_words;
    a.sel_words = a.sel_in_words = (a.max_pixels + 63) / 64;
    a.sel_dilate = dilate;
    a.grid = 8;
    gemm_set_divisors(a);
    return a;
}

static void answer(const char *name, const GemmArgs &a) { printf("%s %d\n", name, (int)gemm_gather(nullptr, a)); }

int main()
{
    const GemmArgs rows = layer(2, 10, 84, true), plain = layer(2, 10, 84, false);
    GemmArgs a = rows;
    answer("unchanged", a);
    a.sel_dilate = 0; // ranked by rows, picked from as if not
    answer("dilate_off", a);
    a = plain;
    a.sel_dilate = 1;
    answer("dilate_on", a);
    a = plain;
    a.sel_words += 1;
    answer("more_words", a);
    a = rows;
    a.max_pixels -= a.Wo;
    answer("fewer_rows", a);
    a = rows;
    a.sel_ranked = 1 << 20;
    answer("ranking_beyond_lds", a);
    a = layer(2, 2, 50, true); // two streams of a map lower than the filter, then one: the zero unit lies before the last tap
    a.S = 1;
    a.zero_word = a.N * a.pix_words;
    answer("fewer_streams", a);
    a = plain; // no longer whole slices per tap, the other divisors made anew
    a.pad = 0;
    a.kw = 33;
    a.dKw = make_fastdiv(33);
    answer("wider_filter", a);
    return 0;
}
