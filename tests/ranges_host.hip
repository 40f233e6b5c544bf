// The kernels' host-and-device range arithmetic behind a C interface, for
// test_ranges.py: compiled for the host alone.
#include "../paper_1904_13342_amd/csrc/ranges.h"

extern "C" void cell_range_of(float X0, float Y0, float eX, float eY, int nx, int ny, int elem, int *first, int *last)
{
    ph::cell_range(X0, Y0, eX, eY, nx, ny, (size_t)elem, *first, *last);
}

extern "C" int sample_beyond_of(int m, int last, float bound, float at, float rate)
{
    return ph::sample_beyond(m, last, bound, at, rate);
}

extern "C" float clip_margin_of(float re_max) { return ph::clip_margin(re_max); }
