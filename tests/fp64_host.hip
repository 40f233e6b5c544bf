// The kernels' FP64 helpers behind a C interface, for test_fp64.py: compiled
// for the host alone, with the estimate as an argument.
#include "../paper_1904_13342_amd/csrc/fp64.h"

extern "C" double rcp64_of(double x, double r) { return ph::rcp64_from(x, r); }
extern "C" double rsqrt64_of(double x, double r) { return ph::rsqrt64_from(x, r); }
extern "C" double div64_of(double n, double d) { return ph::div64(n, d, 1.0 / d); }
