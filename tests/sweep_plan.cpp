// sweep_plan.cpp -- TEST INFRASTRUCTURE: the library's choice of a sweep's shape
// (pencils, chunks, zones per chunk, LDS stride), for tests that have to know
// which path they run.
#include "ppmlr_march.hpp"

extern "C" void sweep_plan(const int n[3], int axis, int elem, int trace, int learned, int wrap, int pencils, int out[4])
{
    const ppmlr::Sweep s = {{n[0], n[1], n[2]}, axis, elem, trace != 0, learned != 0, wrap != 0};
    const ppmlr::March m = ppmlr::sweep_shape(s, pencils);
    out[0] = m.P;
    out[1] = m.C;
    out[2] = m.L;
    out[3] = m.SM;
}
