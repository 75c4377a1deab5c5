// C entry points of the launch arithmetic (csrc/fv_launch_plan.h) for test_launch_plan.py.
#include "fv_launch_plan.h"

extern "C" {
int plan_shortest_zchunk(long long tiles, int nz, int threads) { return fv::shortest_zchunk(tiles, nz, threads); }
}
