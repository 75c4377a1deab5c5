// C entry points of the launch arithmetic (csrc/fv_launch_plan.h) for test_launch_plan.py.
#include "fv_launch_plan.h"

extern "C" {
int plan_shortest_zchunk(long long tiles, int nz, int threads) { return fv::shortest_zchunk(tiles, nz, threads); }
int plan_max_adjoint_blocks() { return (int)fv::max_blocks(fv::ADJ_NT); }
// split[4] = {pieces, slots, lines, closed}; returns the workgroups of `lines` lines
long long plan_adjoint(int n, int periodic, long long lines, int* split)
{
    const fv::AdjointSplit s = fv::adjoint_split(n, periodic != 0);
    split[0] = s.pieces;
    split[1] = s.slots;
    split[2] = s.lines;
    split[3] = s.closed;
    return fv::adjoint_blocks(s, lines);
}
}
