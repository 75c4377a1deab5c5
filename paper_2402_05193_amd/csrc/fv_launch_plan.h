// fv_launch_plan.h -- host arithmetic of launches: how a problem is cut into workgroups
// within the launch limit.  Plain C++, no HIP.
#pragma once

namespace fv {

// A HIP launch has at most 2^32 - 1 threads (blocks x threads of a block).
constexpr long long max_blocks(int threads) { return ((1ll << 32) - 1) / threads; }

// Shortest z chunk with which a stage launch of `tiles` tile columns over nz planes stays
// within the limit (nz if none does).
inline int shortest_zchunk(long long tiles, int nz, int threads)
{
    const long long chunks = max_blocks(threads) / tiles;
    if (chunks < 1) return nz;
    return (int)((nz + chunks - 1) / chunks);
}

// ---- the adjoint of the right-hand side (fv_adjoint.hip)
constexpr int ADJ_NT = 256;    // threads of a workgroup
constexpr int ADJ_CELLS = 64;  // longest piece of a line in one workgroup

// pieces of a line: all of it when periodic and short, else equal pieces of at most
// ADJ_CELLS cells (of 32 or more when there are several, so that a boundary's three halo
// positions and their mirror images lie in one piece); slots = positions per line.  A line
// of one cell is taken as periodic: without halo its cell is one slot instead of eight (an
// open boundary repeats the cell, symmetry needs three).
struct AdjointSplit {
    int pieces, slots, lines;  // per line; per piece; lines of a workgroup
    bool closed;               // the line closes on itself
};

inline AdjointSplit adjoint_split(int n, bool periodic)
{
    AdjointSplit s;
    s.closed = n == 1 || (periodic && n <= ADJ_CELLS + 7);
    s.pieces = s.closed ? 1 : (n + ADJ_CELLS - 1) / ADJ_CELLS;
    s.slots = s.closed ? n : (n + s.pieces - 1) / s.pieces + 7;
    s.lines = ADJ_NT / s.slots;
    return s;
}

// workgroups of `lines` lines
inline long long adjoint_blocks(const AdjointSplit& s, long long lines)
{
    return (lines + s.lines - 1) / s.lines * s.pieces;
}

}  // namespace fv
