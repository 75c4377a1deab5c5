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

}  // namespace fv
