// flb_small.h -- lattices small enough to live in one block's LDS
// (flb_small.hip).
#pragma once

#include "flb_corr_internal.h"

namespace flbdev {

// One site per thread of a block, and sides short enough for direct sums: a
// sample of 32 x 32 takes 6.4 us in its block against 17 for the row and
// column kernels, one of 512 x 2 52 against 13.  The rule looks at a lattice
// alone, so that its sums are the same bits alone and in any batch.
constexpr int kSmallSites = 1024, kSmallSide = 64;
inline bool small_lattice(int nx, int ny)
{
    return nx <= kSmallSide && ny <= kSmallSide && nx * ny <= kSmallSites;
}
// Steps per call from which small lattices step resident: up to three steps
// are one launch of the other kernels, which start faster (32 x 32, one step
// per call: 6.4 against 8 us); from four on 1.1 us a step against 2.7.
constexpr int kResidentMin = 4;

// LDS of a lattice's block, with or without samples, with or without the
// sums beside them.
int small_lds_bytes(int nx, int ny, bool sampled, bool moments, bool keep_sums);

// nsteps steps of the nlat lattices listed (in place in v.pops[v.cur], one
// block of `threads` >= sites each), with a sample of their state before
// them if sample_first, and after every step that reaches a time divisible
// by `every` (0: none).  keep_sums: the sums stay in LDS from the first
// sample of the launch to its end.
hipError_t launch_small(const DeviceView &v, const int32_t *lattices, int nlat, int threads,
                        int lds_bytes, uint32_t nsteps, uint32_t every,
                        bool sample_first, bool keep_sums, bool noise, bool moments,
                        hipStream_t s);

}  // namespace flbdev
