// The grid of a kernel that numbers its workgroups of 256 in one run.  A grid dimension holds fewer
// than 2^32 work-items, 2^24 such workgroups; a call of more takes several rows of 2^23, and the
// surplus workgroups of the last row leave at once.  (Plain C++: a host program can include it.)
#pragma once

namespace coopt {

constexpr unsigned kGridRow = 1u << 23;

struct Grid {
    unsigned x, y;
};

constexpr Grid grid_of(long long workgroups)
{
    return workgroups <= kGridRow ? Grid{(unsigned)workgroups, 1u}
                                  : Grid{kGridRow, (unsigned)((workgroups + kGridRow - 1) / kGridRow)};
}

// A workgroup's number from its place in that grid.
constexpr long long grid_index(unsigned x, unsigned y) { return x + (long long)kGridRow * y; }

}  // namespace coopt
