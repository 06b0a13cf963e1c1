// gd_share.hpp -- how workgroups share a run's work over the dies: plain
// index arithmetic, the same on the host and the device (no HIP types, so
// that it can be compiled and checked on its own).
#pragma once

#include <stdint.h>

namespace gd {

constexpr int kXcd = 8;  // accelerator dies, each with its own L2

// first item of die x's contiguous range of `nitems`
constexpr int32_t xcd_range_lo(int x, int32_t nitems)
{
    return (nitems / kXcd) * x + (x < nitems % kXcd ? x : nitems % kXcd);
}

// The entries of a list of nl that workgroup id of nb takes: first, first +
// step, ... below end.  Every entry is taken by exactly one workgroup,
// whatever nb >= 1.
struct ListShare {
    int32_t first, end, step;
};

constexpr ListShare list_share(int64_t id, int64_t nb, int32_t nl)
{
    // each die's workgroups take a contiguous range; with fewer workgroups
    // than dies some ranges would have none, so they stride over the list
    if (nb < kXcd) return ListShare{int32_t(id), nl, int32_t(nb)};
    const int x = int(id % kXcd);
    return ListShare{xcd_range_lo(x, nl) + int32_t(id / kXcd), xcd_range_lo(x + 1, nl),
                     int32_t((nb - x + kXcd - 1) / kXcd)};
}

}  // namespace gd
