// Tiles of the values-only receiver (receiver_values.hip): which launches cover the rank tiles,
// what a wave owns and where its loads point. Plain integer arithmetic, shared by the kernel and
// its launch and compiled by itself in a host test.
#pragma once

#include <cstdint>

#ifdef __HIPCC__
#define CGTP_HD __host__ __device__
#else
#define CGTP_HD
#endif

namespace cgtp {

// A launch: waves of rt rank tiles x pt point tiles over the rank tiles [first, first + groups *
// rt). part: the last group may have fewer than rt, whose waves skip the ones they do not have.
struct RecvLaunch {
    int rt, pt, part, first, groups;
};

// The launches of a receiver pass over `tiles` rank tiles (at most two; returns how many). A wave
// takes as many rank tiles as there are, up to four: they share a recurrence. It holds eight
// tiles (rank x point), whose sums fill half of the registers of two waves per SIMD; four, two by
// two, with two node slots (twice the sums) or two coefficient sets (half; waves of four rank
// tiles took 4.6 -> 5.4 ms with two slots, 5,000 nodes, lmax 6, R = 128). Every wave has all of
// its tiles: they are cut into the fewest groups, whose sizes differ by one at most, and each
// size is a launch (80 ranks: a group of 3 tiles and one of 2). Skipping in the loop what a group
// of four lacks costs the others more than it saves (2,000 nodes, lmax 4, 32 channels, 27 edges
// a node, R = 80: 339 us; on zeros, 8 tiles, 378; cut 250). Where the edges are split over the
// waves (es) the problem is small, and one launch with skipped tiles is faster than two.
constexpr int recv_launches(int tiles, bool half, bool es, RecvLaunch (&out)[2])
{
    if (tiles == 1) {
        out[0] = {1, 4, 0, 0, 1};
        return 1;
    }
    if (es) {
        out[0] = {2, 2, tiles % 2, 0, (tiles + 1) / 2};
        return 1;
    }
    const int cap = half ? 2 : 4, n = (tiles + cap - 1) / cap, size = tiles / n, larger = tiles % n;
    int k = 0, first = 0;
    for (int more = 1; more >= 0; --more) {
        const int rt = size + more, groups = more ? larger : n - larger;
        if (groups == 0) continue;
        out[k++] = {rt, rt == 1 || (rt == 2 && !half) ? 4 : 2, 0, first, groups};
        first += groups * rt;
    }
    return k;
}

// Rank tiles of a wave whose first is rt0.
CGTP_HD constexpr int wave_rank_tiles(int rt, bool part, int tiles, int rt0)
{
    return part && tiles - rt0 < rt ? tiles - rt0 : rt;
}

// A wave's sender values: 1 KB tiles of 16 ranks x 16 points, np point tiles (an even number) per
// rank tile, from (rank tile rt0, point tile p0) to the end of its last rank tile. The tile goes
// into a load's scalar offset, which the range check of a raw buffer does not cover (past the end
// it wraps), so it has to stay inside by itself: rank tiles past the wave's are never asked for,
// and a point tile past the row's end, whose points are past the grid, reads the row's last one.
CGTP_HD constexpr unsigned value_bytes(int na, int np, int p0) { return (unsigned)(na * np - p0) * 1024u; }
CGTP_HD constexpr int value_point_tile(int pt, int t, int np, int p0)
{
    return pt <= 2 || p0 + t < np ? t : np - 1 - p0;
}
CGTP_HD constexpr unsigned value_offset(int a, int point_tile, int np) { return (unsigned)(a * np + point_tile) * 1024u; }

}  // namespace cgtp
