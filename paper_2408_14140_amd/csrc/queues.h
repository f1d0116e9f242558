// queues.h -- how the tile kernels' work is dealt to the workgroups of a grid.
// Plain constexpr arithmetic, the same on the host and on the device.
#pragma once

#include <stdint.h>

namespace ibx {

// XCDs of the device; workgroups are dispatched to them round-robin by id.
constexpr int NXCD = 8;

// Spreading queues: the entries of an XCD's slab are dealt to NQ queues, each
// served by the XCD's workgroups of one residue, with a counter in a cache
// line of its own.  (A device-scope atomic on a line that many workgroups
// share takes about 12 ns: with one counter per XCD the spreading of
// spheres1000_256 went from 80 to 96 us, with one line for all to 443 us.)
constexpr int NQ = 8;
constexpr int QSTRIDE = 32;         // ints between two counters

// The least grids: every slab has a workgroup, and in the spreading every queue
// has one (a queue without a workgroup would leave its tiles out).
constexpr int SLAB_GRID = NXCD;
constexpr int QUEUE_GRID = NXCD * NQ;

// Workgroups of a persistent launch: those resident at once, a multiple of NXCD,
// and at least `least`, however few compute units the device has.
constexpr int persistent_grid(int ncu, int per_cu, int least)
{
    const int grid = ncu * per_cu / NXCD * NXCD;
    return grid > least ? grid : least;
}

// What workgroup `block` of a grid of `grid` serves of n_act entries: every NQ-th
// one of its XCD's slab from `first` on, `count` in all, shared by nw workgroups of
// which it is the me-th, with counter `queue`.
struct QueueShare {
    int first, count, me, nw, queue;
};

constexpr QueueShare queue_share(int block, int grid, int n_act)
{
    const int per = (n_act + NXCD - 1) / NXCD;
    const int x = block % NXCD, nwg = grid / NXCD, wg = block / NXCD;
    const int end = (x + 1) * per < n_act ? (x + 1) * per : n_act;
    const int sub = wg % NQ, slab = end - x * per;
    return {x * per + sub, slab > sub ? (slab - sub + NQ - 1) / NQ : 0, wg / NQ,
            (nwg - sub + NQ - 1) / NQ, x * NQ + sub};
}

// The entry of its queue that a workgroup takes as its r-th: three by position, then
// what its counter hands out (tick).
constexpr int queue_entry(const QueueShare& s, int r, int tick)
{
    return r == 0   ? s.me
           : r == 1 ? 2 * s.nw - 1 - s.me
           : r == 2 ? 2 * s.nw + s.me
                    : 3 * s.nw + tick;
}

}  // namespace ibx
