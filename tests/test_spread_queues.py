"""The dealing of the spreading's tiles to workgroups (csrc/queues.h), compiled for
the host: whatever the number of compute units and the residency cap, every tile
is taken exactly once, in whatever order the workgroups draw their tickets."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2408_14140_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "queues.h"
using namespace ibx;

// Workgroups of one launch run one after the other, forwards or backwards.
static bool every_entry_once(int grid, int n_act, bool backwards)
{
    std::vector<int> taken(n_act + 1, 0), counter(NXCD * NQ, 0);
    for (int k = 0; k < grid; ++k) {
        const QueueShare s = queue_share(backwards ? grid - 1 - k : k, grid, n_act);
        if (s.nw < 1 || s.queue < 0 || s.queue >= NXCD * NQ)
            return false;
        for (int r = 0;; ++r) {
            const int tick = r > 2 ? counter[s.queue]++ : 0;
            const int q = queue_entry(s, r, tick);
            if (q < 0)
                return false;
            if (q >= s.count)
                break;
            const int e = s.first + q * NQ;
            if (e < 0 || e >= n_act)
                return false;
            ++taken[e];
        }
    }
    for (int e = 0; e < n_act; ++e)
        if (taken[e] != 1)
            return false;
    return true;
}

int main()
{
    const int entries[] = {0, 1, 7, 8, 9, 63, 64, 65, 511, 1000, 20011};
    for (int ncu : {1, 7, 8, 16, 32, 38, 63, 64, 65, 128, 256, 304})
        for (int per_cu : {1, 2, 3, 16, 32})
            for (int n_act : entries)
                for (int b = 0; b < 2; ++b) {
                    const int grid = persistent_grid(ncu, per_cu, QUEUE_GRID);
                    if (grid % NXCD != 0 || !every_entry_once(grid, n_act, b)) {
                        std::printf("ncu %d, %d a unit: grid %d, %d entries\n", ncu, per_cu,
                                    grid, n_act);
                        return 1;
                    }
                }
    return 0;
}
"""


def test_every_tile_is_taken_once_on_any_device(tmp_path):
    src, exe = tmp_path / "queues.cpp", tmp_path / "queues"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC, "-o", str(exe),
                    str(src)], check=True)
    run = subprocess.run([str(exe)], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout
