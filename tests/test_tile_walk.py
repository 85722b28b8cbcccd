"""The walk of workgroups over output tiles with the bands that gemm_deep_kernel is launched with: every tile of every shard exactly
once, for shards of more tile-rows than a band can count too.  Runs on the host, on the functions that the kernel and its launch
use."""
import os
import subprocess

import pytest

from paper_2110_15032_amd import build

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "gemm_device.h"
using namespace sbp;
int main() {
    int bad = 0;
    for (int tm : {1, 3, 4, 5, 31, 32, 33, 64, 254, 255, 256, 257, 300, 511, 512, 513, 1024})
        for (int tn : {1, 2, 3, 7})
            for (int groups : {1, 2, 3, 7, 8, 16, 64}) {
                const int tiles = tm * tn * groups, nblk = (tiles + 7) / 8 * 8, order = deep_band(tm, tn, tiles);
                std::vector<int> seen(tiles, 0);
                if (order < 1 || order > 255) { ++bad; continue; }
                for (int b = 0; b < nblk; ++b) {
                    const TileCoord t = map_tile(b, nblk, tm, tn, groups, order);
                    if (!t.valid) continue;
                    if (t.g < 0 || t.g >= groups || t.tile_m < 0 || t.tile_m >= tm || t.tile_n < 0 || t.tile_n >= tn) { ++bad; continue; }
                    ++seen[(t.g * tm + t.tile_m) * tn + t.tile_n];
                }
                for (int n : seen) bad += n != 1;
            }
    printf("%d\n", bad);
    return bad != 0;
}
"""


def test_every_tile_once(tmp_path):
    if not os.path.exists(build.HIPCC):
        pytest.skip("hipcc is not installed")
    src, exe = tmp_path / "walk.hip", str(tmp_path / "walk")
    src.write_text(PROGRAM)
    subprocess.run([build.HIPCC, "--cuda-host-only", "-O1", "-std=c++17", "-w", "-I", build.CSRC, "-I", os.path.join(build.ROOT, "include"), str(src), "-o", exe], check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, f"{r.stdout.strip()} tiles missed, met twice or out of range (exit status {r.returncode})"
