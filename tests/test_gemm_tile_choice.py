"""Which bf16 GEMM tiles the GPU tests reach (CPU: the library's tile choice is
compiled into a small program).  A tile that no test shape selects would be
compared with nothing."""
import dataclasses
import os
import subprocess

import pytest

from paper_2607_23159_amd import build, synth

from test_gpu_tiles import GRIDS, STAGED_GRIDS

PROGRAM = """
#include <cstdio>
#include "gemm_tile.hpp"
int main() {
  long m, n, k, batch, residual;
  while (std::scanf("%ld %ld %ld %ld %ld", &m, &n, &k, &batch, &residual) == 5)
    std::printf("%d\\n", (int)cs::choose_tile(m, n, k, batch, residual != 0));
  std::printf("%d\\n", (int)cs::N_TILES);
}
"""
TILES = ["W4_256x256", "W4_224x256", "W4_192x256", "W4_160x256", "W4_128x128", "W4_64x64",
         "RING_128x128", "RING_64x128", "RING_64x64", "RING_32x64", "RING_32x32"]


@pytest.fixture(scope="module")
def choose(tmp_path_factory):
    d = tmp_path_factory.mktemp("choice")
    src, exe = str(d / "choice.cpp"), str(d / "choice")
    with open(src, "w") as f:
        f.write(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-I", build.CSRC, src, "-o", exe], check=True)

    def run(shapes):
        text = "".join("%d %d %d %d %d\n" % s for s in shapes)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split()
        assert int(out[-1]) == len(TILES)
        return [TILES[int(t)] for t in out[:-1]]

    return run


def launches(model, grid, n):
    """Epilogue -> (M, N, K, batch, residual) of an evaluation of n streams."""
    m = synth.MODELS[model]
    f, h, w = grid
    rows, d = n * f * h * w, m.hidden
    return {"patch": (rows, d, m.in_ch * 4, 1, 0), "qkv": (rows, 3 * d, d, 1, 0), "out": (rows, d, d, 1, 1),
            "cross q": (rows, d, d, 1, 0), "up": (rows, m.ffn, d, 1, 0), "down": (rows, d, m.ffn, 1, 1),
            "head": (rows, m.in_ch * 4, d, 1, 0), "text": (m.text_len, d, m.text_dim, 1, 0)}


def reached(choose, grids):
    keys, shapes = [], []
    for model, grid, batches in grids:
        for n in batches:
            for epilogue, shape in launches(model, grid, n).items():
                keys.append(epilogue)
                shapes.append(shape)
    return {(t, e) for t, e in zip(choose(shapes), keys)}


def test_every_tile_is_compared(choose):
    missing = set(TILES) - {t for t, _ in reached(choose, GRIDS + STAGED_GRIDS)}
    assert not missing, missing


def test_staged_stores_of_every_large_tile_are_compared(choose):
    # the waves of these tiles hold 128, 112, 96 and 80 rows, and the staged stores
    # split them differently
    got = reached(choose, GRIDS + STAGED_GRIDS)
    for tile in TILES[:4]:
        for epilogue in ("qkv", "up"):
            assert (tile, epilogue) in got, (tile, epilogue)
