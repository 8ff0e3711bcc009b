"""The tile rule of the projection GEMM (csrc/linear_tiles.h), compiled on its
own: no GPU.  The GPU tests of every tile rely on the tiles checked here."""
import subprocess

import pytest

from paper_2607_01817_amd import build
from tests import gemm_shapes as gs

DRIVER = r"""
#include <cstdio>
#include "linear_tiles.h"
using namespace hcms;
int main() {
    long long M, N, K, n_cu;
    int bytes, qkv;
    while (std::scanf("%lld %lld %lld %d %d %lld", &M, &N, &K, &bytes, &qkv, &n_cu) == 6) {
        const TileCost &c = kTiles[linear_tile(M, N, K, bytes, qkv, n_cu)];
        std::printf("%d %d %d\n", c.bm, c.bn, c.per_cu);
    }
}
"""


@pytest.fixture(scope="module")
def tiles(tmp_path_factory):
    d = tmp_path_factory.mktemp("tiles")
    (d / "driver.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", build.CSRC, str(d / "driver.cpp"),
                    "-o", str(d / "driver")], check=True)

    def ask(cases):
        text = "".join(" ".join(map(str, c)) + "\n" for c in cases)
        out = subprocess.run([str(d / "driver")], input=text, text=True, capture_output=True, check=True).stdout
        return [tuple(map(int, ln.split())) for ln in out.splitlines()]

    return ask


def _check(rows, got):
    for (name, more, _, M, N, _), (bm, bn, per_cu) in zip(rows, got):
        assert (bm, bn) == gs.TILES[name], (M, N)
        assert (-(-M // bm) * -(-N // bn) > 256 * per_cu) == more, (M, N)


def test_linear_shapes_take_every_tile(tiles):
    _check(gs.LINEAR, tiles([(M, N, K, es, 0, 256) for _, _, es, M, N, K in gs.LINEAR]))
    assert {r[:3] for r in gs.LINEAR} == {(t, m, e) for t in gs.TILES for m in (False, True) for e in (2, 4)}


def test_qkv_shapes_take_every_tile(tiles):
    rows = [(t, m, es, g[0] * g[1], 3 * H * d, D) for t, m, es, g, D, H, d in gs.QKV]
    _check(rows, tiles([(M, N, K, es, 1, 256) for _, _, es, M, N, K in rows]))
    # fp32 rotations have no 256 x 256 tile.
    assert {r[:3] for r in rows} == {(t, m, e) for t in gs.TILES for m in (False, True) for e in (2, 4)
                                     if (t, e) != ("A", 4)}


def test_small_devices_get_a_tile(tiles):
    for bm, bn, per_cu in tiles([(M, N, 64, es, q, n) for M in (1, 5000) for N in (8, 8000)
                                 for es in (2, 4) for q in (0, 1) for n in (1, 304)]):
        assert (bm, bn) in gs.TILES.values() and per_cu in (1, 2)
