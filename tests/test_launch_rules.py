"""The rules that choose a launch from sizes alone (csrc/launch_rules.h), over
extents that no test could run: built as plain C++ on the host."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1703_09707_amd", "csrc")
MAX_RAYS = 2 ** 31 - 1   # of a lattice block
CU = 256

PROGRAM = r"""
#include <cstdio>
#include <cstring>
#include "launch_rules.h"
using namespace raysh;
int main() {
    char what[32];
    while (std::scanf("%31s", what) == 1) {
        long long nx, ny, n;
        if (!std::strcmp(what, "waves")) {   // form, and the threads of its grid (0: the context's shape)
            if (std::scanf("%lld %lld %lld", &nx, &ny, &n) != 3) return 1;
            const int form = waves_form(nx, ny, n, TileShape{8, 4, 16, 1}, 256);
            long long threads = 0;
            int i = 0;
#define RAYSH_CASE(CX, CY, S, NS, W) \
            if (form == i++) threads = tiles_of(nx, ny, 8 * CX, 8 * CY) * 64 * W;
            RAYSH_FP64_WAVES(RAYSH_CASE)
#undef RAYSH_CASE
            std::printf("%d %lld\n", form, threads);
        } else if (!std::strcmp(what, "rows")) {   // threads of the row pass and of the disk's prefix sums, if they fit
            if (std::scanf("%lld %lld", &nx, &ny) != 2) return 1;
            const long long a = smooth_row_blocks((int)nx, (int)ny), b = disk_prefix_blocks((int)ny);
            std::printf("%lld %lld\n", grid_fits(a, 256) ? a * 256 : 0, grid_fits(b, 256) ? b * 256 : 0);
        } else if (!std::strcmp(what, "disk")) {
            if (std::scanf("%lld %lld %lld", &nx, &ny, &n) != 3) return 1;
            std::printf("%d\n", (int)disk_by_prefix((int)nx, (int)ny, n));
        } else if (!std::strcmp(what, "tiles")) {
            double dx;   // dy = 1
            if (std::scanf("%lld %lld %lf", &nx, &ny, &dx) != 3) return 1;
            const TileGrid g = expansion_tiles(nx, ny, dx, 1.0);
            std::printf("%d %d %lld\n", g.w, g.h, (long long)(g.tiles_x * g.tiles_y));
        } else {
            return 2;
        }
    }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++") or "/opt/rocm/bin/amdclang++"
    d = tmp_path_factory.mktemp("rules")
    src, out = str(d / "rules.cpp"), str(d / "rules")
    with open(src, "w") as f:
        f.write(PROGRAM)
    subprocess.run([cxx, "-O1", "-std=c++17", "-Wall", "-I", CSRC, src, "-o", out], check=True)

    def ask(lines):
        r = subprocess.run([out], input="\n".join(" ".join(map(str, l)) for l in lines), capture_output=True,
                           text=True, check=True)
        return [tuple(map(float, l.split())) for l in r.stdout.splitlines()]
    return ask


def _extents():
    sides = sorted({s + d for k in range(31) for s in (1 << k,) for d in (-1, 0, 1)} | {3, 15, 17, 1000, MAX_RAYS})
    return [(nx, ny) for nx in sides for ny in sides if 1 <= nx and 1 <= ny and nx * ny <= MAX_RAYS]


@pytest.mark.parametrize("stars", [0, 1, 50, 106, 300, 3000, 100_000, 1 << 28])
def test_waves_forms_fit_their_grid(rules, stars):
    """Every lattice that is accepted gets a form that HIP launches (fewer than
    2^32 threads): with 1024 threads for 32 x 16 rays, a lattice of a few rows
    and 2^27 columns does not."""
    ext = _extents()
    got = rules([("waves", nx, ny, stars) for nx, ny in ext])
    assert len(got) == len(ext)
    for (nx, ny), (form, threads) in zip(ext, got):
        assert threads < 2 ** 32, (nx, ny, stars, form)


def test_waves_forms_of_small_lattices(rules):
    """The lattices the forms were measured on keep them."""
    got = rules([("waves", 1000, 1000, 100), ("waves", 250, 250, 1000), ("waves", 100, 100, 3000),
                 ("waves", 2048, 2048, 10000)])
    assert [int(f) for f, _ in got][0] == 0 and all(f > 0 for f, _ in got[1:3]) and got[3][0] == 0


@pytest.mark.parametrize("side", [4096, 6000, 8192, 16384])
def test_full_lattices_keep_the_set_shape(rules, side):
    """Lattices that fill the device run in the context's shape, whose order
    of summation a batch and the lattice's bands share."""
    stars = [1, 100, 1000, 5000, 16384, 20000, 100_000, 1 << 24]
    assert [int(f) for f, _ in rules([("waves", side, side, n) for n in stars])] == [-1] * len(stars)


def test_row_passes_fit_their_grid(rules):
    """The passes that take a wave per row serve maps of up to nearly 2^26
    rows; taller ones, which are accepted too, are left to a thread per output."""
    ext = _extents()
    got = rules([("rows", wx, ny) for wx, ny in ext])
    assert len(got) == len(ext)
    for (wx, ny), (rows, prefix) in zip(ext, got):
        assert rows < 2 ** 32 and prefix < 2 ** 32
        assert rows > 0 or ny * -(-wx // 256) > 2 ** 26 - 4
        assert prefix > 0 or ny > 2 ** 26 - 8


@pytest.mark.parametrize("ratio", [1e-300, 0.05, 0.25, 0.5, 1.0, 2.0, 4.0, 20.0, 1e300])
def test_expansion_tiles_of_thin_lattices(rules, ratio):
    """Tiles follow the cells' aspect, but never so that a lattice of a few
    (32) rows or columns gets more of them than tiles of 64 x 64 rays would be
    (four times as many for 2^20 x 1 rays, three times the time)."""
    ext = _extents()
    got = rules([("tiles", nx, ny, ratio) for nx, ny in ext])
    assert len(got) == len(ext)
    for (nx, ny), (w, h, tiles) in zip(ext, got):
        square = -(-nx // 64) * -(-ny // 64)
        assert w * h == 4096 and tiles == -(-nx // int(w)) * -(-ny // int(h))
        assert tiles <= (square if min(nx, ny) <= 32 else 2 * square), (nx, ny, w, h)
    big = dict(zip(ext, got))[4096, 4096][:2]
    assert big == {0.05: (256, 16), 0.25: (128, 32), 0.5: (128, 32), 1.0: (64, 64), 2.0: (32, 128), 4.0: (32, 128),
                   20.0: (16, 256), 1e-300: (256, 16), 1e300: (16, 256)}[ratio]


def test_disk_rule(rules):
    """Prefix sums where they were measured to be faster, counts where those
    were: radii in pixels, map sides."""
    direct = [(1, 1, 2048), (3, 3, 2048), (4, 4, 1024), (4, 4, 724), (4, 4, 501), (0, 1000, 4096)]
    prefix = [(4, 4, 2048), (5, 5, 1024), (6, 6, 724), (6, 6, 501), (8, 8, 512), (8, 8, 128), (12, 12, 256),
              (25, 25, 2048), (2, 80, 8192)]
    got = rules([("disk", rx, ry, n * n) for rx, ry, n in direct + prefix])
    assert [int(g[0]) for g in got] == [0] * len(direct) + [1] * len(prefix)
