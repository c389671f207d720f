"""Rules of the engine that are host arithmetic alone, compiled from the
headers the library is built from."""
import ctypes as C
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1004_0480_amd", "csrc")


def compile_host(tmp, name, source):
    src, so = tmp / (name + ".cpp"), tmp / (name + ".so")
    src.write_text(source)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC,
                    "-I", os.path.join(ROOT, "include"), str(src), "-o", str(so)], check=True)
    return C.CDLL(str(so))


# ------------------------------------------------------- layout conversions

@pytest.fixture(scope="module")
def row_runs(tmp_path_factory):
    lib = compile_host(tmp_path_factory.mktemp("io"), "io", """
#include "rd_io_cfg.hpp"
extern "C" void split(int64_t nx, int64_t rows, int64_t* out) {
    const rdk::RowRuns r = rdk::row_runs(nx, rows);
    const int64_t v[] = {r.run, r.parts, int64_t(r.blocks), r.deep};
    for (int i = 0; i < 4; ++i) out[i] = v[i];
}
""")

    def split(nx, rows):
        out = (C.c_int64 * 4)()
        lib.split(C.c_int64(nx), C.c_int64(rows), out)
        return list(out)

    return split


def test_conversions_cover_every_unit_once(row_runs):
    """The units that the workgroups of a conversion take (as the kernel forms
    them) are the field's, each once."""
    rng = random.Random(2)
    shapes = [(1, 1), (5, 1), (4096, 1), (4097, 2), (9001, 3), (1 << 16, 1), (3, 5000), (403, 900)]
    shapes += [(int(10 ** rng.uniform(0, 4.5)), int(10 ** rng.uniform(0, 2.5))) for _ in range(200)]
    for nx, rows in shapes:
        run, parts, blocks, _ = row_runs(nx, rows)
        nx4, taken = (nx + 3) // 4, []
        assert run == 1 or parts == 1
        for b in range(blocks):
            group, part = divmod(b, parts)
            total = min(run, rows - group * run) * nx4
            each = -(-total // parts)
            taken += [group * run * nx4 + u for u in range(part * each, min((part + 1) * each, total))]
        assert taken == list(range(rows * nx4)), (nx, rows)


@pytest.mark.parametrize("nx,rows", [(1 << 24, 1), (1 << 22, 4), (1 << 18, 64), (1 << 24, 1 << 10)])
def test_conversions_of_few_long_rows_fill_the_chip(row_runs, nx, rows):
    assert row_runs(nx, rows)[2] >= 4 * 256       # workgroups: several for each compute unit


@pytest.mark.parametrize("nx,rows", [(2052, 1 << 24), (4096, 1 << 24), (64, 1 << 34), (1 << 24, 1 << 16), (1, 1 << 40)])
def test_conversions_of_the_largest_fields_fit_a_launch(row_runs, nx, rows):
    """A launch holds fewer than 2^32 threads: 2^24 - 1 workgroups of 256."""
    run, parts, blocks, _ = row_runs(nx, rows)
    assert 0 < blocks < 1 << 24
    assert -(-rows // run) * parts == blocks and (run == 1 or parts == 1)
    assert run * -(-nx // 4) < 1 << 32                # a run's units are counted in 32 bits


# --------------------------------------------------------------- autotuning

@pytest.fixture(scope="module")
def tune(tmp_path_factory):
    lib = compile_host(tmp_path_factory.mktemp("tune"), "tune", """
#include "rd_tune.hpp"
extern "C" int steps(int trial, int per) { return rdk::tune_steps(trial, per); }
extern "C" int warmup(int per) { return rdk::tune_warmup(per); }
static rdk::PlanCache cache;
static rdk::PlanCache::Key key(int n) { return {n, n, n, 1, 0, 0}; }
extern "C" void put(int n, int march, int best, int general) {
    rd_plan b{}, g{};
    b.kernel = best, g.kernel = general;
    cache.put(key(n), march != 0, b, general ? &g : nullptr);
}
extern "C" int get(int n, int march) {
    bool own;
    const rd_plan* p = cache.get(key(n), march != 0, &own);
    return p ? (own ? 1 : -1) * p->kernel : 0;
}
""")
    return lib


def test_candidates_are_timed_over_whole_launches(tune):
    """No left-over launch is timed, whatever the trial count, and a plan's own
    kernel has run before the first timed launch."""
    for per in (1, 2, 3, 4):
        assert tune.warmup(per) >= per
        for trial in range(1, 40):
            n = tune.steps(trial, per)
            assert n % per == 0 and n % 2 == 0 and trial <= n < trial + 2 * per


def test_tuned_plans_serve_their_own_class_of_grids(tune):
    """A shape's tuned register march is not what a grid that no march takes is
    given, and a tuned ring is not what keeps a grid from its march."""
    march, ring, tring, lds = 8, 4, 7, 5
    tune.put(1, 0, ring, ring)                 # a grid with held faces, tuned alone
    assert tune.get(1, 0) == ring and tune.get(1, 1) == 0
    tune.put(2, 1, march, ring)                # a march's grid: its best other plan serves the rest
    assert tune.get(2, 1) == march and tune.get(2, 0) == -ring        # (negative: not tuned on its own class)
    tune.put(2, 0, tring, tring)               # which are then tuned themselves, and keep that
    tune.put(2, 1, lds, lds)                   # (another plan may beat the march on its own grid)
    assert tune.get(2, 0) == tring and tune.get(2, 1) == lds
    tune.put(3, 1, march, 0)                   # none but marches ran
    assert tune.get(3, 0) == 0 and tune.get(4, 0) == tune.get(4, 1) == 0
    tune.put(3, 1, march, ring)
    assert tune.get(3, 0) == -ring


# ------------------------------------------------------------ tiles of a march

def test_march_tiles_in_both_orders(tmp_path):
    """Every tile once in either order: x, then y, then the z chunk, or the z
    chunk first."""
    lib = compile_host(tmp_path, "tiles", """
#include "rd_tiles.hpp"
extern "C" void tile(int b, int x, int y, int z, int zfast, int* out) {
    const rdk::MarchTile t = rdk::march_tile(b, x, y, z, zfast != 0);
    out[0] = t.x, out[1] = t.y, out[2] = t.z;
}
""")
    out = (C.c_int * 3)()
    for nx, ny, nz in ((1, 1, 1), (3, 5, 7), (1, 4, 2), (6, 1, 9)):
        for zfast in (0, 1):
            got = []
            for b in range(nx * ny * nz):
                lib.tile(b, nx, ny, nz, zfast, out)
                got.append(tuple(out))
            want = ([(x, y, z) for y in range(ny) for x in range(nx) for z in range(nz)] if zfast else
                    [(x, y, z) for z in range(nz) for y in range(ny) for x in range(nx)])
            assert got == want


def test_every_march_kernel_takes_its_plan_order():
    """A plan's order reaches the march kernels: each forms its tile with the
    shared rule, from the arguments' order (the 19-point march ignored it)."""
    for name in ("rd_march.hpp", "rd_march19.hpp"):
        with open(os.path.join(CSRC, name)) as fh:
            assert "march_tile(xcd_tile(blockIdx.x, gridDim.x), a.tiles_x, tiles_y, chunks, a.zfast != 0)" in fh.read()
