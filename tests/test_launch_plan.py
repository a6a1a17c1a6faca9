"""How steps are dealt to launches (launch_plan.hpp), on the host: the counts, and the kind of launch on
grids where one kind was measured well ahead of the others."""
import os
import subprocess

import pytest

import paper_1803_00437_amd as F
from paper_1803_00437_amd import build as B

HERE = os.path.dirname(os.path.abspath(__file__))
STENCIL = {"fd3": 3, "fd5": 5, "lwacm": 1, "mrt": 9}


@pytest.fixture(scope="module")
def deal(tmp_path_factory):
    """deal([(kind, dtype, walls, force, disk, nx, ny, n), ...]) -> [{tile, steps, tiles, ...}, ...]"""
    F.load_library()
    exe = str(tmp_path_factory.mktemp("plan") / "launch_plan_probe")
    rocm = os.path.dirname(os.path.dirname(B.HIPCC))
    subprocess.run(["g++", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", f"-I{rocm}/include",
                    os.path.join(HERE, "launch_plan_probe.cpp"), "-o", exe, f"-L{B.OUT_DIR}", "-lfdlbm",
                    f"-Wl,-rpath,{B.OUT_DIR}", "-Wl,--allow-shlib-undefined"], check=True)

    def run(calls):
        text = "\n".join(" ".join(map(str, (STENCIL.get(k, k), F.DTYPE.get(d, d), int(w), int(f), int(disk), nx, ny, n)))
                         for k, d, w, f, disk, nx, ny, n in calls)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split("\n")
        keys = ("cols", "rows", "steps", "tiles", "fives", "threes", "twos", "ones", "sum", "count")
        rows = [dict(zip(keys, map(int, o.split()))) for o in out if o]
        assert len(rows) == len(calls)
        return rows

    return run


@pytest.mark.parametrize("kind,dtype,nx,ny", [
    ("fd3", "f64", 64, 64), ("fd3", "f32", 1024, 1024), ("fd3", "f16sr", 2048, 2048), ("fd3", "f32", 4096, 4096),
    ("fd5", "f64", 800, 800), ("lwacm", "f32", 191, 191), ("lwacm", "f64", 3000, 3000), ("mrt", "f64", 100, 100),
    ("mrt", "f32", 1300, 1300), ("mrt", "f32", 4096, 4096)])
def test_every_deal_adds_up_and_keeps_the_buffer(deal, kind, dtype, nx, ny):
    ns = list(range(1, 300)) + [997, 1000, 65536, 10 ** 6 + 1]
    for n, d in zip(ns, deal([(kind, dtype, 0, 0, 0, nx, ny, n) for n in ns])):
        assert d["sum"] == n and d["count"] % 2 == n % 2, (n, d)


@pytest.mark.parametrize("one,two,three,want", [
    (46, 74, 119, "twos"),     # FP32 8 x 1024^2: 37 us per step, in threes 39.7
    (10, 10, 15, "threes"),    # FP32 4 x 64^2: as fast in twos, and fewer launches
    (37, 78, 129, "ones"),     # FP16 8 x 1024^2: the one-step kernel takes four columns per lane
    (24, 35, 52, "threes"),    # FP16, odd widths
    (24, 35, 70, "twos"),
    (19, 34, 63, "twos")])     # FP32, 30 grids of 32 to 496 columns
def test_a_batch_takes_the_fastest_deal(deal, one, two, three, want):
    """Times in us of launches of one, two and three steps of all instances."""
    ns = list(range(1, 300)) + [10 ** 6 + 1]
    deals = deal([(0, one, two, three, 0, 0, 0, n) for n in ns])
    for n, d in zip(ns, deals):
        assert d["sum"] == n and d["count"] % 2 == n % 2, (n, d)
    d = deals[95]  # 96 steps: a multiple of three and of four
    assert d[want] == 96 // {"ones": 1, "twos": 2, "threes": 3}[want], d


# us per step, measured: (n, single steps, steps together in the sweep, tiles as planned); the launch
# has to be of the fastest kind, which leads by more than the estimates' spread
ONE, FUSED, TILES = "one", "fused", "tiles"


@pytest.mark.parametrize("kind,dtype,walls,force,nx,ny,n,want", [
    ("fd3", "f64", 0, 0, 1024, 1024, 1, ONE),    # 14.1, -, 20.2
    ("fd3", "f64", 0, 0, 1024, 1024, 2, ONE),
    ("fd3", "f64", 1, 1, 1024, 1024, 2, ONE),    # 15.5, -, 21.4
    ("fd3", "f64", 0, 0, 700, 700, 2, ONE),      # 8.3, -, 10.9
    ("fd3", "f64", 0, 0, 64, 64, 1, TILES),      # 6.7, -, 4.2
    ("fd3", "f32", 0, 0, 64, 64, 2, TILES),      # 9.7, -, 3.7
    ("fd3", "f32", 0, 0, 1024, 1024, 50, TILES),  # 11.2, 10.2, 6.7
    ("fd3", "f64", 0, 0, 64, 64, 10, TILES),     # 6.7, 4.5, 2.3
    ("fd5", "f64", 0, 0, 800, 800, 50, ONE),     # 10.1, 11.1, 13.6
    ("fd5", "f64", 0, 0, 800, 800, 3, ONE),
    ("fd5", "f64", 0, 0, 20000, 16, 50, ONE),    # 8.5, 9.3, 13.2
    ("fd5", "f32", 0, 0, 1001, 777, 50, TILES),  # 22.4, 12.1, 8.9
    ("lwacm", "f32", 0, 0, 1024, 1024, 2, ONE),  # 9.4, -, 11.7
    ("lwacm", "f64", 0, 0, 191, 191, 100, TILES),  # 7.2, 2.9, 1.4
    ("mrt", "f32", 0, 0, 384, 384, 2, ONE),      # 4.6, -, 6.9
    ("mrt", "f32", 1, 1, 128, 2048, 1, ONE),     # 5.1, -, 8.7
    ("mrt", "f64", 0, 0, 384, 384, 2, ONE),      # 6.5, -, 8.6
    ("mrt", "f32", 0, 0, 640, 640, 2, ONE),      # 7.4, -, 10.1
    ("mrt", "f32", 0, 0, 384, 384, 50, TILES),   # 4.6, 3.9, 1.9
    ("mrt", "f32", 0, 0, 8192, 8192, 50, FUSED),  # 866, 232, -
    ("fd3", "f32", 0, 0, 8192, 8192, 50, FUSED),  # 294, 190, -
    ("fd3", "f64", 0, 0, 4096, 4096, 50, FUSED),  # 148, 98, -
])
def test_a_call_takes_the_fastest_kind_of_launch(deal, kind, dtype, walls, force, nx, ny, n, want):
    d, = deal([(kind, dtype, walls, force, 0, nx, ny, n)])
    got = TILES if d["tiles"] else ONE if d["ones"] == n else FUSED
    assert got == want, d


def test_the_gpu_tests_grids_take_every_shape_a_plan_can_give(deal):
    """The bitwise tests of the tiles (test_gpu_tile_routes.py) have to run every shape that grids up to
    1450 nodes a side take, whatever the constants of the plan."""
    from test_gpu_tile_routes import TILE_GRIDS, TILE_KINDS, TILE_STEPS

    sizes = [(s, s + t) for s in list(range(16, 64, 6)) + list(range(64, 1450, 14)) for t in (0, 3)]
    sizes += [(1001, 777), (1021, 770), (500, 2000), (20000, 16), (16, 20000), (8, 3000), (3000, 8)]
    for k, d, bc, force in TILE_KINDS:
        def shapes(grids):
            calls = [(k, d, bc == "walls", force, bc == "disk", nx, ny, TILE_STEPS) for nx, ny in grids]
            return {(r["cols"], r["rows"]) for r in deal(calls) if r["tiles"]}

        assert shapes(TILE_GRIDS) == shapes(sizes + TILE_GRIDS), (k, d, bc, force)
