"""Launch geometry followed on the host (no GPU).  The walk of the slice GEMM's workgroups over the units of C: every unit
that holds a row and a column of C is multiplied over every 64 of k exactly once, whatever the order, the split along
k and the padding.  The scan's launches: none has more threads than a launch may have.  The ESC kernel's blocks: those
that one row or column of the operands leaves open meet as many workgroups as there are.  The FP64 tiles straight from
memory: no load lies outside the operands, and every k is multiplied once."""
import itertools
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def host_program(tmp_path_factory, source):
    exe = tmp_path_factory.mktemp("host") / "program"
    cmd = ["g++", "-std=c++17", "-O1", "-Wno-attributes", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
           "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2511_13778_amd", "csrc"),
           os.path.join(ROOT, "tests", source), "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def run(cases):
        out = subprocess.run([str(exe)], input="\n".join(" ".join(map(str, c)) for c in cases), capture_output=True,
                             text=True, check=True).stdout.split("\n")[:-1]
        assert len(out) == len(cases)
        return [tuple(map(int, ln.split())) for ln in out]
    return run


def golden_times(name):
    return [ln.split() for ln in open(os.path.join(ROOT, "tests", "golden", name)) if not ln.startswith("#")]


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    return host_program(tmp_path_factory, "host_unit_walk.cpp")


@pytest.fixture(scope="module")
def scan_grid(tmp_path_factory):
    return host_program(tmp_path_factory, "host_scan_grid.cpp")


@pytest.fixture(scope="module")
def f64_plan(tmp_path_factory):
    return host_program(tmp_path_factory, "host_f64_plan.cpp")


def test_every_unit_and_part_is_taken_exactly_once(walk):
    # odd and even numbers of blocks, padding-only quadrants on either edge, odd and even numbers of parts, small and large
    # workspaces (which decide between parts with slots and atomics), more units than CUs, a split last round
    mn = [1, 100, 128, 129, 200, 256, 300, 500, 513, 600, 700, 1300, 2300, 2500]
    cases = [(m, n, k, s_cap, tile_mode, 256) for m, n in itertools.product(mn, mn)
             for k in (1, 64, 65, 700, 1000, 3500, 4000, 7500, 20000) for s_cap in (2, 9, 26) for tile_mode in (0, 1)]
    got = walk(cases)
    odd_atomic = 0
    for c, (kind, z, missed, repeated, mixed, few) in zip(cases, got):
        assert (missed, repeated, mixed) == (0, 0, 0), (c, kind, z, missed, repeated, mixed)
        blocks = -(-c[0] // 256) * -(-c[1] // 256)
        odd_atomic += c[4] == 1 and kind == 2 and blocks * z % 2 == 1
    assert odd_atomic > 50        # per-block order, atomics, items that do not divide by the eight XCDs


@pytest.mark.parametrize("m,n,k", [(100, 100, 4000), (600, 600, 7500), (200, 100, 4000), (600, 100, 3500)])
def test_shapes_of_the_gpu_test_take_the_atomic_route(walk, m, n, k):
    # what test_per_block_split_with_padding_quadrants multiplies on the GPU
    (kind, z, missed, repeated, mixed, _), = walk([(m, n, k, 26, 1, 256)])
    assert kind == 2 and -(-m // 256) * -(-n // 256) * z % 2 == 1
    assert (missed, repeated, mixed) == (0, 0, 0)


def test_which_calls_take_the_256_blocks(walk):
    # at most two slices and enough blocks to fill the chip; among them what
    # test_slice_gemm_of_one_or_two_slices multiplies on the GPU
    yes = [(3700, 3900, 1, 1), (3840, 3840, 64, 1), (3700, 3900, 200, 1), (4900, 5100, 130, 2), (4900, 5100, 320, 2), (8192, 8192, 256, 2),
           (3700, 3900, 66000, 2)]
    no = [(3700, 3900, 130, 3), (8192, 8192, 8192, 7), (2048, 2048, 2048, 1), (300, 300, 300, 2)]
    got = walk([(*c, 0, 256) for c in yes + no] + [(*c, 1, 256) for c in yes])
    assert [r[5] for r in got] == [1] * len(yes) + [0] * (len(no) + len(yes))


def test_calls_of_the_gpu_test_of_units_take_them(walk, tmp_path_factory):
    from test_gpu_small import UNITS
    plan = host_program(tmp_path_factory, "host_call_plan.cpp")
    assert [g for g, in plan([(m, n, k, S, S, 0, 1) for m, n, k, S in UNITS])] == [0] * len(UNITS)
    assert [r[0] for r in walk([(*c, 0, 256) for c in UNITS])] == [0, 1, 1, 1, 2, 2]


def test_calls_of_the_gpu_tests_of_tiles_take_them(walk, tmp_path_factory):
    from test_gpu_mid import CARRIES, ONE, TWO, carries_size
    from test_gpu_small import TILES_32
    from test_gpu_streaming import LARGE
    plan = host_program(tmp_path_factory, "host_call_plan.cpp")

    def routes(calls):
        return [g for g, in plan([(m, n, k, S, S, 0, 1) for m, n, k, S in calls])]
    assert routes(TILES_32) == [1] * len(TILES_32)
    assert routes(TWO) == [3] * len(TWO) and routes(ONE) == [2] * len(ONE)
    assert routes([(*carries_size(S), S) for S in CARRIES]) == [3 if S <= 8 else 2 for S in CARRIES]
    assert routes([c[:4] for c in LARGE]) == [0] * len(LARGE)
    assert [r[5] for r in walk([(*c[:4], 0, 256) for c in LARGE])] == [1, 1, 0, 0]
    # batches: tiles with one and two to a CU, units
    assert [g for g, in plan([(400, 300, 3000, 7, 7, 0, 4), (700, 800, 700, 7, 7, 0, 4), (700, 600, 4000, 13, 7, 0, 3),
                              (1000, 1000, 3000, 13, 7, 0, 4)])] == [2, 3, 0, 0]


@pytest.mark.parametrize("num_cu", [4, 12, 36, 100, 250, 304])
def test_other_numbers_of_compute_units(walk, num_cu):
    # a device that shows some of its units only: not always a multiple of eight.  A workgroup keeps its part of k while it
    # walks several units, so it must not meet units of different parts
    mn = [100, 129, 300, 513, 700, 1300]
    cases = [(m, n, k, s_cap, tile_mode, num_cu) for m, n in itertools.product(mn, mn)
             for k in (64, 700, 3500, 7500, 20000) for s_cap in (2, 9, 26) for tile_mode in (0, 1)]
    for c, (kind, z, missed, repeated, mixed, few) in zip(cases, walk(cases)):
        assert (missed, repeated, mixed) == (0, 0, 0), (c, kind, z, missed, repeated, mixed)


def test_scan_launches_stay_within_the_grid_limit(scan_grid):
    # HIP refuses a launch of 2^32 threads or more.  k-contiguous operands of 2^34 elements (137 GB) with ESC blocks of 16
    # come to that in one launch; every size the library accepts must be scanned whole
    sizes = [(1, 1, 1), (256, 300, 65), (8192, 8192, 8192), (8192, 1, 1 << 21), (1 << 15, 1 << 14, 1 << 20), (1 << 22, 1, 1 << 14),
             (1 << 22, 1 << 22, 256), (4000001, 17, 8191), (1, 1 << 21, 1 << 21)]
    cases = [(*s, b, ar, br) for s in sizes for b in (16, 32, 64, 1024) for ar in (0, 1) for br in (0, 1)]
    slabs = 0
    for c, (launches, most, covered, needed) in zip(cases, scan_grid(cases)):
        assert most < 1 << 32 and covered >= needed and covered - needed < 4, (c, launches, most, covered, needed)
        slabs += launches > 1
    assert slabs
    (launches, *_), = scan_grid([(8192, 8192, 8192, 16, 0, 0)])
    assert launches == 1


def test_scan_of_long_blocks_has_workgroups_for_the_chip(scan_grid):
    # k contiguous, ESC blocks of several 64s of k: 64 rows to a workgroup only from one and a half workgroups to a CU on (half with
    # one such operand), below that 16
    up = lambda x: -(-x // 256) * 256
    cases = [(*c, rows) for c, rows in (((2000, 40, 1500, 128, 0, 0), 16), ((2000, 40, 1600, 128, 0, 0), 64), ((155, 208, 4555, 1024, 0, 0), 16),
                                        ((64, 64, 2000, 64, 0, 0), 64), ((6000, 3000, 4555, 48, 0, 0), 16), ((1955, 36, 2987, 1024, 0, 0), 16),
                                        ((160, 1518, 1783, 256, 0, 0), 16), ((600, 40, 1600, 128, 0, 1), 16), ((600, 40, 1700, 128, 0, 1), 64),
                                        ((40, 600, 3201, 256, 1, 0), 16), ((40, 600, 3301, 256, 1, 0), 64))]
    for (m, n, k, b, ar, br, rows), (launches, most, *_) in zip(cases, scan_grid([c[:6] for c in cases])):
        blocks, row_blocks = -(-k // b), up(m) // (64 if ar else rows) + up(n) // (64 if br else rows)
        assert (launches, most // 256) == (1, row_blocks * (blocks if row_blocks * -(-blocks // 4) < 1024 else -(-blocks // 4))), (m, n, k, b)


def test_blocks_of_one_row_or_column_are_spread_over_the_workgroups(tmp_path_factory):
    run = host_program(tmp_path_factory, "host_esc_walk.cpp")
    sizes = [(64, 64), (32, 32), (16, 512), (512, 16), (128, 128), (33, 47), (2, 300), (300, 2), (1, 700), (256, 256), (8, 4096),
             (72, 72), (96, 96), (80, 200), (64, 1000), (512, 512), (1024, 1024)]
    cases = [(a, b, min(a * b, 512)) for a, b in sizes]
    for c, (wrong, most_row, most_col) in zip(cases, run(cases)):
        nbi, nbj, grid = c
        assert wrong == 0, c
        # a block row has nbj blocks, a block column nbi: not far from an even share of either, for each workgroup
        assert most_row <= 3 * -(-nbj // grid) + 1 and most_col <= -(-nbi // grid), (c, most_row, most_col)


@pytest.mark.parametrize("ar,br", list(itertools.product((0, 1), (0, 1))))
def test_fp64_tiles_stay_inside_their_operands(tmp_path_factory, ar, br):
    # the last tile of either side, whose rows end with the operand; a share of a wave may be empty, less than a 16 of k, one, more
    run = host_program(tmp_path_factory, "host_f64_walk.cpp")
    cases = [(m, n, k, 0, k, waves, ar, br, pad) for m, n, pad in ((1, 17, 0), (33, 31, 0), (48, 64, 5)) for k in range(1, 201) for waves in (4, 8)]
    # parts of a split: the first carries the remainder, the others have a multiple of 16 each
    for kt in (128, 129, 135, 200, 1000, 1033):
        for parts in (2, 3):
            per = kt // parts // 16 * 16
            first = kt - (parts - 1) * per
            for z in range(parts):
                kb, k = (0, first) if z == 0 else (first + (z - 1) * per, per)
                cases.append((33, 31, k, kb, kt, 4, ar, br, 0))
    bad = [(c, r) for c, r in zip(cases, run(cases)) if r != (0, 0)]
    assert not bad, (len(bad), len(cases), bad[:10])


def test_fp64_product_of_less_than_a_k_step_never_loads_a_full_one(f64_plan):
    # tiles through LDS take k < 16 in the bounds-checked loop only
    sizes = [(1, 1), (64, 64), (100, 3000), (7000, 7000), (4000, 4000), (1 << 20, 3), (1 << 22, 1 << 22)]
    got = f64_plan([(m, n, k, 1, 0, beta, 0) for m, n in sizes for k in range(1, 16) for beta in (0, 1)])
    assert {mode for direct, _, _, mode in got} == {2}
    assert {direct for direct, *_ in got} == {0, 1} and got[-1][1] == 0
    assert [mode for *_, mode in f64_plan([(64, 64, 16, 1, 1, 0, 0), (64, 64, 17, 1, 1, 0, 0), (65, 64, 32, 1, 1, 0, 0), (64, 64, 64, 1, 1, 0, 1 << 22)])][1:] == [1, 1, 2]


def test_fp64_tile_is_near_the_fastest_measured(f64_plan):
    # a hundred calls timed on every tile; among them those on which a choice that knew neither beta nor the operands' layout, and
    # nothing of k below 50, took the wrong one
    forms = [(0, 128, 128), (0, 64, 64), (1, 16, 16), (1, 32, 32), (1, 32, 64), (1, 64, 32), (1, 48, 64), (1, 64, 48)]
    rows = golden_times("f64_tile_times.txt")
    got = f64_plan([(*r[:3], int(r[3] == "N"), int(r[4] == "T"), int(float(r[5]) != 0), 0) for r in rows])
    off = [float(r[6 + forms.index(g[:3])]) / min(map(float, r[6:])) for r, g in zip(rows, got)]
    assert max(off) < 1.4 and sum(off) / len(off) < 1.05, (max(off), sum(off) / len(off))


def test_route_of_an_emulated_call_is_near_the_fastest_measured(tmp_path_factory):
    # calls timed on every route, 10 to 150 ms on end each; among them those on which an estimate that asked 64 x 64 tiles to be 14 to 28 %
    # better from four to a CU on, and took the cost of few slices from that of many, was up to 38 % off (5 % on average over these)
    run = host_program(tmp_path_factory, "host_call_plan.cpp")
    rows = golden_times("route_times.txt")
    got = run([(*r[:6], 1) for r in rows])
    off = [float(r[6 + g]) / min(float(x) for x in r[6:] if x != "-") for r, (g,) in zip(rows, got)]
    assert max(off) < 1.2 and sum(off) / len(off) < 1.015, (max(off), sum(off) / len(off))


def test_route_does_not_jump_where_the_times_do_not(tmp_path_factory):
    # seven slices: both sides of the four tiles to a CU and of the 64s of k that the times do not step at (2048^3 215 us on units, 211 on tiles,
    # 2500 x 2500 x 960 and 961 on tiles 175 and 189, on units 199 and 213); 4096^3 and 8192^3 are faster on units, by 6 to 7 %
    run = host_program(tmp_path_factory, "host_call_plan.cpp")
    tiles = [(1984, 1984, 2048), (2048, 2048, 2048), (2500, 2500, 960), (2500, 2500, 961), (3000, 3000, 1500)]
    units = [(4096, 4096, 4096), (8192, 8192, 4096), (8192, 8192, 8192)]
    assert [g for g, in run([(*s, 7, 7, 0, 1) for s in tiles + units])] == [3] * len(tiles) + [0] * len(units)


def test_fallback_is_where_it_is_near_the_fastest_measured(tmp_path_factory):
    # guarded calls that fall back, timed with the FP64 product in its own launch and in the last launch of the emulated call; among
    # them those where a rule that knew no split of k and no workgroup alone on its CU took the wrong one
    run = host_program(tmp_path_factory, "host_f64_fold.cpp")
    cases, times = [], []
    for r in golden_times("fold_times.txt"):
        for edge, t in ((32, r[8]), (64, r[9])):
            if t != "-":
                cases.append((*r[:3], int(r[3] == "N"), int(r[4] == "T"), int(float(r[5]) != 0), r[6], edge, 1 << 26))
                times.append((float(r[7]), float(t)))
    off = [t[g] / min(t) for t, (g,) in zip(times, run(cases))]
    assert max(off) < 1.25 and sum(off) / len(off) < 1.02, (max(off), sum(off) / len(off))
    assert 0.1 < sum(g for g, in run(cases)) / len(cases) < 0.9


def test_native_products_share_a_launch_unless_a_split_of_k_is_faster(tmp_path_factory):
    # one launch for more products than workspaces has no memory for a split.  Measured in one launch and split: 12 of 319x588x11522, four at
    # a time, 1114 and 986 us; the four of a complex 661x426x19376 1010 and 937, of 524x591x27591 1799 and 1594
    run = host_program(tmp_path_factory, "host_f64_together.cpp")
    split = [(319, 588, 11522, 1, 1, 12, 4, 36 << 20), (661, 426, 19376, 1, 0, 4, 1, 40 << 20), (524, 591, 27591, 0, 0, 4, 1, 46 << 20)]
    whole = [(96, 80, 112, 1, 0, 9, 4, 4 << 20), (500, 400, 300, 1, 0, 16, 2, 8 << 20), (100, 100, 2000, 1, 1, 24, 2, 6 << 20),
             (1000, 900, 700, 0, 0, 4, 1, 16 << 20)]
    # in one launch and split: the four of a complex 202x275x6305 91 and 116 us, of 534x109x3204 72 and 90, of 52x1197x3094 81 and 97
    whole += [(202, 275, 6305, 0, 0, 4, 1, 64 << 20), (534, 109, 3204, 0, 1, 4, 1, 64 << 20), (52, 1197, 3094, 0, 0, 4, 1, 64 << 20)]
    assert [r for r, in run(split + whole)] == [0] * 3 + [1] * 7


def test_small_outputs_with_a_long_k_are_split(tmp_path_factory):
    # 58x32x4432 behind a verdict that falls back takes 54 us unsplit and 33 in parts, 30x69x4823 41 and 30; 39x235x54713 59 us in twelve
    # parts on 32x32 tiles, which leave every fourth CU idle, and 48 in sixteen.  A short k stays whole
    run = host_program(tmp_path_factory, "host_f64_split.cpp")
    (*_, a), (*_, b), c, (*_, d) = run([(58, 32, 4432, 0, 0, 0, 1), (30, 69, 4823, 0, 0, 0, 1), (39, 235, 54713, 0, 1, 1, 0), (58, 32, 600, 0, 0, 0, 1)])
    assert a > 1 and b > 1 and list(c) == [32, 32, 16] and d == 1


def test_problems_that_cannot_share_units_take_tiles(tmp_path_factory):
    # 104 units a problem: on units four calls one after the other.  The four of a complex 1556x939x331 with counts per block take 317 us so
    # and 192 in one launch on tiles, of 2006x1146x1529 967 and 617
    run = host_program(tmp_path_factory, "host_call_plan.cpp")
    assert all(g != 0 for g, in run([(1556, 939, 331, 14, 7, 1, 4), (2006, 1146, 1529, 14, 7, 1, 4)]))
