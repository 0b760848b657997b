"""The launch rules of the stage kernel on the CPU: what the library chooses for
the knobs that are left to it, and that a knob keeps its meaning whatever the
others are set to or written back."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1912_05371_amd")
BIN = os.path.join(ROOT, "_build", "schedule_harness")
KNOBS = ("wg_per_cu", "xcd_map", "prefetch", "nontemporal", "tile_rows", "pen_split")
OWN = 3  # xcd_map of a launch with work counters of the call's own
SIZES = [(f64, bs, nb) for f64 in (1, 0) for bs in (16, 24, 32)
         for nb in (1, 64, 1727, 1728, 4095, 4096, 20028)]


@pytest.fixture(scope="module")
def harness():
    os.makedirs(os.path.dirname(BIN), exist_ok=True)
    subprocess.run(["/opt/rocm/bin/hipcc", "-x", "c++", "-D__HIP_PLATFORM_AMD__", "-O1", "-std=c++17",
                    "-I/opt/rocm/include", f"-I{os.path.join(ROOT, 'include')}",
                    f"-I{os.path.join(PKG, 'csrc')}", "-o", BIN,
                    os.path.join(ROOT, "tests", "schedule_harness.cpp"), "-x", "none",
                    os.path.join(PKG, "libwacm.so"), f"-Wl,-rpath,{PKG}"], check=True)
    return BIN


def run(harness, cases, early=False):
    """Per case (f64, bs, nb, counters, [(knob, value), ...]): the schedule read
    at the end, the RK stages' and the rhs's; with early, for 1, 2 and 4 runs of
    planes, whether the RK stages load their operands early."""
    text = "".join(f"{f} {bs} {nb} {c} {len(k)} " + " ".join(f"{a} {b}" for a, b in k) + "\n"
                   for f, bs, nb, c, k in cases)
    r = subprocess.run([harness], input=text, capture_output=True, text=True)
    assert r.returncode == 0, (r.returncode, r.stderr)
    rows = [[int(v) for v in line.split()] for line in r.stdout.splitlines()]
    return [tuple(dict(zip(KNOBS, v[i:i + 6])) for i in (0, 6, 12)) for v in rows] if not early \
        else [v[18:21] for v in rows]


@pytest.mark.parametrize("knobs", [[("none", 0)], [("pen_split", 0)], [("wg_per_cu", 2)],
                                   [("nontemporal", 0)], [("pen_split", 2), ("none", 0)]])
def test_an_unrelated_knob_keeps_the_others(harness, knobs):
    """(none: the schedule is written back as it was read)"""
    before = run(harness, [(*s, 1, []) for s in SIZES])
    after = run(harness, [(*s, 1, knobs) for s in SIZES])
    for size, b, a in zip(SIZES, before, after):
        for p, q in zip(b, a):
            for k in ("tile_rows", "prefetch", "xcd_map"):
                assert p[k] == q[k], (size, k)


def test_what_the_library_chooses(harness):
    got = run(harness, [(*s, 1, []) for s in SIZES])
    for (f64, bs, nb), (read, rk, _) in zip(SIZES, got):
        assert read == dict(wg_per_cu=0, xcd_map=-1, prefetch=-1, nontemporal=1, tile_rows=-1,
                            pen_split=1)
        large = nb * bs ** 3 >= 4096 * 24 ** 3 and (bs == 24 or (bs == 32 and f64))
        assert rk["xcd_map"] == (OWN if large else 1)
        assert rk["tile_rows"] == (8 if (f64 and bs >= 24) or large else 0)
    for (f64, bs, nb), (_, rk, _) in zip(SIZES, run(harness, [(*s, 0, []) for s in SIZES])):
        assert rk["xcd_map"] == 1 and rk["tile_rows"] == (8 if f64 and bs >= 24 else 0)


@pytest.mark.parametrize("knob,value", [("tile_rows", 0), ("tile_rows", 8), ("xcd_map", 0),
                                        ("xcd_map", 1), ("xcd_map", 2), ("prefetch", 0),
                                        ("prefetch", 1)])
def test_a_knob_that_is_set_is_taken_as_it_is(harness, knob, value):
    for rows in zip(SIZES, run(harness, [(*s, 1, [(knob, value)]) for s in SIZES]),
                    run(harness, [(*s, 1, []) for s in SIZES])):
        size, got, free = rows
        assert all(s[knob] == value for s in got), size
        for g, f in zip(got, free):
            # (the early loads go with tiles that the library chose)
            skip = (knob, "prefetch") if knob == "tile_rows" else (knob,)
            assert all(g[k] == f[k] for k in KNOBS if k not in skip), size


@pytest.mark.parametrize("tiles", [-1, 0, 8])
def test_early_loads_as_set_with_any_number_of_runs(harness, tiles):
    for value in (0, 1):
        knobs = [("tile_rows", tiles), ("prefetch", value)]
        for size, got in zip(SIZES, run(harness, [(*s, 1, knobs) for s in SIZES], early=True)):
            assert got == [value] * 3, (size, value)
    # left to the library: FP32, and FP64 tiles in whole columns where the tiles
    # are its own too
    for (f64, bs, nb), got in zip(SIZES, run(harness, [(*s, 1, [("tile_rows", tiles)])
                                                       for s in SIZES], early=True)):
        own = f64 and bs >= 24 and tiles < 0
        assert got == ([int(own), 0, 0] if f64 else [1, 1, 1]), (f64, bs, nb)


# (tiles, resident workgroups per compute unit, bs) on 256 compute units, and the
# runs of planes that were fastest, or within 3% of it
@pytest.mark.parametrize("tiles,per_cu,bs,runs", [
    (64, 2, 16, (4,)), (71, 4, 16, (4,)), (71, 1, 24, (2,)), (71, 1, 32, (2,)),
    (372, 4, 16, (2, 4)), (295, 1, 24, (2, 4)), (295, 1, 32, (2, 4)), (736, 2, 16, (2,)),
    # whole columns: 2 runs took 1.08, 1.11, 1.09, 1.07, 1.05, 1.05 and 1.11 times as long
    (442, 4, 16, (1, 4)), (498, 4, 16, (1, 4)), (589, 4, 16, (1, 4)), (1723, 2, 16, (1,)),
    (2612, 3, 16, (1,)), (2166, 2, 24, (1,)), (2712, 2, 24, (1,)),
    (20028, 2, 24, (1,)), (60084, 2, 24, (1,)),
])
def test_runs_of_planes(harness, tiles, per_cu, bs, runs):
    r = subprocess.run([harness, "runs"], input=f"{tiles} {per_cu} 256 {bs}\n",
                       capture_output=True, text=True)
    assert int(r.stdout) in runs
