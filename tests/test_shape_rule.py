"""The sweep shapes that the library gives an instance (no GPU needed): a
helper program linked with the library asks for them."""
import json
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
COMPUTE_UNITS = 256


@pytest.fixture(scope="module")
def shapes(tmp_path_factory):
    from paper_1710_09025_amd import build

    exe = str(tmp_path_factory.mktemp("shape") / "sweep_shape")
    lib = os.path.dirname(build.LIB)
    cmd = [build.hipcc(), "-x", "c++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", build.ROCM_INC,
           os.path.join(ROOT, "tests", "helpers", "sweep_shape.cpp"), "-o", exe, "-x", "none", build.LIB,
           f"-Wl,-rpath,{lib}", "-L", os.path.join(os.path.dirname(build.ROCM_INC), "lib"), "-lamdhip64"]
    subprocess.run(cmd, check=True, capture_output=True, text=True)

    def ask(*cases):
        """(dim, real, L, R, sweeps, tile_rows, group_replicas) each: dicts"""
        args = [str(int(v)) for c in cases for v in c]
        r = subprocess.run([exe, *args], check=True, capture_output=True, text=True)
        keys = ("status", "m", "sets", "tile_rows", "group", "blocks")
        return [dict(zip(keys, map(int, line.split()))) for line in r.stdout.splitlines()]

    return ask


def test_small_lattices_fill_the_chip(shapes):
    """A large population of a lattice of a few blocks: workgroups for every
    SIMD, not one of many waves in step for each compute unit."""
    for L, R in ((2, 100_000), (3, 100_000), (3, 200_000), (4, 100_000), (5, 100_000)):
        (s,) = shapes((3, 0, L, R, 10, 0, 0))
        assert s["status"] == 0 and R / s["tile_rows"] >= 4 * COMPUTE_UNITS, (L, R, s)


# (dim, real couplings, L, R, sweeps, tile_rows, group_replicas), draws of a lane
# in a colour step: 4 for each pass of the group's quads over the tile
EXPLICIT = [
    ((3, 0, 4, 1000, 10, 32, 32), 4), ((3, 0, 4, 1000, 10, 128, 64), 8), ((3, 0, 4, 20000, 10, 128, 64), 8),
    ((3, 0, 4, 1000, 10, 1000, 256), 16), ((3, 0, 5, 1000, 10, 40, 16), 12), ((3, 0, 5, 1000, 10, 128, 128), 4),
    ((3, 0, 6, 1000, 10, 64, 32), 8), ((3, 0, 7, 20000, 10, 64, 32), 8), ((3, 0, 8, 1000, 10, 64, 0), 16),
    ((3, 1, 4, 1000, 10, 128, 128), 4), ((3, 1, 6, 1000, 10, 256, 64), 16), ((3, 1, 8, 20000, 10, 64, 32), 8),
    ((2, 1, 16, 1000, 10, 64, 32), 8),
]


@pytest.mark.parametrize("case,draws", EXPLICIT)
def test_tiles_that_are_asked_for_use_the_lanes_they_have_rows_for(shapes, case, draws):
    """A workgroup sweeps its tile side by side, not a word of 32 replicas in a
    few lanes: no lane draws for more replicas than with quads."""
    (s,) = shapes(case)
    rows = min(case[5], case[3])
    passes = -(-rows // (s["m"] * s["sets"]))
    assert s["status"] == 0 and s["tile_rows"] == case[5]
    assert passes * s["m"] <= draws, (case, s)


@pytest.mark.parametrize("dim,real,sizes", [(3, 0, range(2, 33)), (3, 1, range(2, 22)), (2, 1, range(2, 65, 3))])
def test_reported_shapes_are_taken_back(shapes, dim, real, sizes):
    """tile_rows and group_replicas as pamc_sweep_shape gives them for a default
    shape, passed as options, are accepted and give that shape."""
    cases = [(dim, real, L, R, 10) for L in sizes for R in (1, 30, 1000, 20_000, 500_000)]
    first = shapes(*[c + (0, 0) for c in cases])
    again = shapes(*[c + (s["tile_rows"], s["group"]) for c, s in zip(cases, first)])
    for c, a, b in zip(cases, first, again):
        assert a["status"] == 0 and a == b, (c, a, b)


def test_measured_shapes_are_accepted(shapes):
    """What pamc_autotune reports for the sizes of the shipped file."""
    from paper_1710_09025_amd import build

    with open(os.path.join(os.path.dirname(build.LIB), "tune_cache.jsonl")) as f:
        lines = [json.loads(line) for line in f if line.strip()]
    cases = [(d["dim"], int(d["variant"] >= 128), d["L"], 1000, d["sweeps"], d["tile_rows"], 4 * d["group_quads"])
             for d in lines]
    for c, s in zip(cases, shapes(*cases)):
        assert s["status"] == 0 and s["tile_rows"] >= c[5], (c, s)


@pytest.mark.parametrize("case", [(3, 0, 8, 1000, 10, 16, 2000), (3, 0, 24, 100, 10, 4, 1028), (3, 0, 4, 1000, 10, 8, 1028),
                                  (3, 0, 10, 1000, 10, 0, 64), (3, 0, 4, 1000, 10, 7, 8), (3, 1, 16, 100, 10, 5, 12)])
def test_other_pairs_stay_refused(shapes, case):
    """A group beyond its range, and pairs that nothing reports."""
    (s,) = shapes(case)
    assert s["status"] != 0, (case, s)
