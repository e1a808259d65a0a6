"""Host-side check of the plan of the sort by cell (no GPU).

The plan is compiled from the library's own header into a small host program, which prints it for every key width
from 5 bits (27 cells, the fewest a box may have) to 31 (2^31 - 2 cells, the most) at the edges of the tile sizes and
up to the largest call.  Checked: the digits make up the key, fit the kernels' tables and LDS, and every array lies
inside the scratch of the call and of any larger call's handle.
"""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LDS = 160 * 1024
SCAN = 4096            # elements a workgroup of a scan takes


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    exe = str(tmp_path_factory.mktemp("plan") / "sort_plan")
    r = subprocess.run([cxx, "-std=c++17", "-O1", "-o", exe, os.path.join(HERE, "sort_plan_main.cpp")],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    out = subprocess.run([exe], capture_output=True, text=True, check=True).stdout.splitlines()
    names = ("n", "bits", "tile", "part", "mid", "last", "dbase", "rows", "total", "handle", "run")
    return tuple(map(int, out[0].split())), [dict(zip(names, map(int, line.split()))) for line in out[1:]]


def test_every_key_width_fits_the_tables_and_lds(plans):
    (buckets, most_small, most_big, _), rows = plans
    assert {r["bits"] for r in rows} == set(range(5, 32))
    for r in rows:
        assert r["part"] + r["mid"] + r["last"] == r["bits"], r
        assert 1 << r["part"] <= buckets, r
        most = most_big if r["tile"] == 4096 else most_small
        threads = 1024 if r["tile"] == 4096 else 256
        # a digit of a bucket is scanned four counts to a thread
        assert 2 <= r["last"] <= most and (r["mid"] == 0 or 2 <= r["mid"] <= most), r
        assert r["part"] > 0 or r["mid"] == 0, r
        for bits in (r["part"], r["mid"], r["last"]):
            d, waves = 1 << bits, threads // 64
            assert 20 * min(r["tile"], 2048) + 4 * d + 4 * waves + 2 * waves * d <= LDS, r


def test_every_array_lies_inside_the_scratch(plans):
    (_, _, _, struct), rows = plans
    for r in rows:
        tiles, nb, digit = -(-r["n"] // r["tile"]), 1 << r["part"], max(r["mid"], r["last"])
        assert r["dbase"] >= struct and r["dbase"] % 256 == 0 and r["rows"] % 256 == 0, r
        assert r["rows"] - r["dbase"] >= 4 * (nb << digit), r             # first slot of every bucket's digits
        # counts of every tile, an empty bucket has one
        assert r["total"] - r["rows"] >= 4 * ((tiles + (nb if r["part"] else 0)) << digit), r
        if r["part"]:                                                     # the partition's counts, their sums, the scan's
            need, n = 2 * 4 * nb * tiles + 255, nb * tiles
            while n > SCAN:
                n = -(-n // SCAN)
                need += 2 * 4 * n + 255
            assert r["total"] - r["rows"] >= need, r
        assert r["handle"] >= r["total"], r


def test_no_workgroup_walks_all_tiles_of_a_large_call(plans):
    """The digit sums of a bucket that holds every particle: a run of tiles, then the runs, each a few hundred rows."""
    _, rows = plans
    for r in rows:
        tiles, run = -(-r["n"] // r["tile"]), r["run"]
        runs = -(-tiles // run)
        assert run >= 128 and runs <= 2 * run, r
        assert run == 128 or tiles > run * run // 2, r
        digit, nb = max(r["mid"], r["last"]), 1 << r["part"]
        assert r["rows"] - r["dbase"] >= 4 * ((tiles // run + nb) << digit), r
        # few cells: one digit, however many particles
        assert r["bits"] > 8 or (r["part"], r["mid"]) == (0, 0), r


def test_a_handle_has_room_for_every_smaller_call(plans):
    _, rows = plans
    for big in rows:
        for r in rows:
            if r["n"] <= big["n"] and r["bits"] <= big["bits"]:
                assert big["handle"] >= r["total"], (big, r)
