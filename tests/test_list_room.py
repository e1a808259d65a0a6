"""Host-side check of the lists the force pass holds for a batch of boxes (no GPU).

Compiled from the library's own header: however the particles are spread over boxes, the lists take no more than 64
bytes a particle and a constant, a single box always has the room its parts are cut for, and small batches too.
"""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SLOT, ITEM = 32, 16     # bytes


@pytest.fixture(scope="module")
def printed(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("room") / "list_room")
    r = subprocess.run([hipcc, "-O1", "-o", exe, os.path.join(HERE, "list_room_main.cpp")], capture_output=True,
                       text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return subprocess.run([exe], capture_output=True, text=True, check=True).stdout.split("\n\n")


@pytest.fixture(scope="module")
def rooms(printed):
    names = ("boxes", "n", "cells", "slots", "items", "box_slots", "box_items", "least_slots", "least_items")
    return [dict(zip(names, map(int, line.split()))) for line in printed[0].splitlines()]


def test_lists_take_64_bytes_a_particle_and_a_constant(rooms):
    for r in rooms:
        assert SLOT * r["slots"] <= 64 * r["n"] + 4.3e9, r
        assert ITEM * r["items"] <= ITEM * (min(r["n"], r["cells"]) + 0.16 * r["n"]) + 0.28e9, r


def test_one_box_and_small_batches_have_the_room_their_parts_are_cut_for(rooms):
    for r in rooms:
        if r["boxes"] == 1 and r["box_items"] < 2 ** 31 or 66 * r["n"] < 1 << 24:
            assert r["slots"] >= r["box_slots"] and r["items"] >= r["box_items"], r


def test_least_lists_hold_a_slot_per_particle_and_every_unsplit_item(rooms):
    for r in rooms:
        assert r["least_slots"] == r["n"], r
        unsplit = min(r["n"], r["cells"]) + r["n"] // 64 + r["n"] // 11
        assert r["least_items"] >= min(unsplit, 2 ** 31 - 2), r


def test_parts_are_short_only_where_the_box_gives_few_items(printed):
    for line in printed[1].splitlines():
        S, pairs, least = map(int, line.split())
        assert 256 <= least <= 512, line
        if least > 256:      # parts of this length still give about 2700 items
            assert pairs // (64 * S * least) >= 2700, line
        if least < 512:
            assert pairs // (64 * S * (least + 1)) < 2700, line
