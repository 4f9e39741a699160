"""The block kernels' launch plans on the CPU: every share of every key stream fits the kernels' slot tables.

A small program replays the cut that the kernels make at run time, with the library's own plans and the kernels'
own StreamCut (plan_check.cpp).  The tables' sizes are stated here a second time.
"""
import os
import random
import subprocess

import pytest

import paper_2606_00144_amd as bd
from paper_2606_00144_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TILE, RING = 32, 7                       # keys per tile; tiles that the prefetches run past a share's end
FWD_SLOTS = 2048 + (64 + RING) * TILE    # forward: one table for all pieces of a share
BWD_SLOTS = 4096 + RING * TILE           # backward: one piece at a time


@pytest.fixture(scope="module")
def replay(tmp_path_factory):
    if not os.path.exists(bd.library_path):
        build.build_library()
    exe = tmp_path_factory.mktemp("plans") / "plan_check"
    lib_dir = os.path.dirname(os.path.abspath(bd.library_path))
    r = subprocess.run([build.HIPCC, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", f"-I{build.INCLUDE}",
                        f"-I{build.CSRC}", os.path.join(ROOT, "tests", "plan_check.cpp"), "-x", "none",
                        bd.library_path, f"-Wl,-rpath,{lib_dir}", "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def run(cases):
        text = "".join(" ".join(map(str, (*c[:8], c[8], *c[9]))) + "\n" for c in cases)
        out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, timeout=300)
        assert out.returncode == 0, out.stderr
        rows = [tuple(map(int, line.split())) for line in out.stdout.splitlines()]
        assert len(rows) == len(cases)
        return rows

    return run


def _check(case, row):
    f_nw, tiles, over, f_wrong, b_nw, piece, b_wrong, stream_tiles = row
    assert f_wrong == 0 and b_wrong == 0, (case, row)
    assert over == 0, (case, row)
    assert (tiles + RING) * TILE <= FWD_SLOTS, (case, row)
    assert (-(-piece // TILE) + RING) * TILE <= BWD_SLOTS, (case, row)
    assert 1 <= b_nw <= max(1, stream_tiles), (case, row)     # no workgroup that could never hold an entry


def _case(S, Hkv, G, C, V, ld, L, full, lens=None, at=None):
    return (S, Hkv, Hkv * G, C, V, ld, L, int(full), L if at is None else at, [ld] * V if lens is None else lens)


def test_shares_at_the_tables_edges(replay):
    cases = []
    for units in [(8, 8, 4, 256), (8, 32, 4, 64), (9, 8, 4, 256), (1, 1, 1, 33), (3, 8, 1, 40), (5, 32, 1, 64)]:
        for L in [1, 31, 32, 33, 2047, 2048, 4062, 4063, 4064, 4095, 4096, 4097, 8126, 8127, 131072]:
            cases.append(_case(*units, 0, 0, L, True))
            for V, ld in [(1, 1), (1, 33), (4, 1), (4, 225), (63, 1), (63, 33), (63, 65)]:
                cases.append(_case(*units, V, ld, L, True))
                cases.append(_case(*units, V, ld, L, False))
        for total in (4095, 4096, 4097):                       # the backward's largest share, to the entry
            cases.append(_case(*units, 1, 800, total - 800, True))
    for c, row in zip(cases, replay(cases)):
        _check(c, row)


def test_shares_over_many_lengths(replay):
    r, cases = random.Random(11), []
    for _ in range(6000):
        V = r.choice([0, 1, 2, 4, 8, 31, 63])
        ld = r.choice([1, 32, 33, r.randint(1, 4096), 32 * r.randint(1, 64) + 1]) if V else 0
        full = V == 0 or r.random() < 0.8
        L = r.choice([r.randint(1, 9000), r.randint(1, 140000), 32 * r.randint(1, 300) + 1])
        short = r.random() < 0.5                                # the lengths are known only at run time
        lens = [r.choice([0, ld, r.randint(0, ld)]) if short else ld for _ in range(V)]
        cases.append(_case(r.choice([1, 2, 3, 8, 17, 64]), r.choice([1, 2, 8, 32]), r.choice([1, 4, 5]),
                           r.choice([8, 33, 64, 100, 256]), V, ld, L, full, lens, r.randint(0, L) if short else L))
    for c, row in zip(cases, replay(cases)):
        _check(c, row)


@pytest.mark.parametrize("V,ld,L", [(1, 32, 256), (1, 128, 1024), (0, 0, 1), (0, 0, 33)])
def test_backward_scratch_holds_no_empty_records(V, ld, L):
    # one record of 32 x 128 floats per wave and workgroup, one workgroup per tile of the stream at most
    nb = bd.lib().bd_multiview_attn_bwd_workspace_bytes(1, 1, 1, 16, V, ld, L, 1)
    tiles = (V * ld + L + TILE - 1) // TILE
    rest = 4 * (V + 1) * (16 * 2 * 128 + 2 * 32) + 3 * 256      # dK/dV partials and row statistics, aligned
    assert 0 < nb <= 2 ** 20 + tiles * 8 * 32 * 128 * 4 + rest
