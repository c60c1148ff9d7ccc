"""The apply pass's default split of a camera's rows into runs (CPU): every row
in exactly one run, a run that ends at its own last row, and no run whose rows
span many more blocks than it has steps (a workgroup looks at and stages the
maps of all blocks between its first and its last row), unless it has four
steps or more and all maps are staged at once.  And of the workgroups
among the cameras of a launch: by their bytes over the active ones, whatever
the rest of the rig is.  And of a workgroup's threads over the rows: the least
cost, in steps and serial trips to memory, of the splits into column chunks."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
GXX = shutil.which("g++")
pytestmark = pytest.mark.skipif(GXX is None, reason="no g++")


def compile_host(tmp, name):
    """A program of tests/split, with the headers' device attributes defined away."""
    exe = os.path.join(tmp, name)
    subprocess.run([GXX, "-std=c++17", "-Wall", "-D__host__=", "-D__device__=",
                    os.path.join(HERE, "split", name + ".cpp"), "-o", exe], check=True)
    return exe


@pytest.fixture(scope="module")
def row_runs(tmp_path_factory):
    exe = compile_host(str(tmp_path_factory.mktemp("split")), "row_runs")

    def get(H, lanes, m, nb):
        out = subprocess.run([exe, str(H), str(lanes), str(m), str(nb)], check=True, capture_output=True, text=True)
        runs = [tuple(int(v) for v in ln.split()) for ln in out.stdout.splitlines()]
        assert len(runs) == 2 * m
        return runs[:m], runs[m:]

    return get


# (height, rows at a time, runs, blocks)
CASES = [(1, 1, 1, 1), (1, 512, 1, 16), (7, 3, 3, 16), (40, 2, 20, 64), (480, 16, 30, 16), (480, 3, 160, 16),
         (517, 11, 47, 7), (720, 8, 85, 64), (1080, 1, 36, 16), (1080, 1, 37, 64), (1080, 1, 256, 256),
         (1080, 1, 512, 1024), (2160, 2, 79, 16), (2160, 1, 79, 1024), (32768, 1, 512, 16), (32768, 256, 128, 1000),
         (32767, 5, 8, 3)]


@pytest.mark.parametrize("H,lanes,m,nb", CASES)
def test_runs_cover_rows_and_span_few_blocks(row_runs, H, lanes, m, nb):
    for runs, table_form in zip(row_runs(H, lanes, m, nb), (False, True)):
        rows = [0] * H
        for row0, row1, stride in runs:
            assert 0 <= row0 < row1 <= H and stride >= lanes
            own = [r for s in range(row0, row1, stride) for r in range(s, min(s + lanes, row1))]
            for r in own:
                rows[r] += 1
            assert own[-1] == row1 - 1
            block = lambda r: ((r + 1) * nb - 1) // H
            spanned = block(row1 - 1) - block(row0) + 1
            steps = -(-(row1 - row0) // stride)
            if table_form:
                assert stride == lanes
            # The blocks of its own rows if they were contiguous, or one a step.
            few = spanned <= max(len(own) * nb // H + 2, steps)
            assert few or (not table_form and steps >= 4 and nb <= 64)
        assert rows == [1] * H


@pytest.fixture(scope="module")
def shares(tmp_path_factory):
    exe = compile_host(str(tmp_path_factory.mktemp("shares")), "shares")

    def get(cams, active):
        out = subprocess.run([exe, str(active)] + [f"{b}:{s}" for b, s in cams], check=True,
                             capture_output=True, text=True)
        first = [int(v) for v in out.stdout.split()]
        assert len(first) == len(cams) + 1 and first[0] == 0
        return [b - a for a, b in zip(first, first[1:])]

    return get


HD, VGA, UHD, TINY = (1080 * 5760, 1080), (480 * 1920, 160), (2160 * 12288, 2160), (100, 1)


@pytest.mark.parametrize("cams,active", [
    ([HD] * 14, (1 << 14) - 1), ([HD] * 14, 1), ([HD] * 14, 0x2a), ([HD] * 32, 1 << 31), ([VGA] * 60, 0xff),
    ([VGA] * 64, (1 << 64) - 1), ([VGA] * 64, 1 << 63), ([UHD] * 4 + [HD] * 8 + [VGA] * 4, 0xffff),
    ([UHD] + [VGA] * 12, 2), ([TINY] * 3, 7), ([TINY, UHD], 3), ([(2 ** 31 - 1, 32768)] * 64, (1 << 64) - 1)])
def test_shares_follow_the_active_cameras(shares, cams, active):
    got = shares(cams, active)
    on = [k for k in range(len(cams)) if (active >> k) & 1]
    total = sum(cams[k][0] for k in on)
    workgroups = 256 if sum(cams[k][1] for k in on) <= 12 * 256 else 512
    for k, m in enumerate(got):
        if k not in on:
            assert m == 0
            continue
        fair = 1 + (workgroups - len(on)) * cams[k][0] / total
        assert 1 <= m <= cams[k][1]
        assert m == cams[k][1] or abs(m - fair) < 1.0 + 1e-9
    assert sum(got) <= workgroups
    # A part of a rig is served as a rig of those cameras alone.
    assert [got[k] for k in on] == shares([cams[k] for k in on], (1 << len(on)) - 1)


@pytest.fixture(scope="module")
def layout(tmp_path_factory):
    exe = compile_host(str(tmp_path_factory.mktemp("layout")), "layout")

    def get(width, height, share, max_lanes=512):
        out = subprocess.run([exe, str(-(-width // 4)), str(height), str(share), str(max_lanes)], check=True,
                             capture_output=True, text=True)
        return tuple(int(v) for v in out.stdout.split())

    return get


def cost(groups, height, share, cols, lanes):
    steps, chunks = -(-height // lanes), -(-groups // cols)
    run = -(-steps // min(share, steps))
    return chunks * (run + 2 * -(-run // 6) + 2)


@pytest.mark.parametrize("width,height,share,max_lanes", [
    (1, 1, 1, 512), (4, 32768, 512, 512), (4, 32768, 8, 32), (200, 150, 170, 512), (333, 251, 60, 512), (640, 480, 512, 512),
    (640, 480, 170, 512), (640, 480, 8, 512), (640, 512, 12, 32), (719, 405, 200, 512), (1031, 517, 90, 512),
    (1031, 517, 4, 512), (1280, 720, 85, 512), (1920, 1080, 36, 512), (1920, 1080, 512, 32), (2047, 9, 200, 512),
    (2050, 7, 200, 512), (4096, 2160, 79, 512), (32768, 32768, 512, 512), (32767, 3, 1, 32)])
def test_layout_costs_least(layout, width, height, share, max_lanes):
    cols, lanes, total = layout(width, height, share, max_lanes)
    groups = -(-width // 4)
    assert 1 <= cols and 1 <= lanes <= max_lanes and cols * lanes <= 512
    options = [(c, min(512 // c, max_lanes)) for c in {-(-groups // n) for n in range(1, 9)} if c <= 512]
    assert all(cost(groups, height, share, cols, lanes) <= cost(groups, height, share, c, l) for c, l in options)
    assert total == (256 if -(-height // lanes) <= 12 * 256 else 512)


def test_small_image_keeps_the_chip_busy(layout, shares):
    cols, lanes, total = layout(640, 480, 512)
    assert (cols, lanes) == (160, 3)
    assert shares([(480 * 1920, -(-480 // lanes))], 1) == [160]


def test_ordinary_forms_keep_rows_in_flight(tmp_path):
    compile_host(str(tmp_path), "rows_in_flight")
