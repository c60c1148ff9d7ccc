"""The apply pass at the edges of its split: images of more groups than a
workgroup's threads (column chunks), fewer rows than a workgroup takes at a
time, a group across the image centre together with a ragged row end, runs of
more blocks than the staged maps hold, and maps that do not fit 32-bit
arithmetic, each with the default split and with few long runs, bit for bit
against the oracle."""
import numpy as np
import pytest

from tests.gpu_helpers import assert_ints_equal, oracle_cams, oracle_opts, say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import ringcorr as rc  # noqa: E402
from paper_1910_03517_amd import rt  # noqa: E402

# (W, H, C, bit depth, NB, vblend, largest |a|)
CASES = [
    (2, 3, 3, 8, 1, False, 2.0),
    (2047, 9, 3, 8, 2, False, 2.0),       # 512 groups, the last one ragged
    (2050, 7, 3, 8, 3, False, 2.0),       # two column chunks, the centre inside a group
    (4099, 5, 1, 8, 2, False, 2.0),
    (6147, 4, 1, 12, 2, False, 2.0),
    (35, 517, 3, 8, 200, False, 2.0),     # more blocks in a run than fit at once
    (35, 517, 1, 16, 200, False, 2.0),
    (35, 40, 3, 8, 64, False, 2.0),       # blocks without rows
    (35, 517, 3, 8, 5, True, 2.0),        # row maps in several pieces
    (45, 67, 3, 8, 3, False, 200.0),      # beyond 32-bit arithmetic: the tables
    (45, 67, 3, 8, 3, True, 200.0),       # the same, blended between blocks
    (45, 300, 1, 10, 3, True, 200.0),
]


@pytest.mark.parametrize("grid", [0, 1, 3])
@pytest.mark.parametrize("case", CASES, ids=["x".join(map(str, c)) for c in CASES])
def test_apply_runs_match_oracle(case, grid):
    W, H, C, bd, NB, vb, amax = case
    say("case:", case, "grid", grid)
    rng = np.random.default_rng([5, W, H, C, bd, NB, grid])
    cams = [rt.Camera(W, H, C, bd, 0, p).with_pitch() for p in range(2)]
    opts = rt.Options(n_blocks=NB, band_width=8, vblend=vb, a_max=256.0)
    rig = rt.Rig(cams, opts)
    if grid:
        rig.tune(32, grid)
    dt = np.uint8 if bd == 8 else np.uint16
    frames = [rng.integers(0, 1 << bd, (H, W, C)).astype(dt) for _ in cams]
    top = float((1 << bd) - 1)
    p = np.zeros((2, 2, NB, 3, 2))
    p[..., 0] = rng.uniform(0.25, amax, p.shape[:-1])
    p[..., 1] = rng.uniform(-0.5, 0.5, p.shape[:-1]) * top
    rig.bufs.params.copy_(torch.from_numpy(p))
    rig.build_lut()
    dev, out = rig.upload(frames), rig.alloc_frames()
    co, oo = oracle_cams(cams), oracle_opts(opts)
    for whole in (True, False):
        rig.apply(dev, out, whole=whole)
        torch.cuda.synchronize()
        h, got = rig.bufs.host(), rig.download(out)
        for k in range(2):
            ref = (rc.apply_camera_vblend(frames[k], co[k], oo, h["q16"][k]) if vb else
                   rc.apply_camera(frames[k], co[k], oo, h["lut8"][k], h["q16"][k]))
            assert_ints_equal(got[k], ref, f"cam {k} whole={whole}")
            wh, ws = rc.whole_stats(frames[k], co[k])
            assert_ints_equal(h["whole_hist"][k], wh, f"cam {k} whole_hist")
            assert_ints_equal(h["whole_sums"][k], ws, f"cam {k} whole_sums")
    rig.close()
