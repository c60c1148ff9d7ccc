"""The band pass at the edges of its walk: bands of more pixel groups than the
threads that take them, bands that start or end inside a dword or are no
multiple of four pixels, and blocks of no or few rows, plain and against a
previous frame, bit for bit against the oracle."""
import numpy as np
import pytest

from tests.gpu_helpers import assert_ints_equal, oracle_cams, oracle_opts, say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import ringcorr as rc  # noqa: E402
from paper_1910_03517_amd import rt  # noqa: E402

# (W, H, C, bit depth, NB, band width)
CASES = [
    (2, 5, 3, 8, 2, 1),
    (8, 3, 3, 8, 5, 4),             # blocks without rows
    (43, 66, 3, 8, 3, 7),
    (1031, 40, 3, 8, 2, 24),        # the right band starts inside a dword
    (1027, 33, 1, 8, 2, 30),
    (1025, 33, 1, 12, 2, 31),
    (2200, 9, 3, 8, 2, 1100),       # 275 groups per band row
    (4400, 5, 1, 16, 1, 2111),
]


@pytest.mark.parametrize("case", CASES, ids=["x".join(map(str, c)) for c in CASES])
def test_band_statistics_match_oracle(case):
    W, H, C, bd, NB, B = case
    say("case:", case)
    rng = np.random.default_rng([7, W, H, C, bd, NB, B])
    cams = [rt.Camera(W, H, C, bd, 0, p).with_pitch() for p in range(2)]
    opts = rt.Options(n_blocks=NB, band_width=B)
    rig = rt.Rig(cams, opts)
    dt = np.uint8 if bd == 8 else np.uint16
    prev = [rng.integers(0, 1 << bd, (H, W, C)).astype(dt) for _ in cams]
    frames = [np.where(rng.random((H, W, 1)) < 0.5, p, rng.integers(0, 1 << bd, p.shape)).astype(dt) for p in prev]
    dev, dprev = rig.upload(frames), rig.upload(prev)
    kept = torch.zeros((2, 2, NB, 3, 3), dtype=torch.int64, device="cuda")
    co, oo = oracle_cams(cams), oracle_opts(opts)
    for motion in (False, True):
        b = rig.bufs
        b.band_hist.fill_(-1)
        b.band_sums.fill_(-1)
        if motion:
            rt.rt_motion_stats(rig.ctx, dev, dprev, 20, 0.25, b.band_hist, b.band_sums, kept)
        else:
            rig.stats(dev, whole=False)
        torch.cuda.synchronize()
        h = b.host()
        for k in range(2):
            hist, sums = rc.band_stats(frames[k], co[k], oo)
            assert_ints_equal(h["band_hist"][k], hist, f"cam {k} band_hist motion={motion}")
            assert_ints_equal(h["band_sums"][k], sums, f"cam {k} band_sums motion={motion}")
            if motion:
                assert_ints_equal(kept[k].cpu().numpy(), rc.kept_band_sums(frames[k], prev[k], co[k], oo, 20),
                                  f"cam {k} kept sums")
    rig.close()
