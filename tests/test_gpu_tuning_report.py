"""rt_ctx_tuning reports the split that launches have: the workgroups of the
default one, tiles and shares cut at blocks otherwise."""
import pytest

from tests.gpu_helpers import say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1910_03517_amd import rt  # noqa: E402


def test_segments_of_each_split():
    say("case: rt_ctx_tuning, 1x640x480 and 14x1920x1080")
    one = rt.Rig([rt.Camera(640, 480, 3, 8, 0, 0).with_pitch()], rt.Options())
    assert one.tuning() == (32, 0, 160)           # 160 groups by 3 rows: 160 steps, a workgroup each
    one.tune(8, 0)
    assert one.tuning() == (8, 0, 64)             # blocks of 30 rows in four tiles
    one.tune(32, 7)
    assert one.tuning()[:2] == (32, 7) and one.tuning()[2] >= 16
    one.tune(32, 0)
    assert one.tuning() == (32, 0, 160)
    one.close()
    rig = rt.Rig([rt.Camera(1920, 1080, 3, 8, 0, p).with_pitch() for p in range(14)], rt.Options())
    assert rig.tuning() == (32, 0, 512)
    rig.close()
