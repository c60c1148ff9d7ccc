"""Attention windows over several column chunks, of the smallest and the largest
m, over cameras smaller than the grid, against the oracle."""
import numpy as np
import pytest

from tests.gpu_helpers import rt_cams, say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1910_03517_amd import rt, synth  # noqa: E402
from tests.test_gpu_attention import check, perturbed  # noqa: E402


@pytest.mark.parametrize("m", [1, 5, 64])
def test_attention_windows_over_column_chunks(m):
    say("case: windows m", m)
    rng = np.random.default_rng([53, m])
    spec = [synth.CamSpec(w, h, 1, 8, 0, p) for p, (w, h) in enumerate([(2051, 301), (900, 290), (40, 301)])]
    cams = rt_cams(spec, pad=1)
    rig = rt.Rig(cams, rt.Options(n_blocks=4, band_width=4))
    frames = [synth.tiny_frame(c.height, c.width, c.channels, c.bit_depth, rng) for c in cams]
    check(rig, cams, frames, perturbed(frames, rng, 8, 0.3), 20, 4, m, 3, f"m {m}")
    rig.close()
