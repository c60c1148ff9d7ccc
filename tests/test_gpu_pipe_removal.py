"""Object removal through the pipeline takes the narrow seam form: bands of odd
widths and unaligned starts, blocks without rows, open chains and every sample
format against rt_frameset_removal call by call, bit for bit."""
import numpy as np
import pytest

from tests.gpu_helpers import rt_cams, say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1910_03517_amd import rt, synth  # noqa: E402

# (W, H, channels, bit depth, cameras, blocks, band, closed)
CASES = [(67, 35, 3, 8, 3, 5, 7, True), (1, 3, 3, 8, 2, 2, 4, True), (41, 5, 3, 8, 2, 8, 9, False),
         (130, 90, 1, 8, 3, 4, 33, False), (75, 64, 1, 12, 2, 3, 13, True), (320, 96, 3, 8, 1, 4, 32, True),
         (640, 200, 3, 8, 2, 2, 64, True)]


@pytest.mark.parametrize("fuse", [False, True])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_pipe_removal_equals_calls(case, fuse):
    W, H, C, bd, K, NB, band, closed = case
    say("case:", case, fuse)
    rng = np.random.default_rng([41, W, H, C, bd])
    cams = rt_cams([synth.CamSpec(W, H, C, bd, 0, p) for p in range(K)])
    opts = rt.Options(n_blocks=NB, band_width=band, closed_ring=closed, smoothing=True)
    one, two = rt.Rig(cams, opts), rt.Rig(cams, opts)
    base = [rng.integers(0, 1 << bd, (H, W, C)) for _ in cams]
    dt = np.uint8 if bd == 8 else np.uint16
    sets = []
    for t in range(5):
        now = []
        for f in base:
            f = np.clip(f + rng.integers(-3, 4, f.shape), 0, (1 << bd) - 1)
            f[:H // (2 + t % 2), :] = rng.integers(0, 1 << bd, (1, 1, C))      # a large object moves
            now.append(f.astype(dt))
        sets.append(one.upload(now))
    shape = (K, 2, NB)
    e = dict(device="cuda")
    kept = [torch.zeros(shape + (3, 3), dtype=torch.int64, **e) for _ in range(2)]
    method = [torch.zeros(shape, dtype=torch.uint8, **e) for _ in range(2)]
    want = [one.alloc_frames() for _ in sets]
    for t, f in enumerate(sets):
        one.frameset_removal(f, sets[t - 1] if t else None, want[t], kept[0], method[0])
    got = [two.alloc_frames() for _ in sets]
    pipe = rt.Pipe.for_rig(two, depth=4, lanes=2, group=2, fuse=fuse)
    pipe.set_removal(kept[1], method[1])
    pipe.submit_n(sets, got)
    pipe.join()
    torch.cuda.synchronize()
    for t in range(len(sets)):
        for k in range(K):
            assert torch.equal(got[t][k], want[t][k]), (t, k)
    assert torch.equal(kept[0], kept[1]) and torch.equal(method[0], method[1])
    a, b = one.bufs.host(), two.bufs.host()
    for name in ("band_hist", "band_sums", "params", "valid"):
        assert np.array_equal(a[name], b[name]), name
    pipe.close()
    one.close()
    two.close()
