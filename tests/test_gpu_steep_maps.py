"""Maps at the edge of 32-bit arithmetic in some blocks of a camera and small
ones in the others: the apply pass takes each in its own form, bit for bit
against the oracle, and a steep block costs little more than its own rows."""
import numpy as np
import pytest

from tests.gpu_helpers import assert_ints_equal, oracle_cams, oracle_opts, say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import crossmap as cm  # noqa: E402
from oracle import ringcorr as rc  # noqa: E402
from paper_1910_03517_amd import rt  # noqa: E402

EDGE = [(1 << 23) - 1, 1 << 23, 127 << 16, 255 << 16, 128 << 16]     # slopes in Q16
OFFSET = [0, -(1 << 30), (1 << 31) - 1 - 32768, (1 << 31) - 32768, -(1 << 31), -255 * ((1 << 23) - 1)]

# (W, H, C, cameras, NB, vblend); the last rig has interleaved runs of several blocks
RIGS = [(61, 130, 3, 2, 5, False), (61, 130, 3, 2, 5, True), (61, 67, 1, 2, 3, False), (45, 67, 1, 2, 3, True),
        (1024, 64, 3, 64, 4, False), (1024, 64, 3, 64, 4, True)]


def steep_params(rng, K, NB, blocks):
    p = np.zeros((K, 2, NB, 3, 2))
    p[..., 0] = rng.uniform(0.25, 2.0, p.shape[:-1])
    p[..., 1] = rng.uniform(-40.0, 40.0, p.shape[:-1])
    for j in blocks:
        p[:, :, j, :, 0] = rng.choice(EDGE, (K, 2, 3)) / 65536.0
        p[:, :, j, :, 1] = rng.choice(OFFSET, (K, 2, 3)) / 65536.0
    return p


@pytest.mark.parametrize("rig_case", RIGS, ids=["x".join(map(str, r)) for r in RIGS])
@pytest.mark.parametrize("blocks", [(0,), (1, 2), (-1,)], ids=str)
def test_steep_blocks_match_oracle(rig_case, blocks):
    W, H, C, K, NB, vb = rig_case
    say("case:", rig_case, blocks)
    rng = np.random.default_rng([9, W, H, C, vb, len(blocks), NB + blocks[0]])
    cams = [rt.Camera(W, H, C, 8, 0, p).with_pitch() for p in range(K)]
    opts = rt.Options(n_blocks=NB, band_width=8, vblend=vb, a_max=256.0)
    rig = rt.Rig(cams, opts)
    frames = [rng.integers(0, 256, (H, W, C)).astype(np.uint8) for _ in cams]
    rig.bufs.params.copy_(torch.from_numpy(steep_params(rng, K, NB, blocks)))
    rig.build_lut()
    dev, out = rig.upload(frames), rig.alloc_frames()
    co, oo = oracle_cams(cams), oracle_opts(opts)
    for grid in (0, 1):
        rig.tune(32, grid)
        rig.apply(dev, out, whole=True)
        torch.cuda.synchronize()
        h, got = rig.bufs.host(), rig.download(out)
        for k in sorted({0, 1, K - 1}):
            ref = (rc.apply_camera_vblend(frames[k], co[k], oo, h["q16"][k]) if vb else
                   rc.apply_camera(frames[k], co[k], oo, h["lut8"][k], h["q16"][k]))
            assert_ints_equal(got[k], ref, f"cam {k} grid {grid}")
            assert_ints_equal(h["whole_hist"][k], rc.whole_stats(frames[k], co[k])[0], f"cam {k} whole_hist")
    rig.close()


@pytest.mark.parametrize("K,W,H,NB", [(2, 61, 130, 5), (40, 1024, 64, 4)])
def test_steep_cross_maps_match_oracle(K, W, H, NB):
    say("case: cross", K, W, H, NB)
    rng = np.random.default_rng([10, K, W])
    cams = [rt.Camera(W, H, 3, 8, 0, p).with_pitch() for p in range(K)]
    opts = rt.Options(n_blocks=NB, band_width=8, a_max=256.0)
    rig = rt.Rig(cams, opts)
    frames = [rng.integers(0, 256, (H, W, 3)).astype(np.uint8) for _ in cams]
    x = rt.CrossSet(rig.sizes)
    p = rng.uniform(-1.0, 1.0, (K, 2, NB, 12))
    p[..., 9:] *= 60.0
    p[:, :, 1, :9] = rng.choice([127.0, -127.0, 128.0, 0.0, (2 ** 23 - 1) / 65536.0], (K, 2, 9))
    p[:, :, 1, 9:] = rng.choice([0.0, -16000.0, 32767.0, -32768.0], (K, 2, 3))
    p[:, :, 2, :3] = 42.0                      # in range as a whole row: 3 x 42 x 255 below 2^15
    x.params3.copy_(torch.from_numpy(p))
    rt.rt_build_cross(rig.ctx, x)
    dev, out = rig.upload(frames), rig.alloc_frames()
    rt.rt_apply_cross(rig.ctx, dev, out, x, rig.bufs.whole_hist, rig.bufs.whole_sums)
    torch.cuda.synchronize()
    got, q = rig.download(out), x.host()["q3"]
    for k in sorted({0, 1, K - 1}):
        assert_ints_equal(got[k], cm.apply_camera_cross(frames[k], oracle_cams(cams)[k], oracle_opts(opts), q[k]), f"cam {k}")
    rig.close()


def test_one_steep_block_costs_little():
    """One block of sixteen beyond 32-bit arithmetic: the exact form takes up to
    three times a fast block's time, so at most 1 + 2 / 16 of the pass without
    it, and a tenth for the spread of the measurement."""
    say("case: time of a steep block, 8x1920x1080")
    cams = [rt.Camera(1920, 1080, 3, 8, 0, p).with_pitch() for p in range(8)]
    rig = rt.Rig(cams, rt.Options(a_max=256.0))
    gen = torch.Generator(device="cuda").manual_seed(3)
    dev = [torch.randint(0, 256, (1080, c.pitch_bytes), generator=gen, dtype=torch.uint8, device="cuda") for c in cams]
    out = rig.alloc_frames()

    def apply_us():
        for _ in range(5):
            rig.apply(dev, out, whole=True)
        rt.rt_ctx_timing(rig.ctx, 60, 1)
        for _ in range(60):
            rig.apply(dev, out, whole=True)
        t = sorted(rt.rt_ctx_apply_times(rig.ctx, 60))
        rt.rt_ctx_timing(rig.ctx, 0, 1)
        return t[30] * 1e3

    rig.frameset(dev, out)
    small = apply_us()
    rig.bufs.params[:, :, 5, :, 0] = 200.0
    rig.build_lut()
    steep = apply_us()
    say(f"  {small:.1f} -> {steep:.1f} us")
    assert steep <= (1.0 + 2.0 / 16.0 + 0.1) * small
    rig.close()
