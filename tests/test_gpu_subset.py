"""Launches over a part of a large rig (the default split is worked out in the
kernel then): rings of one camera of every format, from one camera to all but
one, through rt_frameset_batch, and rt_apply in both forms, 3x3 maps and the
look-ahead launch under rt_ctx_set_active; outputs and whole-frame statistics
equal those of the full rig, and nothing of an inactive camera changes."""
import numpy as np
import pytest

from tests.gpu_helpers import rt_cams, say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1910_03517_amd import rt, synth  # noqa: E402

OUT = ("band_hist", "band_sums", "whole_hist", "whole_sums", "params", "valid", "lut8", "q16", "weights")


def rig_of(n, rgb_only=False, **opts):
    kinds = [(3, 8), (1, 8), (1, 12)]
    spec = [synth.CamSpec(40 + 17 * (k % 5), 30 + 41 * (k % 4), *(kinds[0] if rgb_only else kinds[k % 3]), k, 0)
            for k in range(n)]
    return rt.Rig(rt_cams(spec), rt.Options(n_blocks=3, band_width=8, **opts)), spec


def frames_of(spec, seed):
    rng = np.random.default_rng(seed)
    return [rng.integers(0, 1 << c.bit_depth, (c.height, c.width, c.channels)).astype(np.uint8 if c.bit_depth == 8 else np.uint16)
            for c in spec]


MASKS = [(64, 1), (64, 1 << 63), (64, (1 << 64) - 2), (64, 0x8421084210842108), (5, 0b10110)]


@pytest.mark.parametrize("n,mask", MASKS, ids=lambda v: hex(v))
@pytest.mark.parametrize("vblend", [False, True])
def test_frameset_batch_equals_full_rig(n, mask, vblend):
    say("case: subset", n, hex(mask), vblend)
    rig, spec = rig_of(n, vblend=vblend)
    dev = rig.upload(frames_of(spec, [21, n]))
    full, part = rig.alloc_frames(), rig.alloc_frames()
    rig.frameset(dev, full)
    torch.cuda.synchronize()
    want = rig.bufs.host()
    for name in OUT:
        getattr(rig.bufs, name).fill_(0)
    rig.frameset_batch(mask, [f if (mask >> k) & 1 else None for k, f in enumerate(dev)],
                       [f if (mask >> k) & 1 else None for k, f in enumerate(part)])
    torch.cuda.synchronize()
    got = rig.bufs.host()
    for k in range(n):
        on = (mask >> k) & 1
        assert torch.equal(part[k], full[k] if on else torch.zeros_like(full[k])), f"camera {k}"
        for name in OUT:
            ref = want[name][k] if on else np.zeros_like(want[name][k])
            assert np.array_equal(got[name][k], ref), f"camera {k}: {name}"
    rig.close()


@pytest.mark.parametrize("n,mask", MASKS[2:], ids=lambda v: hex(v))
def test_set_active_equals_full_rig(n, mask):
    say("case: set_active", n, hex(mask))
    rig, spec = rig_of(n, rgb_only=True)
    dev = rig.upload(frames_of(spec, [22, n]))
    x = rt.CrossSet(rig.sizes)
    outs = {}
    for active in ((1 << n) - 1, mask):
        rig.set_active(active)
        for name in ("apply", "apply whole", "cross", "ahead"):
            out = rig.alloc_frames()
            rig.bufs.whole_hist.zero_()
            if name == "cross":
                rt.rt_frameset_cross(rig.ctx, dev, out, rig.bufs, x)
            elif name == "ahead":
                lut, whole = rt.LutSet(rig.sizes), rt.WholeSet(rig.sizes)
                rt.rt_frameset_ahead(rig.ctx, None, None, None, None, dev, lut, whole, rig.bufs)
                rt.rt_frameset_ahead(rig.ctx, dev, out, lut, whole, None, None, None, rig.bufs)
                rig.bufs.whole_hist.copy_(whole.whole_hist)
            else:
                if name == "apply":
                    rig.frameset(dev, rig.alloc_frames())
                rig.apply(dev, out, whole=name == "apply whole")
            torch.cuda.synchronize()
            outs[active, name] = out, rig.bufs.whole_hist.clone()
    for name in ("apply", "apply whole", "cross", "ahead"):
        (fo, fh), (po, ph) = outs[(1 << n) - 1, name], outs[mask, name]
        for k in range(n):
            on = (mask >> k) & 1
            assert torch.equal(po[k], fo[k] if on else torch.zeros_like(fo[k])), f"{name}: camera {k}"
            if on:
                assert torch.equal(ph[k], fh[k]), f"{name}: camera {k} whole_hist"
    rig.close()
