"""Training steps of the surrogate network at the edges of their launch forms:
rt_mlp_train against the separate calls bit for bit, per-step losses, gradients
and gathered rows included, on both sides of 256 rows (weight gradients, Adam
and loss in one launch) and of 2048 (rows read through the indices); and the
loss gradient of the second hidden layer rounded once per term."""
import numpy as np
import pytest

from tests.gpu_helpers import say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1910_03517_amd import rt, synth  # noqa: E402

F32 = dict(device="cuda", dtype=torch.float32)
WIDTHS = {"xb": 576, "tb": 6, "h1": 256, "h2": 256, "y": 6, "dy": 6, "dz1": 256, "dz2": 256}


def work_of(n):
    return {k: torch.zeros((n, c), **F32) for k, c in WIDTHS.items()}


@pytest.mark.parametrize("batch", [1, 63, 255, 256, 257, 1024, 2047, 2048, 2049])
def test_train_equals_separate_calls(batch):
    say("case: train", batch)
    rng = np.random.default_rng([31, batch])
    steps, n = 3, 3 * batch + 5
    X = torch.as_tensor(rng.uniform(0, 2, (n, 576)).astype(np.float32), device="cuda")
    T = torch.as_tensor(rng.normal(1, 0.3, (n, 6)).astype(np.float32), device="cuda")
    idx = torch.as_tensor(rng.permutation(n)[:steps * batch].astype(np.int32), device="cuda")
    P = synth.mlp_init(4)
    nets = [[rt.MlpTensors(P)] + [rt.MlpTensors(None) for _ in range(3)] for _ in range(2)]     # w, g, m, v
    a, b = work_of(batch), work_of(batch)
    la, lb = torch.full((steps,), -1.0, **F32), torch.full((steps,), -1.0, **F32)
    w, g, m, v = nets[0]
    rt.rt_mlp_train(w, g, m, v, X, T, idx, batch, steps, 7, 3e-3, a, la)
    w, g, m, v = nets[1]
    for s in range(steps):
        rows = idx[s * batch:(s + 1) * batch]
        rt.rt_gather_rows(X, 576, rows, batch, b["xb"])
        rt.rt_gather_rows(T, 6, rows, batch, b["tb"])
        rt.rt_mlp_forward(w, b["xb"], batch, b["h1"], b["h2"], b["y"])
        rt.rt_mlp_backward(w, b["xb"], b["h1"], b["h2"], b["y"], b["tb"], batch, g, b["dy"], b["dz1"], b["dz2"])
        rt.rt_mlp_adam(w, g, m, v, 7 + s, 3e-3)
        rt.rt_mlp_mse(b["y"], b["tb"], batch, lb[s:s + 1])
    torch.cuda.synchronize()
    assert torch.equal(la, lb)
    for k in WIDTHS:
        assert torch.equal(a[k], b[k]), k
    for x, y in zip(*nets):
        hx, hy = x.host(), y.host()
        for k in rt.MlpTensors.NAMES:
            assert np.array_equal(hx[k], hy[k]), k


def test_hidden_gradient_is_rounded_once_per_term():
    """dZ2 = (dY W3^T) where H2 > 0 as six fused multiply-adds: each term and sum
    exact in 80 bits, then rounded to float32 once (the few sums that do not
    fit 64 bits of mantissa may differ in the last place)."""
    say("case: dZ2, 300 rows")
    rng = np.random.default_rng(32)
    n = 300
    P = synth.mlp_init(6)
    w, g, k = rt.MlpTensors(P), rt.MlpTensors(None), work_of(n)
    X = torch.as_tensor(rng.uniform(0, 0.2, (n, 576)).astype(np.float32), device="cuda")
    T = torch.as_tensor(rng.normal(1, 0.3, (n, 6)).astype(np.float32), device="cuda")
    rt.rt_mlp_forward(w, X, n, k["h1"], k["h2"], k["y"])
    rt.rt_mlp_backward(w, X, k["h1"], k["h2"], k["y"], T, n, g, k["dy"], k["dz1"], k["dz2"])
    torch.cuda.synchronize()
    dy, h2, z = (k[name].cpu().numpy() for name in ("dy", "h2", "dz2"))
    W3 = P["w3"].reshape(256, 6)
    t = np.zeros((n, 256), np.float32)
    for o in range(6):
        t = (np.longdouble(dy[:, o:o + 1]) * np.longdouble(W3[:, o][None]) + np.longdouble(t)).astype(np.float32)
    ref = np.where(h2 > 0, t, np.float32(0))
    assert np.mean(z != ref) < 1e-3
    assert np.max(np.abs(z - ref) / np.maximum(np.spacing(np.abs(ref)), 1e-38)) <= 1.0
