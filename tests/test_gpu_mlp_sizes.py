"""The network's passes at the edges of the kernels' tiles: rows around the
16-row blocks and the 32-row rounds of the gradient waves, hidden sizes around
the 16-column tiles, the 4-wide products and the limit of the fused passes.
Gradients against the fp64 network: |g - r| <= 2^-23 sqrt(n + 2 H) times the
largest magnitude that the same sums of absolute values reach."""
import numpy as np
import pytest
import torch

import paper_2508_07071_amd as fk

pytestmark = pytest.mark.gpu
F, O = fk.FK_MODEL_FEATURES, fk.FK_MODEL_OUTPUTS


def passes(ws, x, t, absolute=False):
    """y, dy and the flat gradient in fp64; absolute: with every product's
    magnitude in its place (masks from the plain pass)."""
    acts = [x]
    for i, (w, b) in enumerate(ws):
        z = acts[-1] @ w.T + b
        acts.append(z if i == 3 else np.maximum(z, 0.0))
    dy = 2.0 * (acts[-1] - t) / t.size
    if absolute:
        mags = [np.abs(x)]
        for i, (w, b) in enumerate(ws):
            mags.append(mags[-1] @ np.abs(w).T + np.abs(b))
        src, g, wabs = mags, 2.0 * (mags[-1] + np.abs(t)) / t.size, True
    else:
        src, g, wabs = acts, dy, False
    grads = []
    for i in reversed(range(4)):
        grads[:0] = [(g.T @ src[i]).ravel(), g.sum(0)]
        if i:
            g = (g @ (np.abs(ws[i][0]) if wabs else ws[i][0])) * (1 if wabs else acts[i] > 0)
    return acts[-1], dy, np.concatenate(grads), (mags[-1] if absolute else None)


@pytest.mark.parametrize("hidden,n", [(1, 1), (3, 15), (16, 16), (17, 17), (31, 255), (64, 257), (100, 33), (127, 65),
                                      (128, 512), (128, 1000), (129, 40)])
def test_forward_loss_and_gradients(hidden, n):
    g = np.random.default_rng(hidden * 1000 + n)
    dims = (F, hidden, hidden, hidden, O)
    ws = [((g.uniform(-1, 1, (b, a)) * np.sqrt(6.0 / a)).astype(np.float32),
           g.uniform(-0.1, 0.1, b).astype(np.float32)) for a, b in zip(dims[:-1], dims[1:])]
    x, t = g.standard_normal((n, F)).astype(np.float32), g.uniform(0, 0.8, (n, O)).astype(np.float32)
    w64 = [(w.astype(np.float64), b.astype(np.float64)) for w, b in ws]
    ry, rdy, rg, _ = passes(w64, x.astype(np.float64), t.astype(np.float64))
    _, _, mg, my = passes(w64, x.astype(np.float64), t.astype(np.float64), absolute=True)
    eps = 2.0 ** -23 * np.sqrt(n + 2 * hidden)

    m = fk.fk_model_create(hidden, 0)
    try:
        fk.fk_model_set_params(m, np.concatenate([v.ravel() for wb in ws for v in wb]))
        dx, dt = (torch.from_numpy(v).cuda() for v in (x, t))
        wsp = torch.full((fk.fk_mlp_workspace_floats(m, n),), float("nan"), device="cuda")
        y, dy = (torch.full((n, O), float("nan"), device="cuda") for _ in range(2))
        loss = torch.empty(1, device="cuda")
        grad = torch.full((fk.fk_model_param_count(m),), float("nan"), device="cuda")
        fk.fk_mlp_forward(m, dx, wsp, y)
        fk.fk_mlp_mse(y, dt, dy, loss)
        first = None
        for _ in range(2):  # a second backward pass from the same workspace gives the same bits
            fk.fk_mlp_backward(m, dx, wsp, dy, grad)
            torch.cuda.synchronize()
            if first is None:
                first = grad.clone()
            assert torch.equal(first, grad)
        assert np.all(np.abs(y.cpu().numpy() - ry) <= eps * my)
        assert abs(float(loss) - np.mean((ry - t) ** 2)) <= 1e-5 * np.mean((ry - t) ** 2) + 1e-12
        assert np.all(np.abs(grad.cpu().numpy() - rg) <= eps * mg)
        # the model's own passes (its workspace instead of the caller's)
        l2, g2 = fk.fk_model_loss_grad(m, x, t)
        assert np.array_equal(g2, grad.cpu().numpy()) and l2 == float(loss)
    finally:
        fk.fk_model_destroy(m)
