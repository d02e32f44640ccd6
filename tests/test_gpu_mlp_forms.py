"""The network's forward pass on many rows of a narrow network, which takes one
product per layer, gives the bits of the fused pass of fewer rows: outputs and
hidden layers, on both sides of the rows at which the form changes."""
import pytest
import torch

import paper_2508_07071_amd as fk

pytestmark = pytest.mark.gpu
F, O = fk.FK_MODEL_FEATURES, fk.FK_MODEL_OUTPUTS


def forward(m, hidden, x):
    n = x.shape[0]
    ws = torch.full((fk.fk_mlp_workspace_floats(m, n),), float("nan"), device="cuda")
    y = torch.full((n, O), float("nan"), device="cuda")
    fk.fk_mlp_forward(m, x, ws, y)
    return torch.cat([y] + [ws[i * n * hidden:(i + 1) * n * hidden].view(n, hidden) for i in range(3)], 1)


@pytest.mark.parametrize("hidden,limit", [(1, 12288), (8, 12288), (60, 12288), (127, 12288), (16, 32768), (48, 98304)])
def test_forms_agree(hidden, limit):
    g = torch.Generator().manual_seed(hidden)
    m = fk.fk_model_create(hidden, 3)
    try:
        for n in (limit, limit + 37):
            x = torch.randn(n, F, generator=g).cuda()
            whole = forward(m, hidden, x)
            parts = torch.cat([forward(m, hidden, x[i:i + 4096].contiguous()) for i in range(0, n, 4096)])
            assert not whole.isnan().any() and torch.equal(whole, parts), n
    finally:
        fk.fk_model_destroy(m)
