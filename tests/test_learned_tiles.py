"""The loss gradient of the hopping network at the edges of its 16-bond tiles and of
the two tiles a wavefront takes together (tbk_mlp_loss_grad).

A batch of nb bonds equals the batch of 2 nb bonds whose second half has weight
zero, up to the factor 1/2 of the mean: 1 / (2 nb) is exactly half of 1 / nb in
float and bfloat16 rounding does not depend on a factor of two, so every term is
halved exactly.  Only the order of float sums within a wavefront (two tiles of
16 terms each, 2^-24 per addition) may differ: held to 1e-5 of the largest
gradient component, the loss (double sums) to 1e-13.
"""
import numpy as np
import pytest
import torch

from paper_2509_06525_amd import synth, tbkpm
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb", [1, 15, 16, 17, 31, 33, 64, 129, 1000, 2047, 2048, 2049])
def test_gradient_at_tile_edges(nb):
    rng = np.random.default_rng(nb)
    n = 2 * nb
    x = torch.from_numpy(rng.normal(0, 1, (n, 16)).astype(np.float32)).to(G.DEV)
    X = x.to(torch.bfloat16).view(torch.int16).contiguous()
    target = G.to_dev(rng.normal(0, 0.1, n).astype(np.float32))
    weight = G.to_dev(rng.uniform(0.5, 1.5, n).astype(np.float32))
    masked = weight.clone()
    masked[nb:] = 0
    P = torch.from_numpy(synth.init_mlp_params(7, out_scale=1.0)).to(G.DEV)
    loss1, g1 = tbkpm.mlp_loss_grad(X[:nb].contiguous(), target[:nb].contiguous(), P, weight=weight[:nb].contiguous())
    loss2, g2 = tbkpm.mlp_loss_grad(X, target, P, weight=masked)
    assert abs(loss1 - 2 * loss2) <= 1e-13 * abs(loss1)
    assert (g1 - 2 * g2).abs().max().item() <= 1e-5 * g1.abs().max().item()
    y = tbkpm.mlp_forward(X, P)
    want = ((y[:nb] - target[:nb]).double() ** 2 * weight[:nb].double()).mean().item()
    assert abs(loss1 - want) <= 1e-6 * want
