"""The gradient of models whose diagonal's mean cancels (a staggered potential,
eps against U) through the sector form, which takes it from a difference of two
expectations: the vectors' scale keeps that difference as exact as the bracket
itself.  Bar: the gradient's 1e-8 of the other sector tests.  In complex128
against long double on the host the worst of the ten draws is off by 1e-9 at most
with the bracket summed directly and with this scale (either model), by 4e-8 with
one from the mean of D."""
import numpy as np
import pytest
import torch

from oracle import core as oc
from oracle.model import make_model
from paper_2408_00836_amd.model import Batch, Hubbard

pytestmark = pytest.mark.gpu

MODELS = {
    "staggered": dict(U=4.0, eps=[700.0, -700.0] * 3),
    "eps against U": dict(U=400.0, eps=[-100.0] * 6),
}


@pytest.mark.parametrize("key", list(MODELS))
def test_gradient_where_the_mean_of_d_cancels(gpu, key):
    kw, L, draws = MODELS[key], 2, 10
    rng = np.random.default_rng(5)
    models, thetas, refs = [], [], []
    for _ in range(draws):
        t = 1.0 + 0.1 * rng.standard_normal(5)
        m = Hubbard(1, 6, t=t, **kw)
        th = rng.uniform(-0.2, 0.2, m.n_params(L))
        models.append(m)
        thetas.append(th)
        refs.append(oc.energy_grad(make_model(1, 6, t=t, **kw), th, L))
    worst = 0.0
    for m, th, (E_ref, g_ref) in zip(models, thetas, refs):
        for f in (m.energy_grad, m.sector_energy_grad):
            E, g = f(torch.tensor(th, device=gpu))
            assert abs(E.item() - E_ref) <= 1e-12 * max(1.0, abs(E_ref), 4200.0)
            worst = max(worst, float(np.max(np.abs(g.cpu().numpy() - g_ref))))
    b = Batch(models, [L] * draws)
    _, g = b.energy_grad(torch.tensor(np.concatenate(thetas), device=gpu))
    worst = max(worst, float(np.max(np.abs(g.cpu().numpy() -
                                           np.concatenate([r[1] for r in refs])))))
    print(f"[scale] {key}: worst gradient error {worst:.2e}", flush=True)
    assert worst <= 1e-8
