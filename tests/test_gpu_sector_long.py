"""Sector rows of 16 sites off half filling against the oracle's sector: 6 and
7 spin-up electrons (rows of 8008 and 11440 amplitudes: other slots, orbit
lists and thread chunks than half filling's 12870), bonds in both
orders with and without a Jordan-Wigner string, an odd cycle, and the general
diagonal.  Bars as in test_gpu_sector: |dE| <= 1e-12 max(1, |E|), gradient
1e-8, amplitudes of H psi 1e-10."""
import numpy as np
import pytest
import torch

from oracle import sector as osec
from oracle.model import make_graph_model
from paper_2408_00836_amd.model import Hubbard

pytestmark = pytest.mark.gpu

BONDS = [(0, 1), (2, 1), (3, 2), (3, 4), (5, 6), (6, 8), (9, 7), (10, 11), (12, 11), (13, 14),
         (15, 14), (0, 15), (12, 4), (8, 5)]


@pytest.mark.parametrize("n_up,general", [(6, True), (7, False)])
def test_long_rows_off_half_filling(gpu, n_up, general):
    rng = np.random.default_rng(n_up)
    bonds = np.asarray(BONDS, dtype=np.int32)
    kw = dict(t=1.0 + 0.2 * rng.standard_normal(len(BONDS)), U=3.0)
    if general:
        kw.update(V=rng.uniform(-0.4, 0.4, len(BONDS)), eps=rng.uniform(-0.3, 0.3, 16))
    spins = [0] * n_up + [1] * (16 - n_up)
    rng.shuffle(spins)
    m = Hubbard.graph(16, bonds, site_spin=spins, **kw)
    om = make_graph_model(16, bonds, site_spin=spins, **kw)
    th = rng.uniform(-0.5, 0.5, om.params_per_layer)
    print(f"[sector] 16 sites, {n_up} up", flush=True)
    t = torch.tensor(th, device=gpu)
    E, g = m.sector_energy_grad(t)
    E_ref, g_ref = osec.energy_grad(om, th, 1)
    assert abs(E.item() - E_ref) <= 1e-12 * max(1.0, abs(E_ref))
    assert np.max(np.abs(g.cpu().numpy() - g_ref)) <= 1e-8
    psi = m.sector_state(t)
    got = m.sector_apply_h(psi).cpu().numpy().ravel()
    ref = osec.ham_apply(om, np.ascontiguousarray(psi.cpu().numpy().ravel()))
    assert np.max(np.abs(got - ref)) <= 1e-10
