"""The sector form's host plan (sector_plan.cpp), compiled with g++ and read
directly: what the kernels index with it stays inside the angles and the
reduction slots of a layer, and the scale of the reverse sweep's vectors."""
import os
import subprocess

import numpy as np
import pytest

from oracle.model import greedy_matchings

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2408_00836_amd", "csrc")

# stdin: sites, bonds, U, then per bond i j t V, then eps and start spin per
# site; stdout: "name values..." lines
DRIVER = r"""
#include <cstdio>
#include <iostream>
#include "sector_plan.hpp"
using namespace hv;
int main()
{
    int ns, nb;
    double U;
    std::cin >> ns >> nb >> U;
    std::vector<int32_t> i(nb), j(nb), spin(ns);
    std::vector<double> t(nb), V(nb), eps(ns);
    for (int b = 0; b < nb; ++b)
        std::cin >> i[b] >> j[b] >> t[b] >> V[b];
    for (int s = 0; s < ns; ++s)
        std::cin >> eps[s] >> spin[s];
    Model m;
    std::string err = build_graph_model(ns, nb, i.data(), j.data(), t.data(), U, V.data(),
                                        eps.data(), nullptr, spin.data(), m);
    sec::SectorPlan P;
    if (err.empty())
        err = sec::plan_sector(m, P);
    if (!err.empty()) {
        std::printf("error %s\n", err.c_str());
        return 1;
    }
    std::printf("per %d\nphases %zu\nmix %.17g\n", m.params_per_layer(), P.sites.size(), P.mix);
    for (const sec::SecGate &g : P.gates)
        std::printf("gate %d %d %.17g\n", g.slot, g.last, g.t);
    return 0;
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, exe = d / "dump.cpp", d / "dump"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC, str(src),
                    os.path.join(CSRC, "sector_plan.cpp"), os.path.join(CSRC, "model.cpp"),
                    "-o", str(exe)], check=True)

    def run(ns, bonds, U=2.0, t=None, V=None, eps=None, spins=None):
        nb = len(bonds)
        t = np.ones(nb) if t is None else t
        V = np.zeros(nb) if V is None else V
        eps = np.zeros(ns) if eps is None else eps
        spins = [s & 1 for s in range(ns)] if spins is None else spins
        lines = [f"{ns} {nb} {U!r}"]
        lines += [f"{i} {j} {float(a)!r} {float(b)!r}" for (i, j), a, b in zip(bonds, t, V)]
        lines += [f"{float(e)!r} {s}" for e, s in zip(eps, spins)]
        out = subprocess.run([str(exe)], input="\n".join(lines), text=True, check=True,
                             capture_output=True).stdout
        res = {"gate": []}
        for line in out.splitlines():
            name, *v = line.split()
            if name == "gate":
                res["gate"].append((int(v[0]), int(v[1]), float(v[2])))
            else:
                res[name] = float(v[0])
        return res
    return run


def path(n):
    return [(k, k + 1) for k in range(n - 1)]


GRAPHS = {
    "1 site": (1, []),
    "4 sites, no bonds": (4, []),
    "16 sites, no bonds": (16, []),
    "2 sites": (2, path(2)),
    "5 path": (5, path(5)),
    "two far bonds": (9, [(0, 8), (3, 4)]),
    "star": (8, [(0, k) for k in range(1, 8)]),
    "complete": (6, [(a, b) for a in range(6) for b in range(a + 1, 6)]),
}


@pytest.mark.parametrize("key", list(GRAPHS))
def test_gates_stay_in_the_layers_parameters(plan, key):
    # a pass reads theta[layer * per + slot] for every position and, where a
    # slot's sum ends, adds to reduction slot `slot - 1` of per - 1 groups
    ns, bonds = GRAPHS[key]
    r = plan(ns, bonds)
    per, groups = int(r["per"]), len(set(greedy_matchings(bonds)))
    assert per == 1 + groups and len(r["gate"]) == 4 * r["phases"]
    for slot, last, t in r["gate"]:
        assert 0 <= slot < per
        if last or t != 0.0:
            assert slot >= 1
    # every phase's groups are each summed once, in runs of equal slots
    for p in range(int(r["phases"])):
        slots = [g[0] for g in r["gate"][4 * p:4 * p + 4]]
        ends = [g[1] for g in r["gate"][4 * p:4 * p + 4]]
        want = [1 if q == 0 or slots[q - 1] != slots[q] else 0 for q in range(4)]
        assert ends == (want if bonds else [0] * 4)
    # and every bond is applied once a layer
    assert sum(1 for g in r["gate"] if g[2] != 0.0) == len(bonds)


def mean_h2(ns, bonds, U, t, V, eps, spins):
    """|H psi|^2 of a state spread evenly over the sector with random phases:
    the mean over its basis states of D^2 plus the squares of H's hops."""
    up = [p for p in range(1 << ns) if bin(p).count("1") == spins.count(0)]
    dn = [p for p in range(1 << ns) if bin(p).count("1") == spins.count(1)]
    tot = 0.0
    for u in up:
        for d in dn:
            n = [(u >> i & 1) + (d >> i & 1) for i in range(ns)]
            D = U * bin(u & d).count("1") + sum(e * k for e, k in zip(eps, n))
            D += sum(v * n[i] * n[j] for (i, j), v in zip(bonds, V))
            tot += D * D + sum(a * a * ((p >> i ^ p >> j) & 1) for (i, j), a in zip(bonds, t)
                               for p in (u, d))
    return tot / (len(up) * len(dn))


def staggered(n, e):
    return [e if i % 2 == 0 else -e for i in range(n)]


MODELS = {
    "U": dict(U=4.0),
    "general": dict(U=4.0, V=[0.5, -0.3, 0.2, 0.4, -0.1], eps=[0.3, -0.2, 0.1, 0.4, -0.5, 0.2]),
    "staggered": dict(U=4.0, eps=staggered(6, 1e3)),
    "eps against U": dict(U=1e4, eps=[-2.5e3] * 6),
    "eps against U, weak hops": dict(U=8.0, t=[1e-3] * 5, eps=[-2.0] * 6),
    "V against U": dict(U=-20.0, V=[6.0] * 5),
    "off half filling": dict(U=3.0, eps=staggered(6, 50.0), spins=[0, 0, 1, 0, 0, 0]),
    "one spin": dict(U=3.0, eps=[1.0, 2.0, 3.0, 4.0, 5.0, 6.0], spins=[0] * 6),
}


@pytest.mark.parametrize("key", list(MODELS))
def test_mix_is_near_the_root_of_h(plan, key):
    # m = 2^k nearest to sqrt |H psi|: m^4 within a factor of four of |H psi|^2,
    # whatever cancels in the mean of D
    kw = dict(t=[1.0] * 5, V=[0.0] * 5, eps=[0.0] * 6, spins=[0, 1, 0, 1, 0, 1])
    kw.update(MODELS[key])
    m = plan(6, path(6), **kw)["mix"]
    h2 = mean_h2(6, path(6), **kw)
    assert m == 2.0 ** round(np.log2(m))
    assert 0.25 * (1 - 1e-9) <= m ** 4 / h2 <= 4.0 * (1 + 1e-9)
