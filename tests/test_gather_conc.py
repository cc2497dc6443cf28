"""The reaction phase over reactions with three to six net species (an
equilibrium term of more than four entries reads its list in two parts), and
the concentration-form kernel's own gather over list lengths around its blocks
of eight entries.  Rates, Jacobian and concentration form against the oracle
(the bars of the other parity tests), bitwise equal at every launch shape.
"""
import numpy as np
import pytest

from synth import draw_states
from test_gather_lists import SHAPES, hub_mechanism, ref_gross
from test_gpu_conc import densify, gpu_conc
from test_gpu_parity import JAC_TOL, RATE_TOL, check_jac, enorm_per_state

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    return t


def net_mechanism(n_species, n_reactions):
    """Species with one hydrogen atom (the first two thirds) or two; reactions
    with 6, 5, 4 and 3 net species in turn: 3 = 3, 3 = 2, 2 = 2 and 2 = 1
    molecules.  S0 takes part in every one."""
    ones = 2 * n_species // 3
    h = [1 if k < ones else 2 for k in range(n_species)]
    out = ["pyjac-mech 1", "elements 1", "  H 1.008", f"species {n_species}"]
    for k in range(n_species):
        out += [f"  S{k} {1.008 * h[k]!r} 1000.0 1 H {h[k]}"]
        out += [f"    {2.5 + 0.01 * k} 1e-4 0.0 0.0 0.0 {100.0 - 7 * k} {1.0 + 0.1 * k}"] * 2
    out += [f"reactions {n_reactions}"]
    for i in range(n_reactions):
        a = [1 + (i + q) % (ones - 1) for q in range(5)]
        two = ones + i % (n_species - ones)
        reac, prod = [([0, a[0], a[1]], [a[2], a[3], a[4]]), ([0, a[0], a[1]], [a[2], two]),
                      ([0, a[0]], [a[1], a[2]]), ([0, a[0]], [two])][i % 4]
        side = lambda s: f"{len(s)} " + " ".join(f"S{k} 1" for k in s)  # noqa: E731
        out += ["reaction elementary kc", "reactants " + side(reac), "products " + side(prod),
                f"arrhenius {1.0e3 * (1 + i % 7)} {0.1 * (i % 5)} {50.0 * (i % 11)}"]
    return "\n".join(out + ["end"]) + "\n"


def conc_of(text, phi, p, W):
    Y = np.vstack([phi[1:], 1 - phi[1:].sum(axis=0)])
    rho = p / (8314.462618 * phi[0] * (Y / W[:, None]).sum(axis=0))
    return np.vstack([phi[:1], rho * Y / W[:, None]])


def every_shape(M, which, call):
    first, tried = None, 0
    from paper_1605_03262_amd import PyjacError
    for ts, nt in SHAPES:
        try:
            M.set_variant(which, ts, nt)
        except PyjacError:
            continue
        tried += 1
        out = call()
        first = out if first is None else first
        assert np.array_equal(out, first), (ts, nt)
    assert tried >= 4
    M.set_variant(which, 0, 0)
    return first


def check_conc(torch, ref, M, c, N):
    out, (colptr, rowidx) = every_shape(M, 2, lambda: gpu_conc(torch, M, c)), M.conc_pattern()
    assert np.array_equal(out, gpu_conc(torch, M, c))
    e = enorm_per_state(densify(out, colptr, rowidx, N), ref.eval_jacobian_conc(c))
    assert e.max() <= JAC_TOL, e.max()


@pytest.mark.parametrize("n_species,n_reactions", [(9, 1), (9, 4), (12, 9), (17, 64), (33, 130)])
def test_net_species(torch, oracle_built, n_species, n_reactions):
    from oracle import RefMech
    from paper_1605_03262_amd import Mechanism
    text = net_mechanism(n_species, n_reactions)
    ref, M = RefMech(text=text), Mechanism(text=text)
    phi, p = draw_states(n_species, n_species, 9)
    d_phi, d_p = torch.from_numpy(phi).cuda(), torch.from_numpy(p).cuda()
    rr = ref.eval_rates(phi, p)
    w = every_shape(M, 0, lambda: M.eval_rates(d_phi, d_p)["wdot"].cpu().numpy())
    assert np.max(np.abs(w - rr["wdot"]) / ref_gross(rr, n_species)) <= RATE_TOL
    check_jac(every_shape(M, 1, lambda: M.eval_jacobian(d_phi, d_p).cpu().numpy()), ref.eval_jacobian(phi, p))
    ones = 2 * n_species // 3
    W = np.array([1.008 if k < ones else 2.016 for k in range(n_species)])
    check_conc(torch, ref, M, conc_of(text, phi, p, W), n_species)


@pytest.mark.parametrize("n_species,n_reactions", [(4, 1), (4, 7), (5, 8), (5, 9), (6, 16), (6, 17), (17, 129),
                                                   (33, 511), (33, 513)])
def test_gather_lists_conc(torch, oracle_built, n_species, n_reactions):
    from oracle import RefMech
    from paper_1605_03262_amd import Mechanism
    text = hub_mechanism(n_species, n_reactions)
    phi, p = draw_states(n_species, n_species, 9)
    check_conc(torch, RefMech(text=text), Mechanism(text=text), conc_of(text, phi, p, np.full(n_species, 2.016)), n_species)
