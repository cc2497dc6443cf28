"""Species gathers of the reaction phase at list lengths around their blocks of
eight entries: mechanisms of isomers in which species 0 takes part in every
reaction (a list of up to 512 entries in one reaction chunk), species 1 in
none, and the others in a few.  Rates and Jacobian against the oracle (1e-12
and E_norm 1e-10, the bars of the other parity tests), bitwise equal at every
launch shape.
"""
import numpy as np
import pytest

from synth import draw_states

SHAPES = [(16, 1024), (16, 512), (32, 1024), (64, 1024), (8, 512), (8, 1024), (4, 512), (4, 1024), (2, 512),
          (2, 1024), (8, 256), (4, 256)]


def hub_mechanism(n_species, n_reactions):
    out = ["pyjac-mech 1", "elements 1", "  H 1.008", f"species {n_species}"]
    for k in range(n_species):
        out += [f"  S{k} 2.016 1000.0 1 H 2"] + [f"    {2.5 + 0.01 * k} 1e-4 0.0 0.0 0.0 {100.0 - 7 * k} {1.0 + 0.1 * k}"] * 2
    out += [f"reactions {n_reactions}"]
    for i in range(n_reactions):
        k = 2 + i % (n_species - 2)
        out += ["reaction elementary kc", "reactants 1 S0 1", f"products 1 S{k} 1",
                f"arrhenius {1.0e3 * (1 + i % 7)} {0.1 * (i % 5)} {50.0 * (i % 11)}"]
    return "\n".join(out + ["end"]) + "\n"


@pytest.mark.gpu
@pytest.mark.parametrize("n_species,n_reactions", [(4, 1), (4, 7), (5, 8), (5, 9), (6, 16), (6, 17), (17, 129),
                                                   (33, 511), (33, 513)])
def test_gather_lists(oracle_built, n_species, n_reactions):
    import torch
    from oracle import RefMech
    from paper_1605_03262_amd import Mechanism, PyjacError
    text = hub_mechanism(n_species, n_reactions)
    ref, M = RefMech(text=text), Mechanism(text=text)
    n = 9
    phi, p = draw_states(n_species, n_species, n)
    Jr, rr = ref.eval_jacobian(phi, p), ref.eval_rates(phi, p)
    gross = ref_gross(rr, n_species)
    d_phi, d_p = torch.from_numpy(phi).cuda(), torch.from_numpy(p).cuda()
    first = None
    for ts, nt in SHAPES:
        try:
            M.set_variant(1, ts, nt)
            M.set_variant(0, ts, nt)
        except PyjacError:
            continue
        J = M.eval_jacobian(d_phi, d_p).cpu().numpy()
        r = M.eval_rates(d_phi, d_p)["wdot"].cpu().numpy()
        if first is None:
            first = (J, r)
            e = np.linalg.norm(J - Jr, axis=0) / np.linalg.norm(Jr, axis=0)
            assert e.max() <= 1e-10, (ts, nt, e.max())
            assert np.max(np.abs(r - rr["wdot"]) / gross) <= 1e-12
        assert np.array_equal(J, first[0]) and np.array_equal(r, first[1]), (ts, nt)
    assert first is not None


def ref_gross(r, n_species):
    """Sum of the gross rates over the reactions (every reaction involves
    species 0): the scale no production rate exceeds."""
    return (np.abs(r["rop_f"]) + np.abs(r["rop_r"])).sum(axis=0)[None, :]
