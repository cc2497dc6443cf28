"""The launch shape chosen by a call's batch size: the same bits as a set shape
on both sides of every batch size at which the rule changes tiles (2, 4, 8 or
16 states per tile while that gives every CU at most one, 256 CUs), and on
small chunks of the finite-difference Jacobian."""
import numpy as np
import pytest

from synth import config_mechanism, config_states

SET = {0: (16, 512), 1: (8, 512), 2: (8, 512)}


@pytest.mark.gpu
@pytest.mark.parametrize("cfg", [0, 1])
@pytest.mark.parametrize("n", [1, 3, 512, 513, 1024, 1025, 2048, 2049, 4096, 4097])
def test_shape_rule(cfg, n):
    import torch
    from paper_1605_03262_amd import Mechanism
    text = config_mechanism(cfg).to_text()
    phi, p = config_states(cfg, n)
    d_phi, d_p = torch.from_numpy(phi).cuda(), torch.from_numpy(p).cuda()
    conc = torch.cat([d_phi[:1], torch.abs(torch.cat([d_phi[1:], 1.0 - d_phi[1:].sum(0, keepdim=True)])) * 0.01])
    auto, fixed = Mechanism(text=text), Mechanism(text=text)
    for which, (ts, nt) in SET.items():
        fixed.set_variant(which, ts, nt)
    a, b = auto.eval_rates(d_phi, d_p), fixed.eval_rates(d_phi, d_p)
    for k in a:
        assert torch.equal(a[k], b[k]), k
    assert torch.equal(auto.eval_jacobian(d_phi, d_p), fixed.eval_jacobian(d_phi, d_p))
    assert torch.equal(auto.eval_jacobian_conc(conc), fixed.eval_jacobian_conc(conc))
    if n <= 64:
        assert torch.equal(auto.eval_jacobian_fd(d_phi, d_p, chunk_states=2),
                           fixed.eval_jacobian_fd(d_phi, d_p, chunk_states=64))
    fixed.set_variant(1, 0, 0)                            # back to the automatic choice
    assert torch.equal(auto.eval_jacobian(d_phi, d_p), fixed.eval_jacobian(d_phi, d_p))
    assert np.isfinite(a["wdot"].cpu().numpy()).all()
