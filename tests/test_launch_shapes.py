"""The launch shapes of calls without a set or tuned shape, read from the kernel
names that the profiler sees.
"""
import re

import pytest

from synth import config_mechanism, draw_states, make_mechanism

pytestmark = pytest.mark.gpu


def launched_shapes(torch, call):
    """(tile states, threads) of the tile kernels that `call` launches."""
    from torch.profiler import ProfilerActivity, profile
    call()
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CPU, ProfilerActivity.CUDA]) as prof:
        call()
        torch.cuda.synchronize()
    names = {e.name for e in prof.events()}
    found = [m for m in (re.search(r"tile(?:_multi)?_kernel(?:<|ILi)(\d+)(?:, |ELi)(\d+)", k) for k in names) if m]
    assert found, sorted(names)
    return {(int(m[1]), int(m[2])) for m in found}


def mechanism(species):
    if species == 200:
        mix = {"elementary": 840, "thirdbody": 120, "falloff_lindemann": 60, "falloff_sri": 36, "falloff_troe": 144}
        return make_mechanism(1805, 200, 1200, ["C", "H", "O", "N", "Ar"], dict(C=5, H=12, O=3, N=1), mix)
    return config_mechanism({13: 0, 53: 1, 111: 2, 360: 3}[species])


def calls_of(torch, M, n):
    """The three kernel families' calls on n states, by their number."""
    N = M.n_species
    phi, p = (torch.from_numpy(a).cuda() for a in draw_states(3, N, n))
    conc = torch.cat([phi[:1], torch.full((N, n), 1e-3, dtype=torch.float64, device="cuda")])
    out = torch.empty((max(N * N, 3 * N + 1 + len(M.conc_pattern()[1])), n), dtype=torch.float64, device="cuda")
    return {0: lambda: M.eval_rates(phi, p, rop_f=False, rop_r=False, pres_mod=False),
            1: lambda: M.eval_jacobian(phi, p, out=out[:N * N]),
            2: lambda: M.eval_jacobian_conc(conc, out=out[:3 * N + 1 + len(M.conc_pattern()[1])])}, phi, p, out


@pytest.mark.parametrize("species,n,which,good", [
    (13, 3000, 1, {(16, 512), (8, 256), (16, 1024), (4, 256)}), (13, 4099, 2, {(8, 256)}), (13, 100_000, 1, {(64, 1024)}),
    (53, 3000, 1, {(4, 256)}), (53, 30_000, 1, {(4, 256), (8, 512)}),
    (111, 9000, 1, {(4, 256)}), (111, 20_001, 1, {(4, 256)}), (111, 9000, 2, {(4, 256)}), (111, 20_001, 2, {(4, 256)}),
    (200, 4096, 1, {(4, 1024)}), (200, 7000, 2, {(4, 1024)}), (360, 2051, 1, {(2, 1024)})])
def test_chosen_shape(species, n, which, good):
    """The rule takes a shape that measured within 7 % of the best one."""
    import torch
    from paper_1605_03262_amd import Mechanism
    M = Mechanism(text=mechanism(species).to_text())
    shapes = launched_shapes(torch, calls_of(torch, M, n)[0][which])
    assert len(shapes) == 1 and shapes <= good


@pytest.mark.parametrize("species,n", [(13, 100_000), (53, 30_000), (111, 20_001)])
def test_reported_shape(species, n):
    """get_variant names the shape that a large batch runs in (rates and
    concentration form), the shape of work lists (Jacobian), and a set shape."""
    import torch
    from paper_1605_03262_amd import Mechanism, _lib
    M = Mechanism(text=mechanism(species).to_text())
    calls, phi, p, out = calls_of(torch, M, n)
    for which in (0, 2):
        assert launched_shapes(torch, calls[which]) == {M.get_variant(which)[:2]}, which
    items = [(M.handle, n, n, phi.data_ptr(), p.data_ptr(), out.data_ptr())]
    work_list = lambda: _lib.pyjac_eval_jacobian_multi(items, torch.cuda.current_stream().cuda_stream)  # noqa: E731
    assert launched_shapes(torch, work_list) == {M.get_variant(1)[:2]}
    for which, call in calls.items():
        M.set_variant(which, 4, 512)
        assert M.get_variant(which)[:2] == (4, 512) and launched_shapes(torch, call) == {(4, 512)}, which
