"""Builds and gradients on both sides of the sizes where the chunks per wave of an item, and the waves
that share a chunk, change with the primitives, the precision and the basis, against the oracle
(tolerances of the small-system and gradient tests)."""
import numpy as np
import pytest

import oracle
from he_inputs import jittered_lattice
from gpu_util import announce, assert_close, rel

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "mixed": 1e-6}


def _system(n, g, atoms, tau):
    m = int(np.ceil(n ** (1 / 3) - 1e-9))
    s = jittered_lattice((m, m, m), seed=300 + n, tau=tau, spacing=4.0 if n < 100 else 5.0)
    e, c = 0.25 * 3.0 ** np.arange(g - 1, -1, -1.0), np.linspace(0.2, 0.6, g)
    if atoms:
        e, c = e * np.random.default_rng(n).uniform(0.6, 1.4, n)[:, None], np.tile(c, (n, 1))
    return np.ascontiguousarray(s.xyz[:n]), np.ascontiguousarray(s.dens[:n, :n]), e, c


@pytest.mark.parametrize("n,g,atoms,precision,tau", [
    (19, 1, False, "fp64", 1e-10), (20, 1, True, "mixed", 1e-10), (25, 2, True, "fp64", 1e-10),
    (26, 2, False, "mixed", 1e-10), (15, 3, False, "fp64", 1e-12), (16, 3, True, "fp64", 1e-12),
    (64, 3, True, "mixed", 1e-8), (65, 3, False, "mixed", 1e-8), (76, 3, False, "fp64", 1e-8),
    (77, 3, False, "fp64", 1e-8), (128, 3, True, "fp64", 1e-6), (129, 3, True, "fp64", 1e-6),
    (27, 4, False, "fp64", 1e-10), (28, 4, True, "fp64", 1e-10), (170, 4, False, "mixed", 1e-6),
    (171, 4, False, "fp64", 1e-6), (170, 6, False, "fp64", 1e-5)])
def test_build_either_side_of_a_line(n, g, atoms, precision, tau):
    import torch
    import paper_2509_21039_amd as hfk
    dev = torch.device("cuda:0")
    xyz, dens, e, c = _system(n, g, atoms, tau)
    announce("item lines n=%d g=%d atoms=%d %s" % (n, g, atoms, precision))
    build, ref = (hfk.fock_atoms, oracle.fock_atoms) if atoms else (hfk.fock, oracle.fock)
    ws = hfk.new_workspace((hfk.workspace_bytes_atoms if atoms else hfk.workspace_bytes)(n, g, precision), dev)
    G, E2 = build(torch.tensor(xyz, device=dev), torch.tensor(dens, device=dev), e, c, tau, precision, workspace=ws)
    Gr, Er, kept = ref(xyz, dens, e, c, tau)
    assert_close(G.cpu().numpy(), Gr, TOL[precision])
    assert rel(float(E2.item()), Er) < TOL[precision]
    assert hfk.read_stats(ws)["quartets"] == kept


@pytest.mark.parametrize("n,g,atoms,precision,tau", [
    (40, 1, False, "fp64", 1e-10), (41, 1, True, "mixed", 1e-10), (100, 2, False, "fp64", 1e-8),
    (101, 2, True, "fp64", 1e-8), (72, 2, True, "mixed", 1e-8), (73, 2, False, "mixed", 1e-8),
    (150, 4, False, "mixed", 1e-5), (151, 4, False, "fp64", 1e-5)])
def test_gradient_either_side_of_a_line(n, g, atoms, precision, tau):
    import torch
    import paper_2509_21039_amd as hfk
    dev = torch.device("cuda:0")
    xyz, dens, e, c = _system(n, g, atoms, tau)
    announce("item lines gradient n=%d g=%d atoms=%d %s" % (n, g, atoms, precision))
    dx, _, E2 = hfk.fock_grad(torch.tensor(xyz, device=dev), torch.tensor(dens, device=dev), e, c, tau, precision,
                              want_dens=False)
    gr, Er, _ = (oracle.grad_atoms if atoms else oracle.grad)(xyz, dens, e, c, tau)
    assert_close(dx.cpu().numpy(), gr, 1e-10 if precision == "fp64" else 1e-6)
    assert rel(float(E2.item()), Er) < TOL[precision]
