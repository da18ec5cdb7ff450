"""Fock builds on both sides of the sizes where the pair order, the items and the sharing of a
chunk between waves change, against the oracle (FP64 builds agree with it to a few 1e-15 at
these sizes: 1e-12; FP32 integrals to a few 1e-8: 1e-6)."""
import numpy as np
import pytest

import oracle
from he_inputs import jittered_lattice
from gpu_util import announce, assert_close, rel

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "mixed": 1e-6}


def _cut(n, spacing, tau):
    m = int(np.ceil(n ** (1 / 3) - 1e-9))
    s = jittered_lattice((m, m, m), seed=500 + n, tau=tau, spacing=spacing)
    return np.ascontiguousarray(s.xyz[:n]), np.ascontiguousarray(s.dens[:n, :n])


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n,g,atoms,spacing,tau", [
    (1, 6, False, 2.0, 0.0), (10, 3, False, 2.0, 1e-12), (11, 3, False, 2.0, 1e-12), (10, 4, True, 2.0, 0.0),
    (27, 6, False, 3.0, 1e-10), (28, 6, False, 3.0, 1e-10), (27, 5, True, 3.0, 1e-10), (70, 3, False, 4.0, 1e-8),
    (71, 3, False, 4.0, 1e-8), (109, 2, True, 4.0, 1e-8), (110, 2, True, 4.0, 1e-8), (127, 5, False, 5.0, 1e-6),
    (128, 5, False, 5.0, 1e-6), (180, 3, False, 5.0, 1e-8), (181, 3, False, 5.0, 1e-8), (257, 1, False, 5.0, 1e-8)])
def test_either_side_of_a_rule(n, g, atoms, spacing, tau, precision):
    import torch
    import paper_2509_21039_amd as hfk
    dev = torch.device("cuda:0")
    xyz, dens = _cut(n, spacing, tau)
    e, c = 0.25 * 3.0 ** np.arange(g - 1, -1, -1.0), np.linspace(0.2, 0.6, g)
    if atoms:
        e, c = e * np.random.default_rng(n).uniform(0.6, 1.4, n)[:, None], np.tile(c, (n, 1))
    announce("small systems n=%d g=%d atoms=%d %s" % (n, g, atoms, precision))
    build, ref = (hfk.fock_atoms, oracle.fock_atoms) if atoms else (hfk.fock, oracle.fock)
    ws = hfk.new_workspace((hfk.workspace_bytes_atoms if atoms else hfk.workspace_bytes)(n, g, precision), dev)
    X, D = torch.tensor(xyz, device=dev), torch.tensor(dens, device=dev)
    Gr, Er, kept = ref(xyz, dens, e, c, tau)
    for _ in range(2):   # the second call finds the first one's workspace
        G, E2 = build(X, D, e, c, tau, precision, workspace=ws)
        assert_close(G.cpu().numpy(), Gr, TOL[precision])
        assert rel(float(E2.item()), Er) < TOL[precision]
        assert hfk.read_stats(ws)["quartets"] == kept


@pytest.mark.parametrize("n,g,atoms,precision,spacing,tau", [
    (24, 3, False, "fp64", 2.0, 1e-10), (25, 3, False, "mixed", 2.0, 1e-10), (48, 6, False, "fp64", 4.0, 1e-8),
    (49, 2, True, "mixed", 3.0, 1e-10), (109, 3, False, "mixed", 5.0, 1e-8), (110, 3, False, "mixed", 5.0, 1e-8),
    (128, 3, False, "fp64", 5.0, 1e-8), (129, 3, True, "fp64", 5.0, 1e-8)])
def test_gradient_either_side_of_a_rule(n, g, atoms, precision, spacing, tau):
    # tolerances of the gradient tests
    import torch
    import paper_2509_21039_amd as hfk
    dev = torch.device("cuda:0")
    xyz, dens = _cut(n, spacing, tau)
    e, c = 0.25 * 3.0 ** np.arange(g - 1, -1, -1.0), np.linspace(0.2, 0.6, g)
    if atoms:
        e, c = e * np.random.default_rng(n).uniform(0.6, 1.4, n)[:, None], np.tile(c, (n, 1))
    announce("small systems gradient n=%d g=%d atoms=%d %s" % (n, g, atoms, precision))
    X, D = torch.tensor(xyz, device=dev), torch.tensor(dens, device=dev)
    G = torch.randn((n, n), dtype=torch.float64, device=dev, generator=torch.Generator(dev).manual_seed(n))
    scale = torch.full((1,), 0.7, dtype=torch.float64, device=dev)
    dx, dd, E2 = hfk.fock_grad(X, D, e, c, tau, precision, g_e2=scale, fock_in=G)
    gr, Er, _ = (oracle.grad_atoms if atoms else oracle.grad)(xyz, dens, e, c, tau)
    assert_close(dx.cpu().numpy(), 0.7 * gr, 1e-10 if precision == "fp64" else 1e-6)
    assert rel(float(E2.item()), Er) < TOL[precision]
    assert torch.equal(dd, 0.7 * G)


@pytest.mark.parametrize("n,precision", [(1303, "fp64"), (1092, "mixed")])
def test_wide_workgroups(n, precision):
    # the first sizes with eight waves per workgroup (rows of F in LDS); thinly spread atoms
    import torch
    import paper_2509_21039_amd as hfk
    dev = torch.device("cuda:0")
    xyz, dens = _cut(n, 9.0, 1e-7)
    e, c = np.array([6.36242139, 1.15892300, 0.31364979]), np.array([0.15432897, 0.53532814, 0.44463454])
    announce("wide workgroups n=%d %s" % (n, precision))
    G, E2 = hfk.fock(torch.tensor(xyz, device=dev), torch.tensor(dens, device=dev), e, c, 1e-7, precision)
    Gr, Er, _ = oracle.fock(xyz, dens, e, c, 1e-7)
    assert_close(G.cpu().numpy(), Gr, TOL[precision])
    assert rel(float(E2.item()), Er) < TOL[precision]
