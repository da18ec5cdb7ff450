"""The primitive-term screen of the quartet kernels: builds over geometries and contractions
where most primitive quartets are negligible, against the oracle, which sums every one.

A left-out term is below 1e-10 min(tau, 1e-10) <= 1e-20, and a matrix element sums at most
n^2 quartets of g^4 terms (40^2 * 1296 = 2e6): 2e-14 at most against elements of order one.
FP64 builds of this size agree with the oracle to a few 1e-15, so 1e-12 holds both with room."""
import numpy as np
import pytest

import oracle
from he_inputs import jittered_lattice
from gpu_util import announce, assert_close, rel

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "mixed": 1e-6}


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch, torch.device("cuda:0")


def _basis(g, order):
    """Even-tempered exponents from tight to diffuse, one negative coefficient from g = 3 on."""
    e = 0.2 * 3.5 ** np.arange(g - 1, -1, -1.0)
    c = np.linspace(0.2, 0.6, g)
    if g > 2:
        c[1] = -0.1
    p = {"tight_first": np.arange(g), "diffuse_first": np.arange(g)[::-1], "shuffled": np.random.default_rng(g).permutation(g)}[order]
    return e[p], c[p]


def _system(g, order, tau, spacing, atoms):
    s = jittered_lattice((3, 3, 4), seed=40 + g, tau=tau, spacing=spacing)
    e, c = _basis(g, order)
    if atoms:
        scale = np.random.default_rng(g).uniform(0.6, 1.4, s.natoms)
        e, c = e * scale[:, None], np.tile(c, (s.natoms, 1))
    return s, e, c


@pytest.mark.parametrize("atoms", [False, True])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("g,order,tau,spacing", [
    (1, "tight_first", 1e-10, 3.0), (2, "diffuse_first", 1e-10, 3.0), (3, "tight_first", 1e-12, 4.0),
    (3, "shuffled", 1e-8, 3.0), (4, "tight_first", 1e-10, 3.0), (5, "diffuse_first", 1e-10, 3.0),
    (6, "tight_first", 1e-12, 3.0), (6, "shuffled", 0.0, 4.0)])
def test_forward_vs_oracle(torch_dev, atoms, precision, g, order, tau, spacing):
    import paper_2509_21039_amd as hfk
    torch, dev = torch_dev
    s, e, c = _system(g, order, tau, spacing, atoms)
    announce("term screen g=%d %s tau=%g spacing=%g atoms=%d %s" % (g, order, tau, spacing, atoms, precision))
    build = hfk.fock_atoms if atoms else hfk.fock
    G, E2 = build(torch.tensor(s.xyz, device=dev), torch.tensor(s.dens, device=dev), e, c, tau, precision)
    Gr, Er, _ = (oracle.fock_atoms if atoms else oracle.fock)(s.xyz, s.dens, e, c, tau)
    assert_close(G.cpu().numpy(), Gr, TOL[precision])
    assert rel(float(E2.item()), Er) < TOL[precision]


@pytest.mark.parametrize("atoms", [False, True])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("g,order,tau,spacing", [
    (1, "tight_first", 1e-10, 3.0), (2, "diffuse_first", 1e-10, 3.0), (3, "tight_first", 1e-12, 4.0),
    (3, "shuffled", 1e-8, 3.0), (4, "tight_first", 1e-10, 3.0), (5, "diffuse_first", 1e-8, 4.0)])
def test_gradient_vs_oracle(torch_dev, atoms, precision, g, order, tau, spacing):
    # the derivative bounds carry max(1, 2 mu R, sqrt p) per pair, so the same count holds
    import paper_2509_21039_amd as hfk
    torch, dev = torch_dev
    s, e, c = _system(g, order, tau, spacing, atoms)
    announce("term screen gradient g=%d %s tau=%g spacing=%g atoms=%d %s" % (g, order, tau, spacing, atoms, precision))
    dx, _, E2 = hfk.fock_grad(torch.tensor(s.xyz, device=dev), torch.tensor(s.dens, device=dev), e, c, tau, precision,
                              want_dens=False)
    gr, Er, _ = (oracle.grad_atoms if atoms else oracle.grad)(s.xyz, s.dens, e, c, tau)
    # the FP64 gradient's rows are of degree 7 with a derivative near 3e-12 (tolerance of the gradient tests)
    assert_close(dx.cpu().numpy(), gr, 1e-10 if precision == "fp64" else TOL["mixed"])
    assert rel(float(E2.item()), Er) < TOL[precision]


@pytest.mark.parametrize("grad", [False, True])
@pytest.mark.parametrize("atoms", [False, True])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("g,order,tau,spacing", [
    (1, "tight_first", 1e-10, 3.0), (2, "diffuse_first", 1e-10, 3.0), (3, "tight_first", 1e-12, 4.0),
    (3, "shuffled", 1e-8, 3.0), (4, "tight_first", 0.0, 4.0), (6, "tight_first", 1e-10, 4.0)])
def test_batched_vs_oracle(torch_dev, grad, atoms, precision, g, order, tau, spacing):
    # molecules whose pairs start at odd places, so that a unit's kets lie in two blocks of 64
    import paper_2509_21039_amd as hfk
    torch, dev = torch_dev
    shapes = [(1, 1, 1), (2, 2, 3), (1, 1, 2), (2, 3, 3), (3, 3, 3), (1, 2, 2)]
    mols = [jittered_lattice(sh, seed=60 + k, tau=tau, spacing=spacing) for k, sh in enumerate(shapes)]
    e, c = _basis(g, order)
    off = np.cumsum([0] + [m.natoms for m in mols])
    eb, cb = (np.tile(e, (off[-1], 1)), np.tile(c, (off[-1], 1))) if atoms else (e, c)
    if atoms:
        eb = eb * np.random.default_rng(g).uniform(0.6, 1.4, off[-1])[:, None]
    announce("term screen batched g=%d %s tau=%g spacing=%g atoms=%d %s grad=%d" % (g, order, tau, spacing, atoms, precision, grad))
    G, E2, dx = hfk.fock_batched(off, torch.tensor(np.concatenate([m.xyz for m in mols]), device=dev),
                                 torch.tensor(np.concatenate([m.dens.ravel() for m in mols]), device=dev), eb, cb, tau,
                                 precision, with_grad=grad)
    G, E2, at = G.cpu().numpy(), E2.cpu().numpy(), 0
    for k, m in enumerate(mols):
        n, rows = m.natoms, slice(off[k], off[k + 1])
        ek, ck = (eb[rows], cb[rows]) if atoms else (e, c)
        Gr, Er, _ = (oracle.fock_atoms if atoms else oracle.fock)(m.xyz, m.dens, ek, ck, tau)
        assert_close(G[at:at + n * n].reshape(n, n), Gr, TOL[precision], str(k))
        assert rel(E2[k], Er) < TOL[precision], k
        at += n * n
        if grad:
            gr, _, _ = (oracle.grad_atoms if atoms else oracle.grad)(m.xyz, m.dens, ek, ck, tau)
            # a one-atom molecule has no gradient: an absolute floor, as in the batched tests
            tol = 1e-10 if precision == "fp64" else TOL["mixed"]
            assert np.linalg.norm(dx[off[k]:off[k + 1]].cpu().numpy() - gr) <= tol * max(np.linalg.norm(gr), 1e-6), k
