"""Large builds on both sides of the sizes where their workgroups widen from four waves to eight and
to sixteen: the workgroups per compute unit that the LDS holds, and G against the oracle's
element-wise definition.

Rows i and j of F take 16 n bytes of LDS next to the Boys table (18,864 bytes FP64, 8,576 FP32), 256
bytes per wave and 16 (FP32: 256) beside, of 163,840: four FP64 workgroups of four waves fit up to 1316
atoms, two of eight up to 3812; six FP32 ones of four waves up to 1090, two of eight up to 4440.

A thin lattice (9 bohr) whose neighbours survive the screen.  FP64 builds agree with the oracle to a
few 1e-15 of the largest element at these sizes, FP32 integrals to a few 1e-8."""
import numpy as np
import pytest

import oracle
from he_inputs import HE_STO3G_COEFS as C3, HE_STO3G_EXPS as E3, jittered_lattice
from gpu_util import announce, rel

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "mixed": 1e-6}


@pytest.mark.parametrize("n,g,atoms,precision,per_cu", [
    (1316, 3, False, "fp64", 4), (1317, 3, False, "fp64", 2), (1090, 3, False, "mixed", 6),
    (1091, 3, False, "mixed", 3), (3813, 3, False, "fp64", 1), (4441, 3, False, "mixed", 1),
    (1317, 3, True, "fp64", 2), (1091, 3, True, "mixed", 3), (3813, 3, True, "fp64", 1), (4441, 3, True, "mixed", 1),
    (1317, 1, False, "fp64", None), (1091, 1, True, "mixed", None), (3813, 2, False, "fp64", None),
    (1317, 2, True, "fp64", None), (4441, 2, False, "mixed", None)])
def test_either_side_of_a_width(n, g, atoms, precision, per_cu):
    import torch
    import paper_2509_21039_amd as hfk
    dev, tau = torch.device("cuda:0"), 1e-7
    m = int(np.ceil(n ** (1 / 3) - 1e-9))
    s = jittered_lattice((m, m, m), seed=900 + n, tau=tau, spacing=9.0)
    xyz, dens = np.ascontiguousarray(s.xyz[:n]), np.ascontiguousarray(s.dens[:n, :n])
    e, c = np.array(E3[3 - g:]), np.array(C3[3 - g:])
    build, schwarz, element = hfk.fock, oracle.schwarz, oracle.fock_element
    if atoms:
        e, c = e * np.random.default_rng(n).uniform(0.9, 1.1, n)[:, None], np.tile(c, (n, 1))
        build, schwarz, element = hfk.fock_atoms, oracle.schwarz_atoms, oracle.fock_element_atoms
    announce("wide workgroups n=%d g=%d atoms=%d %s" % (n, g, atoms, precision))
    ws = hfk.new_workspace((hfk.workspace_bytes_atoms if atoms else hfk.workspace_bytes)(n, g, precision), dev)
    G, E2 = build(torch.tensor(xyz, device=dev), torch.tensor(dens, device=dev), e, c, tau, precision, workspace=ws)
    st, G = hfk.read_stats(ws), G.cpu().numpy()
    Q = schwarz(xyz, e, c)
    q = np.sort(Q[Q * Q.max() >= tau])[::-1]
    assert len(q) > n     # pairs of neighbours among them
    kept = sum(int((q[: x + 1] * v >= tau).sum()) for x, v in enumerate(q))
    assert st["quartets"] == kept
    if per_cu:
        assert st["groups"] == per_cu * torch.cuda.get_device_properties(0).multi_processor_count
    i, j = np.tril_indices(n)
    near = np.flatnonzero((Q * Q.max() >= tau) & (i != j))
    rng = np.random.default_rng(n)
    at = [(int(i[x]), int(j[x])) for x in rng.choice(near, 4)] + [(int(x), int(x)) for x in rng.integers(0, n, 2)]
    at += [(n - 1, 0), (n - 1, n - 1)]
    for a, b in at:
        ref = element(xyz, dens, e, c, tau, Q, a, b)
        assert abs(G[a, b] - ref) < TOL[precision] * np.abs(G).max(), (a, b, G[a, b], ref)
    assert np.array_equal(G, G.T)
    assert rel(float(E2.item()), 0.5 * float(np.sum(dens * G))) < 1e-12
