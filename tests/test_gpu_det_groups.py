"""Workgroups of the deterministic strategy: each owns a copy of F and of the ket vector, which the
final kernels sum one after another, so a small system gains nothing from a sixth per compute unit.
The build against the oracle and bit for bit against itself at the largest size that had six."""
import numpy as np
import pytest

import oracle
from he_inputs import mixed_lattice, random_cluster
from gpu_util import announce, assert_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,atoms", [(64, False), (64, True), (82, False)])
def test_deterministic_mixed_groups(n, atoms):
    import torch
    import paper_2509_21039_amd as hfk
    dev = torch.device("cuda:0")
    s = mixed_lattice((4, 4, 4), seed=19, tau=1e-9) if atoms else random_cluster(n, 83, box=14.0, tau=1e-9)
    build, ref = (hfk.fock_atoms, oracle.fock_atoms) if atoms else (hfk.fock, oracle.fock)
    size = hfk.workspace_bytes_atoms if atoms else hfk.workspace_bytes
    announce("deterministic mixed n=%d atoms=%d" % (n, atoms))
    X, D = torch.tensor(s.xyz, device=dev), torch.tensor(s.dens, device=dev)
    runs = []
    for _ in range(2):
        ws = hfk.new_workspace(size(n, 3, "mixed"), dev)
        G, _ = build(X, D, s.exps, s.coefs, s.tau, "mixed", strategy=hfk.STRATEGY_DETERMINISTIC, workspace=ws)
        runs.append(G.cpu().numpy())
        assert hfk.read_stats(ws)["groups"] <= 5 * torch.cuda.get_device_properties(0).multi_processor_count
    assert np.array_equal(*runs)
    assert_close(runs[0], ref(s.xyz, s.dens, s.exps, s.coefs, s.tau)[0], 1e-6)
