"""The SCF on both sides of the size up to which its dense part runs in one workgroup, odd and
even, against the oracle's numpy SCF.  The density is converged to an error matrix below 1e-10,
so the energy (quadratic in it) is held to 1e-10 relative and the density to 1e-7."""
import numpy as np
import pytest

from oracle.scf import scf as oracle_scf
from he_inputs import HE_STO3G_COEFS as C3, HE_STO3G_EXPS as E3, H_STO3G_EXPS as H3, mixed_lattice
from gpu_util import announce, rel

pytestmark = pytest.mark.gpu


def _molecules(n):
    """H2 molecules and helium atoms in turn on a jittered lattice: a closed shell of n atoms."""
    rng, xyz, Z = np.random.default_rng(n), [], []
    for p in mixed_lattice((4, 4, 4), seed=77, tau=1e-9, spacing=4.0).xyz:
        if len(Z) % 3 == 0 and len(Z) + 2 <= n:
            axis = rng.normal(size=3)
            axis *= 0.7 / np.linalg.norm(axis)
            xyz += [p - axis, p + axis]
            Z += [1.0, 1.0]
        elif len(Z) < n:
            xyz.append(p)
            Z.append(2.0)
    Z = np.array(Z)
    return np.array(xyz), Z, np.where(Z[:, None] == 1.0, np.array(H3), np.array(E3)), np.tile(C3, (n, 1))


@pytest.mark.parametrize("n", [2, 3, 27, 63, 64, 65])
@pytest.mark.parametrize("guess", [False, True])
def test_scf_vs_oracle(n, guess):
    import torch
    import paper_2509_21039_amd as hfk
    dev = torch.device("cuda:0")
    xyz, Z, e, c = _molecules(n)
    tau, nocc = 1e-9, int(Z.sum()) // 2
    announce("scf n=%d guess=%d" % (n, guess))
    start = torch.eye(n, dtype=torch.float64, device=dev) if guess else None
    r = hfk.scf(torch.tensor(xyz, device=dev), Z, e, c, nocc, tau, d_tol=1e-10, e_tol=1e-11, dens0=start)
    assert r["converged"]
    D, eps = r["D"].cpu().numpy(), r["eps"].cpu().numpy()
    assert np.all(np.diff(eps) >= 0.0) and abs(D - D.T).max() < 1e-12
    if not guess:
        ref = oracle_scf(xyz, Z, e, c, nocc, tau, d_tol=1e-10, e_tol=1e-11)
        assert rel(r["E"], ref["E"]) < 1e-10
        assert abs(D - ref["D"]).max() < 1e-7
        assert abs(eps - ref["eps"]).max() < 1e-7
    else:
        again = hfk.scf(torch.tensor(xyz, device=dev), Z, e, c, nocc, tau, d_tol=1e-10, e_tol=1e-11, dens0=r["D"])
        assert again["converged"] and rel(again["E"], r["E"]) < 1e-10
