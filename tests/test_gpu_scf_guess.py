"""The SCF from a density of the caller's, against the oracle's SCF from the same density (energy,
density and orbital energies; tolerances of the SCF tests on both sides of 64 atoms)."""
import numpy as np
import pytest

from oracle.scf import scf as oracle_scf
from he_inputs import HE_STO3G_COEFS as C3, HE_STO3G_EXPS as E3, H_STO3G_EXPS as H3, jittered_lattice
from gpu_util import announce, rel

pytestmark = pytest.mark.gpu


def _chains(n):
    """Helium atoms and H2 molecules in turn along a jittered lattice: a closed shell of n atoms."""
    rng, xyz, Z = np.random.default_rng(n + 5), [], []
    for p in jittered_lattice((5, 5, 5), seed=31, tau=0.0, spacing=4.0).xyz:
        if len(Z) + 2 <= n and len(xyz) % 3 != 0:
            axis = rng.normal(size=3)
            axis *= 0.7 / np.linalg.norm(axis)
            xyz += [p - axis, p + axis]
            Z += [1.0, 1.0]
        elif len(Z) < n:
            xyz.append(p)
            Z.append(2.0)
    Z = np.array(Z)
    return np.array(xyz), Z, np.where(Z[:, None] == 1.0, np.array(H3), np.array(E3)), np.tile(C3, (n, 1))


@pytest.mark.parametrize("n", [4, 28, 63, 64, 65])
@pytest.mark.parametrize("guess", ["identity", "random"])
def test_scf_from_a_guess_vs_oracle(n, guess):
    import torch
    import paper_2509_21039_amd as hfk
    dev, tau = torch.device("cuda:0"), 1e-9
    xyz, Z, e, c = _chains(n)
    nocc = int(Z.sum()) // 2
    m = np.random.default_rng(n).uniform(size=(n, n))
    D0 = np.eye(n) if guess == "identity" else np.eye(n) + 0.02 * (m + m.T)
    announce("scf from a guess n=%d %s" % (n, guess))
    ref = oracle_scf(xyz, Z, e, c, nocc, tau, d_tol=1e-10, e_tol=1e-11, D0=D0)
    assert ref["converged"]
    r = hfk.scf(torch.tensor(xyz, device=dev), Z, e, c, nocc, tau, d_tol=1e-10, e_tol=1e-11,
                dens0=torch.tensor(D0, device=dev))
    assert r["converged"] and rel(r["E"], ref["E"]) < 1e-10
    assert abs(r["D"].cpu().numpy() - ref["D"]).max() < 1e-7
    assert abs(r["eps"].cpu().numpy() - ref["eps"]).max() < 1e-7


def test_eigenproblem_with_nan_names_no_library_routine():
    # three atoms: the library's own one-workgroup eigenproblem, not the linear-algebra library's
    import torch
    import paper_2509_21039_amd as hfk
    dev = torch.device("cuda:0")
    xyz, Z, e, c = _chains(3)
    announce("scf nan guess n=3")
    with pytest.raises(hfk.HfkError) as err:
        hfk.scf(torch.tensor(xyz, device=dev), Z, e, c, 2, 1e-9,
                dens0=torch.full((3, 3), float("nan"), dtype=torch.float64, device=dev))
    assert err.value.status == hfk.HFK_EHIP
    assert "did not converge" in str(err.value) and "dsyevd" not in str(err.value)
