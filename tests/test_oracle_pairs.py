"""The oracle's builds from lists of significant pairs and their primitive products, against its
plain definition, which forms every integral from the four centres over all pairs.

Both sum the same terms in FP64 in different orders, at most n^2 g^4 = 1.3e6 of them: errors
random in sign stay near sqrt(1.3e6) 1e-16 = 1e-13 of the largest element, held at 1e-12."""
import numpy as np
import pytest

from he_inputs import jittered_lattice, random_basis_rows, random_cluster


def test_build_over_significant_pairs_of_a_thin_lattice(oracle_lib):
    # 9 bohr apart: 125 of 7875 pairs survive; their far products underflow to zero
    s = jittered_lattice((5, 5, 5), seed=8, tau=1e-7, spacing=9.0)
    Q = oracle_lib.schwarz(s.xyz, s.exps, s.coefs)
    assert (Q * Q.max() >= s.tau).sum() < len(Q) // 10
    G, _, kept = oracle_lib.fock(s.xyz, s.dens, s.exps, s.coefs, s.tau)
    sig = Q[Q * Q.max() >= s.tau]
    assert kept == sum(int((sig[: x + 1] * q >= s.tau).sum()) for x, q in enumerate(sig))
    for i, j in [(0, 0), (3, 3), (124, 124), (7, 2), (90, 89), (124, 0)]:
        ref = oracle_lib.fock_element(s.xyz, s.dens, s.exps, s.coefs, s.tau, Q, i, j)
        assert abs(G[i, j] - ref) < 1e-12 * np.abs(G).max()


@pytest.mark.parametrize("n,g,tau", [(1, 2, 0.0), (5, 3, 0.0), (6, 6, 1e-6)])
def test_kept_integrals_contract_to_the_plain_definition(oracle_lib, n, g, tau):
    from oracle.scf import two_electron
    s = random_cluster(n, 60 + n, box=5.0)
    e, c = random_basis_rows(n, g, 70 + n)
    ref, _ = oracle_lib.fock_bruteforce_atoms(s.xyz, s.dens, e, c, tau)
    G = two_electron(s.xyz, e, c, tau)(s.dens)
    assert np.abs(G - ref).max() < 1e-12 * np.abs(ref).max()
    assert np.abs(oracle_lib.fock_atoms(s.xyz, s.dens, e, c, tau)[0] - ref).max() < 1e-12 * np.abs(ref).max()


def test_gradient_energy_is_the_builds(oracle_lib):
    s = random_cluster(9, 31, box=6.0)
    e, c = random_basis_rows(9, 4, 32)
    _, Eg, kept = oracle_lib.grad_atoms(s.xyz, s.dens, e, c, 1e-9)
    _, E, kept_f = oracle_lib.fock_atoms(s.xyz, s.dens, e, c, 1e-9)
    assert kept == kept_f and abs(Eg - E) < 1e-12 * abs(E)
