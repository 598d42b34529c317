"""Primitive pairs kept by the plan: those left out (and the two orders of a
shell's pair with itself held as one) must not show in double precision.

Integral blocks against the oracle, relative to the product of the Schwarz
factors of their pairs.  Tolerance: a block is a sum of N primitive terms,
whose rounding is at most about N 2^-53 of that product; 64 covers the
operations of one term and the transfers over centres a few bohr apart.
"""
import numpy as np
import pytest

from oracle import oracle as o
from paper_2507_09772_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch

    from paper_2507_09772_amd import jk
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    torch.cuda.init()
    return torch, jk


def contracted(ls, nprim, sep, seed, signs):
    """Shells of nprim primitives with exponents over seven decades, alternately
    on two atoms sep bohr apart; signs: coefficients of both signs."""
    rng = np.random.default_rng(seed)
    n = len(ls) * nprim
    exps = np.exp(rng.uniform(np.log(0.02), np.log(2e5), n))
    # primitives of about unit norm
    coefs = rng.uniform(0.2, 1.0, n) * exps ** (0.75 + 0.5 * np.repeat(np.asarray(ls), nprim))
    if signs:
        coefs *= np.where(rng.random(n) < 0.5, -1.0, 1.0)
    return synth.Molecule(l=np.asarray(ls, np.int32), nprim=np.full(len(ls), nprim, np.int32),
                          atom=np.arange(len(ls), dtype=np.int32) % 2, exps=exps, coefs=coefs,
                          coords=np.array([[0.1, -0.2, 0.3], [0.1, -0.2 + 0.6 * sep, 0.3 + 0.8 * sep]]), spherical=False)


@pytest.mark.parametrize("nprim,sep,signs", [(1, 2.0, False), (2, 0.0, True), (6, 1.7, False), (9, 6.0, True),
                                             (16, 0.0, False), (16, 3.0, True), (16, 40.0, False)])
def test_blocks_of_contracted_shells(env, nprim, sep, signs):
    _, jk = env
    ls = [0, 0, 1, 1, 0]
    mol = contracted(ls, nprim, sep, 500 + nprim, signs)
    print("contracted", nprim, sep, signs, flush=True)
    plan = jk.Plan(mol)
    Q = plan.schwarz()
    worst = 0.0
    for I, J, K, L in [(0, 0, 0, 0), (1, 1, 0, 0), (0, 1, 0, 1), (2, 2, 2, 2), (3, 2, 3, 2), (3, 3, 1, 4), (2, 0, 4, 4),
                       (2, 4, 3, 0), (4, 0, 2, 2), (1, 4, 1, 4)]:
        ref = o.eri_block(mol, I, J, K, L)
        got = plan.eri_block(I, J, K, L)
        scale = Q[I, J] * Q[K, L]
        if scale < 1e-250:
            continue
        err = np.abs(got - ref).max() / scale
        worst = max(worst, err)
        assert err <= 64 * nprim ** 4 * 2.0 ** -53, ((I, J, K, L), err)
    print("worst", worst, flush=True)
    plan.close()


@pytest.mark.parametrize("nprim,signs", [(3, False), (16, True)])
def test_matrices_of_contracted_shells(env, nprim, signs):
    """J and K against the oracle: the quartets of one wave hold different
    numbers of primitive pairs (shells on two atoms)."""
    torch, jk = env
    ls = [0, 1, 0, 1, 2, 0, 1, 2]
    mol = contracted(ls, nprim, 2.5, 900 + nprim, signs)
    nao = mol.nao
    rng = np.random.default_rng(3)
    D = rng.standard_normal((2, nao, nao))
    D = D + D.transpose(0, 2, 1)
    J0, K0, _ = o.jk(mol, D, 0.0, mode=1)
    plan = jk.Plan(mol, 0.0)
    # every element is a sum of at most nao^2 integrals, each off by at most
    # its rounding above
    tol = 64 * nprim ** 4 * 2.0 ** -53 * nao ** 2 * float(plan.schwarz().max()) ** 2 * np.abs(D).max()
    for prec in ("fp64", "mixed"):
        J, K = plan.execute(torch.from_numpy(D).cuda(), precision=prec, mix_threshold=0.0)
        torch.cuda.synchronize()
        print("matrices", nprim, prec, np.abs(J.cpu().numpy() - J0).max(), np.abs(K.cpu().numpy() - K0).max(), tol, flush=True)
        assert np.abs(J.cpu().numpy() - J0).max() <= tol
        assert np.abs(K.cpu().numpy() - K0).max() <= tol
    plan.close()


@pytest.mark.parametrize("nprim,nwater", [(2, 1), (4, 1), (5, 2), (16, 1)])
def test_shared_quartets(env, nprim, nwater):
    """Few quartets of long contractions: neighbouring lanes share a quartet's
    ket primitive pairs (2, 4, 8, 16 or 32 of them).  Against the oracle, with
    density screening (lanes of dropped quartets beside others) and J alone."""
    torch, jk = env
    elems, xyz = synth.water_lattice(nwater, 77)
    rng = np.random.default_rng(nprim)
    shells = []
    for l in (0, 1, 2, 0):
        e = np.exp(rng.uniform(np.log(0.1), np.log(500.0), nprim))
        shells.append((l, e, synth._contract_norm(e, rng.uniform(0.2, 1.0, nprim), l)))
    mol = synth.build_molecule(synth.BasisTemplate("long", False, {"O": shells, "H": shells[:2]}), elems, xyz)
    D = synth.random_density(mol.nao, 3 * nwater, 78, 2)
    Dd = torch.from_numpy(D).cuda()
    plan = jk.Plan(mol, 1e-13)
    J0, K0, _ = o.jk(mol, D, 1e-13, mode=1)
    J, K = plan.execute(Dd)
    J1, _ = plan.execute(Dd, flags=jk.JK_DO_J)
    plan.set_density_screening(1e-12)
    J2, K2 = plan.execute(Dd)
    torch.cuda.synchronize()
    for x, y in ((J, J0), (K, K0), (J1, J0), (J2, J0), (K2, K0)):
        # (the screened contributions are below 1e-12 each, some 1e2 of them per element)
        assert np.abs(x.cpu().numpy() - y).max() <= 1e-10, (nprim, nwater)
    plan.close()
