"""Rows from 64 kets in contraction classes of 4096 quartets and more: one s
and one p shell per atom, so that (ss|ss) has 3081, 4186 and 22155 quartets
and prefixes of up to 78, 91 and 210 kets, against the oracle."""
import numpy as np
import pytest

from oracle import oracle as o
from paper_2507_09772_amd import synth

pytestmark = pytest.mark.gpu
TOL = 1e-10  # the repository's FP64 bar


@pytest.fixture(scope="module")
def env():
    import torch

    from paper_2507_09772_amd import jk
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    torch.cuda.init()
    return torch, jk


def cluster(natom, seed):
    rng = np.random.default_rng(seed)
    l, ex, co = [], [], []
    for _ in range(natom):
        for ll in (0, 1):
            e = rng.uniform(0.3, 1.5, 2)
            l.append(ll)
            ex.append(e)
            co.append(synth._contract_norm(e, rng.uniform(0.3, 1.0, 2), ll))
    return synth.Molecule(l=np.asarray(l, np.int32), nprim=np.full(2 * natom, 2, np.int32),
                          atom=np.repeat(np.arange(natom, dtype=np.int32), 2), exps=np.concatenate(ex),
                          coefs=np.concatenate(co), coords=rng.uniform(-2.0, 2.0, (natom, 3)), spherical=False)


@pytest.mark.parametrize("natom,nset,rows", [(12, 1, False), (13, 2, True), (20, 1, True)])
def test_rows(env, natom, nset, rows):
    torch, jk = env
    mol = cluster(natom, 80 + natom)
    D = synth.random_density(mol.nao, 4, 81, nset)
    J0, K0, _ = o.jk(mol, D, 1e-13, mode=1)
    plan = jk.Plan(mol, 1e-13)
    plan.profile(True)
    J, K = plan.execute(torch.from_numpy(D).cuda())
    torch.cuda.synchronize()
    npair = natom * (natom + 1) // 2
    ss = [t for t in plan.timings() if (t.li, t.lj, t.lk, t.ll) == (0, 0, 0, 0)]
    print("rows", natom, [(t.kind, t.nquartets) for t in ss], flush=True)
    assert sum(t.nquartets for t in ss) == npair * (npair + 1) // 2
    assert any(t.kind == 1 for t in ss) == rows
    assert np.abs(J.cpu().numpy() - J0).max() <= TOL
    assert np.abs(K.cpu().numpy() - K0).max() <= TOL
    plan.close()
