"""One launch per angular class: molecules whose contraction classes exceed
one launch's list (64), with and without the K rows of row mode, against the
oracle; and the same build timed class by class."""
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


def many_contractions(ncontr, natom, seed):
    """natom atoms, each with one s shell of every length 1..ncontr and a p
    shell: ncontr (ncontr + 1) / 2 types of (s, s) pairs."""
    rng = np.random.default_rng(seed)
    l, npr, atom, ex, co = [], [], [], [], []
    lengths = [(0, n) for n in range(1, ncontr + 1)] + [(1, 2)]
    shells = []
    for ll, n in lengths:
        e = np.exp(rng.uniform(np.log(0.1), np.log(30.0), n))
        shells.append((ll, e, synth._contract_norm(e, rng.uniform(0.2, 1.0, n), ll)))
    for a in range(natom):
        for ll, e, c in shells:
            l.append(ll)
            npr.append(e.size)
            atom.append(a)
            ex.append(e)
            co.append(c)
    return synth.Molecule(l=np.asarray(l, np.int32), nprim=np.asarray(npr, np.int32), atom=np.asarray(atom, np.int32),
                          exps=np.concatenate(ex), coefs=np.concatenate(co),
                          coords=rng.uniform(-2.5, 2.5, (natom, 3)), spherical=False)


@pytest.mark.parametrize("ncontr,natom,nset", [(5, 2, 1), (12, 2, 2), (4, 12, 1)])
def test_many_contraction_classes(env, ncontr, natom, nset):
    torch, jk = env
    mol = many_contractions(ncontr, natom, 60 + ncontr)
    D = synth.random_density(mol.nao, 4, 61, nset)
    J0, K0, _ = o.jk(mol, D, 1e-13, mode=1)
    plan = jk.Plan(mol, 1e-13)
    st = plan.stats()
    print("contractions", ncontr, natom, st.nclasses, st.nquartets, flush=True)
    Dd = torch.from_numpy(D).cuda()
    for timed in (False, True):
        plan.profile(timed)
        J, K = plan.execute(Dd)
        torch.cuda.synchronize()
        assert np.abs(J.cpu().numpy() - J0).max() <= TOL
        assert np.abs(K.cpu().numpy() - K0).max() <= TOL
        assert plan.stats().nquartets_evaluated == st.nquartets
    assert sum(t.nquartets for t in plan.timings()) == st.nquartets
    # counted on the device, class by class (threshold 0: every quartet in FP64)
    plan.profile(False)
    J, K = plan.execute(Dd, precision="mixed", mix_threshold=0.0)
    torch.cuda.synchronize()
    assert np.abs(J.cpu().numpy() - J0).max() <= TOL and np.abs(K.cpu().numpy() - K0).max() <= TOL
    s2 = plan.stats()
    assert s2.nquartets_evaluated == st.nquartets and s2.nquartets_fp32 == 0
    plan.close()
