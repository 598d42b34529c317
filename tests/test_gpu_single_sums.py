"""The single-precision pass sums a quartet's primitive integrals smallest first.

K of mixed builds against FP64 builds of the same molecules, root mean square
over seeds, relative: with the primitive pairs in ascending order of their size
2.5e-12 (4 waters) and 2.1e-12 (7 waters, two densities) in basis A, in
descending order 2.9e-12 and 2.7e-12; the limits lie half way."""
import numpy as np
import pytest

from paper_2507_09772_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nw,nset,limit", [(4, 1, 2.7e-12), (7, 2, 2.4e-12)])
def test_mixed_error(nw, nset, limit):
    import torch

    from paper_2507_09772_amd import jk
    assert torch.cuda.is_available()
    print("single sums", nw, flush=True)
    err = []
    for seed in range(12):
        elems, xyz = synth.water_lattice(nw, [7, seed, nw])
        mol = synth.build_molecule(synth.make_basis("A"), elems, xyz)
        D = torch.from_numpy(synth.random_density(mol.nao, synth.OCC_PER_WATER * nw, [8, seed], nset)).cuda()
        plan = jk.Plan(mol, 1e-13)
        _, K0 = plan.execute(D)
        _, K = plan.execute(D, precision="mixed")
        torch.cuda.synchronize()
        assert plan.stats().nquartets_fp32 > 0
        err.append(((K - K0).norm() / K0.norm()).item())
        plan.close()
    rms = float(np.sqrt(np.mean(np.square(err))))
    print("rms", rms, flush=True)
    assert rms <= limit
