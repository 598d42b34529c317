"""Family-2 tiles: quartets on one to four waves (36 to 225 slots), one to
eight steps a tile, several densities, against the oracle; and bitwise
repeatable in the fixed-order mode."""
import os

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


@pytest.fixture()
def tiles_only(env):
    """Family 2 and tiles for every class that has them."""
    _, jk = env
    try:
        for c in jk.canonical_classes():
            for p in ("fp64", "fp32"):
                _, avail = jk.tune_get(*c, p)
                jk.tune_set(*c, p, 2 if avail & 2 else 0)
                jk.tune_set_row(*c, p, 2)
        yield
    finally:
        for c in jk.canonical_classes():
            for p in ("fp64", "fp32"):
                jk.tune_set(*c, p, 0)
                jk.tune_set_row(*c, p, 0)
        jk.tune_load(os.path.join(os.path.dirname(jk.__file__), "tune_gfx950.txt"))


@pytest.mark.parametrize("basis,nw,nset", [("C", 1, 2), ("B", 3, 1), ("B", 2, 3)])
def test_tiles(env, tiles_only, basis, nw, nset):
    torch, jk = env
    wl = synth.small_workload(nw, basis, seed=810 + nw, nset=nset)
    print("family-2 tiles", basis, nw, nset, flush=True)
    J0, K0, _ = o.jk(wl.mol, wl.D, wl.cutoff, mode=1)
    D = torch.from_numpy(wl.D).cuda()
    plan = jk.Plan(wl.mol, wl.cutoff)
    flags = jk.JK_DO_J | jk.JK_DO_K
    J, K = plan.execute(D)
    Jd, Kd = plan.execute(D, flags=flags | jk.JK_DETERMINISTIC)
    Je, Ke = plan.execute(D, flags=flags | jk.JK_DETERMINISTIC)
    _, K1 = plan.execute(D, flags=jk.JK_DO_K)
    torch.cuda.synchronize()
    for M, M0 in ((J, J0), (K, K0), (Jd, J0), (Kd, K0), (K1, K0)):
        assert np.abs(M.cpu().numpy() - M0).max() <= TOL
    assert torch.equal(Jd, Je) and torch.equal(Kd, Ke)
    plan.close()
