"""Family-2 tiles of several steps: a tile walks up to eight steps of kets of
one bra where a contraction class has 16384 tiles of one step and more.  Two
densities, J and K, K alone, with density screening (steps that are skipped or
end the tile) and in the fixed-order mode, against the oracle."""
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


def steps_of_classes(mol, Q, cutoff):
    """{(lanes of a quartet, steps of a tile)} over the contraction classes with
    tiles of several steps, from the planner's rule."""
    nc = [1, 3, 6, 10, 15]
    keys = sorted({(int(l), int(n)) for l, n in zip(mol.l, mol.nprim)}, reverse=True)
    of = {k: [i for i in range(mol.nshell) if (mol.l[i], mol.nprim[i]) == k] for k in keys}
    pairs = {}
    for x, a in enumerate(keys):
        for b in keys[x:]:
            q = np.array([Q[i, j] for i in of[a] for j in of[b] if a != b or i >= j])
            pairs[a, b] = -np.sort(-q)
    out = set()
    names = list(pairs)
    for x, bra in enumerate(names):
        for ket in names[x:]:
            # the kernels' class: the pair of the larger angular momenta in front
            B, K = (bra, ket) if (bra[0][0], bra[1][0]) >= (ket[0][0], ket[1][0]) else (ket, bra)
            slots = nc[B[0][0]] * nc[K[0][0]]
            if nc[B[0][0]] * nc[B[1][0]] * nc[K[0][0]] * nc[K[1][0]] < 18:
                continue  # (not built as family 2)
            qw = 1 if slots >= 64 else 64 // slots
            cnt = np.searchsorted(-pairs[K], -cutoff / np.maximum(pairs[B], 1e-300), side="right")
            if B == K:
                cnt = np.minimum(cnt, np.arange(cnt.size) + 1)
            steps = min(8, int(((cnt + qw - 1) // qw).sum()) // 8192)
            if steps > 1:
                out.add((slots, steps))
    return out


@pytest.mark.parametrize("basis,nw", [("B", 6), ("C", 2)])
def test_tiles_of_several_steps(env, basis, nw):
    torch, jk = env
    wl = synth.small_workload(nw, basis, seed=840, nset=2)
    print("steps", basis, nw, flush=True)
    J0, K0, _ = o.jk(wl.mol, wl.D, wl.cutoff, mode=1)
    Js0, Ks0, _ = o.jk(wl.mol, wl.D, wl.cutoff, mode=1, dscreen=1e-6)
    D = torch.from_numpy(wl.D).cuda()
    flags = jk.JK_DO_J | jk.JK_DO_K
    try:
        for c in jk.canonical_classes():
            _, avail = jk.tune_get(*c, "fp64")
            jk.tune_set(*c, "fp64", 2 if avail & 2 else 0)
            jk.tune_set_row(*c, "fp64", 2)
        plan = jk.Plan(wl.mol, wl.cutoff)
        steps = steps_of_classes(wl.mol, plan.schwarz(), wl.cutoff)
        print(sorted(steps), flush=True)
        # several steps with several quartets a wave, and with several waves a quartet
        assert max(s for _, s in steps) >= 5 and any(n <= 32 for n, _ in steps)
        assert basis == "B" or any(n > 64 for n, _ in steps)
        J, K = plan.execute(D)
        _, K1 = plan.execute(D, flags=jk.JK_DO_K)
        Jd, Kd = plan.execute(D, flags=flags | jk.JK_DETERMINISTIC)
        Je, Ke = plan.execute(D, flags=flags | jk.JK_DETERMINISTIC)
        plan.set_density_screening(1e-6)
        Js, Ks = plan.execute(D)
        torch.cuda.synchronize()
        for M, M0 in ((J, J0), (K, K0), (K1, K0), (Jd, J0), (Kd, K0), (Js, Js0), (Ks, Ks0)):
            assert np.abs(M.cpu().numpy() - M0).max() <= TOL
        assert torch.equal(Jd, Je) and torch.equal(Kd, Ke)
        plan.close()
    finally:
        for c in jk.canonical_classes():
            jk.tune_set(*c, "fp64", 0)
            jk.tune_set_row(*c, "fp64", 0)
        jk.tune_load(os.path.join(os.path.dirname(jk.__file__), "tune_gfx950.txt"))
