"""Batches against the oracle, molecule by molecule: three densities, short and
long bras (64- and 256-lane rows), D rows staged in LDS and read from memory, in
FP64 and mixed precision.

Mixed tolerance: as for single precision, a quartet is off by at most 1e-4 of
Q_ij Q_kl (roots good to 3e-6, three recurrences of them, some ten Cartesian
integrals in a spherical one).
"""
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
    assert torch.cuda.is_available()
    torch.cuda.init()
    wls = [synth.small_workload(n, b, seed=950 + n, nset=3) for b, n in (("A", 1), ("B", 1), ("A", 6), ("B", 3), ("A", 2))]
    ref = [o.jk(w.mol, w.D, w.cutoff, mode=1)[:2] for w in wls]
    return torch, jk, wls, ref


@pytest.mark.parametrize("staged", [True, False])
def test_batch(env, staged):
    torch, jk, wls, ref = env
    saved = os.environ.get("JK_NO_DSTAGE")
    os.environ["JK_NO_DSTAGE"] = "0" if staged else "1"
    try:
        plans = [jk.Plan(w.mol, w.cutoff) for w in wls]
    finally:
        os.environ.pop("JK_NO_DSTAGE") if saved is None else os.environ.update(JK_NO_DSTAGE=saved)
    Ds = [torch.from_numpy(w.D).cuda() for w in wls]
    for prec in ("fp64", "mixed"):
        print("batch", prec, staged, flush=True)
        Js, Ks = ([torch.full_like(D, np.nan) for D in Ds] for _ in range(2))
        b = jk.Batch(plans, nset=3, precision=prec)
        b.execute(Ds, Js, Ks)
        torch.cuda.synchronize()
        n, n32 = b.stats()
        assert n == sum(p.stats().nquartets for p in plans) and (n32 > 0) == (prec == "mixed")
        for w, p, J, K, (J0, K0) in zip(wls, plans, Js, Ks, ref):
            nf = [2 * l + 1 if w.mol.spherical else (l + 1) * (l + 2) // 2 for l in w.mol.l]
            Q = np.repeat(np.repeat(p.schwarz(), nf, 0), nf, 1)
            for s in range(3):
                A = np.abs(w.D[s])
                dj, dk = np.abs(J[s].cpu().numpy() - J0[s]), np.abs(K[s].cpu().numpy() - K0[s])
                tj, tk = (TOL, TOL) if prec == "fp64" else (TOL + 1e-4 * Q * (Q * A).sum(), TOL + 1e-4 * Q @ A @ Q)
                assert (dj <= tj).all() and (dk <= tk).all(), (prec, w.name, s, dj.max(), dk.max())
        b.close()


@pytest.mark.parametrize("copies", [2, 40])
def test_copies(env, copies):
    """The same molecule 2 and 40 times: launches that leave the device idle (the
    LDS sizes of a kernel together, the double-precision pass as tiles) and ones
    that fill it (apart, rows); every copy against the oracle."""
    torch, jk, wls, ref = env
    w, (J0, K0) = wls[3], ref[3]
    a, (Ja, Ka) = wls[0], ref[0]
    plan, small = jk.Plan(w.mol, w.cutoff), jk.Plan(a.mol, a.cutoff)
    D, d = torch.from_numpy(w.D).cuda(), torch.from_numpy(a.D).cuda()
    Ds = [D, d] * copies
    for prec in ("fp64", "mixed"):
        print("copies", prec, copies, flush=True)
        Js, Ks = ([torch.full_like(x, np.nan) for x in Ds] for _ in range(2))
        b = jk.Batch([plan, small] * copies, nset=3, precision=prec)
        b.execute(Ds, Js, Ks)
        torch.cuda.synchronize()
        n, n32 = b.stats()
        assert n == copies * (plan.stats().nquartets + small.stats().nquartets)
        nf = [2 * l + 1 for l in w.mol.l]
        Q = np.repeat(np.repeat(plan.schwarz(), nf, 0), nf, 1)
        A = np.abs(w.D)
        tj, tk = ((TOL, TOL) if prec == "fp64" else
                  (TOL + 1e-4 * Q * np.einsum("kl,skl->s", Q, A)[:, None, None], TOL + 1e-4 * Q @ A @ Q))
        for J, K in zip(Js[::2], Ks[::2]):
            assert (np.abs(J.cpu().numpy() - J0) <= tj).all() and (np.abs(K.cpu().numpy() - K0) <= tk).all(), (prec, copies)
        for J, K in zip(Js[1::2], Ks[1::2]):
            assert np.abs(J.cpu().numpy() - Ja).max() <= 1e-9 and np.abs(K.cpu().numpy() - Ka).max() <= 1e-9
        b.close()
