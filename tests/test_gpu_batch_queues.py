"""The persistent form of a batch in mixed precision (a queue per precision on
branches of their own), replayed without waiting in between: every replay starts
from cleared queue heads, so J and K equal the form with one launch per class."""
import os

import numpy as np
import pytest

from paper_2507_09772_amd import synth

pytestmark = pytest.mark.gpu


def test_replays_of_the_queues():
    import torch

    from paper_2507_09772_amd import jk
    assert torch.cuda.is_available()
    wls = synth.batch_workload(nmol=8, nset=1, seed=17)
    print("queues", [w.mol.nwater for w in wls], flush=True)
    table = os.path.join(os.path.dirname(jk.__file__), "tune_gfx950.txt")
    saved = os.environ.get("JK_BATCH_PERSIST")
    try:
        # every class with both passes and row tasks of family 1
        for c in jk.canonical_classes():
            jk.tune_set_split(*c, 1)
            for p in ("fp64", "fp32"):
                _, avail = jk.tune_get(*c, p)
                jk.tune_set(*c, p, 1 if avail & 1 else 0)
        plans = [jk.Plan(w.mol, w.cutoff) for w in wls]
        Ds = [torch.from_numpy(w.D).cuda() for w in wls]
        out = {}
        batches = []
        for persist in ("0", "1"):
            os.environ["JK_BATCH_PERSIST"] = persist
            b = jk.Batch(plans, nset=1, precision="mixed")
            batches.append(b)
            Js, Ks = ([torch.full_like(D, np.nan) for D in Ds] for _ in range(2))
            for rep in range(4 if persist == "1" else 1):
                b.execute(Ds, Js, Ks)
            torch.cuda.synchronize()
            out[persist] = Js + Ks
            print("persist", persist, flush=True)
        for x, y in zip(out["0"], out["1"]):
            # (the same quartets in the same precisions, added in another order)
            assert (x - y).abs().max().item() <= 1e-9
        for b in batches:
            b.close()
    finally:
        if saved is None:
            os.environ.pop("JK_BATCH_PERSIST", None)
        else:
            os.environ["JK_BATCH_PERSIST"] = saved
        for c in jk.canonical_classes():
            jk.tune_set_split(*c, 1)
            for p in ("fp64", "fp32"):
                jk.tune_set(*c, p, 0)
        jk.tune_load(table)
