"""A batch is made and run at once on a stream that does not wait for the null
stream: its tasks and descriptors are there, and J and K are the single builds'."""
import pytest

from paper_2507_09772_amd import synth

pytestmark = pytest.mark.gpu


def test_first_run_on_a_side_stream():
    import torch

    from paper_2507_09772_amd import jk
    assert torch.cuda.is_available()
    wls = synth.batch_workload(nmol=16, nset=1, seed=19)
    print("side stream", [w.mol.nwater for w in wls], flush=True)
    plans = [jk.Plan(w.mol, w.cutoff) for w in wls]
    Ds = [torch.from_numpy(w.D).cuda() for w in wls]
    ref = [p.execute(D) for p, D in zip(plans, Ds)]
    Js, Ks = ([torch.zeros_like(D) for D in Ds] for _ in range(2))
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    b = jk.Batch(plans, nset=1)
    with torch.cuda.stream(side):
        b.execute(Ds, Js, Ks)
    side.synchronize()
    for J, K, (J0, K0) in zip(Js, Ks, ref):
        assert (J - J0).abs().max().item() <= 1e-12 and (K - K0).abs().max().item() <= 1e-12
    torch.cuda.synchronize()
    b.close()
