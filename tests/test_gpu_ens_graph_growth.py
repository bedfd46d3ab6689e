"""An ensemble's kept graph grows with the runs of plain steps that it meets: calls of
growing, then shrinking length, some with replays of the graph before in flight, equal
the plain launches bit for bit."""
import numpy as np
import pytest

from paper_1506_00716_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nstlist,calls", [(100, [4, 5, 8, 20, 50, 6, 3]), (7, [5, 23, 9])])
def test_growing_runs(nbmod, gpu_ctx, nstlist, calls):
    import torch
    print(f"[ens graph] growth nstlist={nstlist}", flush=True)
    out = []
    for use_graph in (True, False):
        ens = nbmod.Ensemble(gpu_ctx, 3)
        state = []
        for i, n in enumerate([1000, 1331, 1728]):
            rng = np.random.default_rng(i)
            k = inputs.lattice_edge(n)
            j = np.arange(n)
            x = (np.stack([j % k, (j // k) % k, j // (k * k)], 1) + 0.5) * 0.28
            m = inputs.Model(r_cut=0.9, r_list=1.05, coulomb="rf")
            s = inputs.System(box=np.full(3, k * 0.28), x=x, q=inputs.alternating_charges(n), sigma=np.full(n, 0.25),
                              epsilon=np.full(n, 0.5), mass=np.full(n, 16.0), model=m)
            state.append((nbmod.System(gpu_ctx, s), torch.tensor(x, device=gpu_ctx.device),
                          torch.tensor(rng.normal(0.0, 0.3, (n, 3)), device=gpu_ctx.device),
                          torch.zeros((n, 3), dtype=torch.float32, device=gpu_ctx.device)))
            ens.add(*state[-1])
        rows = [ens.step(n, 0.001, nstlist=nstlist, use_graph=use_graph, energies=True) for n in calls]
        out.append([t.cpu().numpy() for st in state for t in st[1:]] + rows)
        ens.close()
    assert all(np.array_equal(a, b) for a, b in zip(*out))
    assert all(np.isfinite(a).all() for a in out[0])
