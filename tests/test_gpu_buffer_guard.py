"""The list-buffer guard counts a list lifetime once, whichever kernel measures it.

A rebuild's largest displacement is measured by the gather before it or, where a call
or some members of a batch begin with the rebuild, by the build's own first kernel; the
two leave different numbers of partials.  Atoms that translate together by 0.06 nm in one
lifetime (half the buffer is 0.05) and hardly move afterwards make one unsafe lifetime.
"""
import numpy as np
import pytest

from paper_1506_00716_amd import inputs

pytestmark = pytest.mark.gpu

DT, DRIFT = 0.001, 30.0  # 0.03 nm a step


def drifting(nbmod, ctx, n):
    import torch
    # a lattice at 0.35 nm: forces far too small to move an atom by the buffer
    k = inputs.lattice_edge(n)
    i = np.arange(n)
    x = (np.stack([i % k, (i // k) % k, i // (k * k)], 1) + 0.5) * 0.35
    m = inputs.Model(r_cut=0.9, r_list=1.0, coulomb="rf")
    s = inputs.System(box=np.full(3, k * 0.35), x=x, q=inputs.alternating_charges(n), sigma=np.full(n, 0.3),
                      epsilon=np.full(n, 0.5), mass=np.full(n, 16.0), model=m)
    x = torch.tensor(s.x, dtype=torch.float64, device=ctx.device)
    v = torch.zeros_like(x)
    v[:, 0] = DRIFT
    return nbmod.System(ctx, s), x, v, torch.zeros((s.n, 3), dtype=torch.float32, device=ctx.device)


@pytest.mark.parametrize("n", [1728, 21952])
def test_relaxation_after_dynamics(nbmod, gpu_ctx, n):
    print(f"[guard] minimize N={n}", flush=True)
    g, x, v, f = drifting(nbmod, gpu_ctx, n)
    g.md_step(x, v, f, DT, 2, nstlist=2)
    before = g.buffer_stats()
    assert before["unsafe_lifetimes"] == 1
    g.minimize(x, f, n_iter=4, f_tol=1e-3, max_disp=1e-5, nstlist=1)
    assert g.buffer_stats() == before
    g.close()


@pytest.mark.parametrize("apart", [0, 1])
def test_batch_that_begins_with_a_rebuild(nbmod, gpu_ctx, apart):
    # apart: the members' counters differ, so that one at a time is due
    print(f"[guard] ensemble apart {apart}", flush=True)
    ens = nbmod.Ensemble(gpu_ctx, 2)
    keep = [drifting(nbmod, gpu_ctx, n) for n in (1728, 4096)]
    for k in keep:
        ens.add(*k)
    ens.step(3, DT, nstlist=2)  # both at step 2: 0.06 nm
    for g, x, v, f in keep:
        assert g.buffer_stats()["unsafe_lifetimes"] == 1
        v.zero_()
    keep[1][0].step += apart
    ens.step(2, DT, nstlist=2)
    ens.step(2, DT, nstlist=2)
    for g, x, v, f in keep:
        assert g.buffer_stats()["unsafe_lifetimes"] == 1
    ens.close()
