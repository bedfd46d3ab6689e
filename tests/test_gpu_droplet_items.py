"""Systems with much empty space: the pair kernel's form follows the work items of the
built list, not the box's mean density, and every form gives the same bits.

A droplet's launches without energies (the first after the build, in dynamics with
rebuilds, and in a batch) against its energy passes, which always take a wave per item.
"""
import numpy as np
import pytest

from paper_1506_00716_amd import inputs

pytestmark = pytest.mark.gpu


def droplet(n, fac):
    rng = np.random.default_rng(n)
    k = inputs.lattice_edge(n)
    i = np.arange(n)
    x = (np.stack([i % k, (i // k) % k, i // (k * k)], 1) + 0.5) * 0.26 + rng.uniform(-0.01, 0.01, (n, 3))
    m = inputs.Model(r_cut=0.9, r_list=1.0, coulomb="ewald", ewald_beta=3.12)
    return inputs.System(box=np.full(3, max(k * 0.26 * fac, 2.1)), x=x, q=inputs.alternating_charges(n),
                         sigma=np.full(n, 0.25), epsilon=np.full(n, 0.5), mass=np.full(n, 16.0),
                         v=rng.normal(0.0, 0.3, (n, 3)), model=m)


@pytest.mark.parametrize("n,fac", [(1000, 4.0), (5832, 1.0), (21952, 2.0), (32768, 4.0)])
def test_forms_agree(nbmod, gpu_ctx, n, fac):
    import torch
    s = droplet(n, fac)
    print(f"[droplet] N={n} box {fac}", flush=True)

    def state(g):
        x = torch.tensor(s.x, dtype=torch.float64, device=gpu_ctx.device)
        v = torch.tensor(s.v, dtype=torch.float64, device=gpu_ctx.device)
        g.build_pairlist(x)  # (an arena that holds the list: a batch does not grow it)
        g.state_import(x, v, g.state_export(x, v))  # (the list is dropped)
        return g, x, v, torch.zeros((s.n, 3), dtype=torch.float32, device=gpu_ctx.device)

    g, x, v, f = state(nbmod.System(gpu_ctx, s))
    fe = torch.zeros_like(f)
    for _ in range(2):  # with the estimate or the count at hand, and again
        g.compute_forces(x, f, energies=False)
        g.compute_forces(x, fe)
        assert torch.equal(f, fe) and float(f.abs().max()) > 0.0
    g.md_step(x, v, f, 0.001, 7, nstlist=3, nstenergy=0)
    r, xr, vr, fr = state(nbmod.System(gpu_ctx, s))
    r.md_step(xr, vr, fr, 0.001, 7, nstlist=3, nstenergy=1)  # (energies: a wave per item)
    ens = nbmod.Ensemble(gpu_ctx, 2)
    mem = [state(nbmod.System(gpu_ctx, s)) for _ in range(2)]
    for k in mem:
        ens.add(*k)
    ens.step(7, 0.001, nstlist=3)
    for _, xm, vm, fm in [(r, xr, vr, fr)] + mem:
        assert torch.equal(x, xm) and torch.equal(v, vm) and torch.equal(f, fm)
    ens.close()
    g.close()
    r.close()
