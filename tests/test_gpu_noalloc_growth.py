"""The allocation-free call with a list that outgrows its estimate: it grows inside the
library's array and returns, bit for bit, what the handle (with a grown arena) returns;
a system whose grown list does not fit the array gets NB_ERR_CAPACITY."""
import numpy as np
import pytest

from paper_1506_00716_amd import inputs

pytestmark = pytest.mark.gpu


def crowded(n, fac, coulomb, lj):
    """n atoms on a lattice in the corner of a box of fac times its edge."""
    rng = np.random.default_rng(n)
    k = inputs.lattice_edge(n)
    i = np.arange(n)
    x = (np.stack([i % k, (i // k) % k, i // (k * k)], 1) + 0.5) * 0.24 + rng.uniform(-0.01, 0.01, (n, 3))
    m = inputs.Model(r_cut=0.9, r_list=1.0, coulomb=coulomb, lj=lj, ewald_beta=3.12 if coulomb == "ewald" else 0.0)
    return inputs.System(box=np.full(3, k * 0.24 * fac), x=x, q=inputs.alternating_charges(n),
                         sigma=rng.uniform(0.2, 0.25, n), epsilon=rng.uniform(0.2, 1.0, n), mass=np.full(n, 16.0),
                         model=m)


@pytest.mark.parametrize("coulomb,lj", [("ewald", "lb"), ("rf", "single")])
@pytest.mark.parametrize("n,fac", [(2744, 4.0), (5832, 3.0)])
def test_grown_call_equals_the_handle(nbmod, gpu_ctx, n, fac, coulomb, lj):
    import torch
    s = crowded(n, fac, coulomb, lj)
    print(f"[noalloc growth] N={n} {coulomb} {lj}", flush=True)
    x = torch.tensor(s.x, dtype=torch.float64, device=gpu_ctx.device)
    f = torch.zeros((n, 3), dtype=torch.float32, device=gpu_ctx.device)
    g = nbmod.System(gpu_ctx, s)
    size = g.arena.numel()
    e, w = g.compute_forces(x, f)
    assert size < g.arena.numel() <= nbmod.NOALLOC_MAX_BYTES
    g.close()
    for _ in range(2):
        fn = torch.full_like(f, float("nan"))
        en, wn = nbmod.compute_forces_noalloc(gpu_ctx, s, x, fn)
        assert torch.equal(f, fn) and np.array_equal(e, en) and np.array_equal(w, wn)


def test_growth_past_the_array(nbmod, gpu_ctx):
    import torch
    s = crowded(46656, 4.0, "rf", "single")
    assert nbmod.arena_bytes(nbmod.make_params(s.n, s.box, s.model)) <= nbmod.NOALLOC_MAX_BYTES
    print("[noalloc growth] past the array", flush=True)
    x = torch.tensor(s.x, dtype=torch.float64, device=gpu_ctx.device)
    f = torch.zeros((s.n, 3), dtype=torch.float32, device=gpu_ctx.device)
    with pytest.raises(nbmod.NbError) as exc:
        nbmod.compute_forces_noalloc(gpu_ctx, s, x, f)
    assert exc.value.code == nbmod.NB_ERR_CAPACITY
