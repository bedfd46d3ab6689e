"""Block-per-item launches at both ends of an item's make-up: many entries of few
i-clusters each (a gas: about 18 entries of 2 an item), and few that list all 8
(groups of atoms far apart: 24 such entries in a row per group).  Against the energy
pass (a wave per item) bit for bit, and against the FP64 oracle.

The oracle bound is the 1e-5 rel-RMS of the force tests.
"""
import numpy as np
import pytest

import oracle
from paper_1506_00716_amd import inputs

pytestmark = pytest.mark.gpu


def gas(n, edge):
    """n atoms at random, no two closer than 0.25 nm: most cluster pairs hold one atom pair."""
    rng = np.random.default_rng(n)
    x = np.zeros((0, 3))
    while len(x) < n:
        c = rng.uniform(0.0, edge, 3)
        d = x - c
        d -= np.rint(d / edge) * edge
        if not len(x) or (d ** 2).sum(1).min() > 0.25 ** 2:
            x = np.concatenate([x, c[None]])
    return x, edge


def blobs(m):
    """m^3 groups of 4^3 atoms at 0.1 nm, 1.1 nm apart: every cluster of a group is within
    r_list of every cluster of a face neighbour, and of no other group's."""
    b, i = np.meshgrid(np.arange(m ** 3), np.arange(64), indexing="ij")
    corner = np.stack([b % m, (b // m) % m, b // (m * m)], -1)
    place = np.stack([i % 4, (i // 4) % 4, i // 16], -1)
    return (corner * 1.1 + place * 0.1 + 0.4).reshape(-1, 3), m * 1.1


@pytest.mark.parametrize("coulomb,lj", [("rf", "single"), ("ewald", "lb")])
@pytest.mark.parametrize("kind", ["one", "eight"])
def test_full_items(nbmod, gpu_ctx, kind, coulomb, lj):
    import torch
    x, edge = gas(1500, 12.0) if kind == "one" else blobs(3)
    rng = np.random.default_rng(1)
    m = inputs.Model(r_cut=1.0, r_list=1.12, coulomb=coulomb, lj=lj, ewald_beta=2.5 if coulomb == "ewald" else 0.0,
                     sigma=0.1)
    s = inputs.System(box=np.full(3, edge), x=x, q=rng.uniform(-0.5, 0.5, len(x)), sigma=np.full(len(x), 0.1),
                      epsilon=rng.uniform(0.2, 1.0, len(x)), mass=np.full(len(x), 16.0), model=m)
    g = nbmod.System(gpu_ctx, s)
    x = torch.tensor(s.x, dtype=torch.float64, device=gpu_ctx.device)
    f = torch.zeros((s.n, 3), dtype=torch.float32, device=gpu_ctx.device)
    fe = torch.zeros_like(f)
    g.build_pairlist(x)
    st = g.stats()
    per_entry, per_item = st["cluster_pairs"] / st["entries"], st["entries"] / st["items"]
    print(f"[split full] {kind} {coulomb} {lj}: {per_entry:.2f} cluster pairs an entry, {per_item:.1f} entries an item",
          flush=True)
    g.compute_forces(x, f, energies=False)
    g.compute_forces(x, fe)
    g.close()
    assert torch.equal(f, fe)
    fr, _, _ = oracle.forces(s)
    fn = f.cpu().numpy().astype(np.float64)
    assert np.sqrt(((fn - fr) ** 2).sum() / (fr ** 2).sum()) <= 1e-5
