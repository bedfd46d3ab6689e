"""md_step that runs out of list capacity in a rebuild hands back x, v and also the
forces of the last full step, though it has enqueued steps past the rebuild by then:
bit for bit those of a run that ends there.
"""
import ctypes

import numpy as np
import pytest

from paper_1506_00716_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pme", [False, True])
@pytest.mark.parametrize("nstlist,n_steps", [(1, 3), (2, 7), (5, 5), (5, 6), (5, 16)])
def test_forces_of_the_last_full_step(nbmod, gpu_ctx, nstlist, n_steps, pme):
    import torch
    m = inputs.Model(r_cut=0.9, r_list=1.0, coulomb="ewald", ewald_beta=3.12,
                     pme_grid=(36, 36, 36) if pme else None)
    s = inputs.lattice_system(5832, 8.46, 58, m, True)
    print(f"[late capacity] forces: nstlist {nstlist} steps {n_steps} pme {pme}", flush=True)

    def run(n):
        # a list of the uniform lattice, then the atoms at 11 times its density
        g = nbmod.System(gpu_ctx, s)
        x = torch.tensor(s.x, dtype=torch.float64, device=gpu_ctx.device)
        g.build_pairlist(x)
        x.copy_(torch.tensor(0.45 * s.x, dtype=torch.float64, device=gpu_ctx.device))
        v = torch.tensor(s.v, dtype=torch.float64, device=gpu_ctx.device)
        f = torch.full((s.n, 3), 7.0, dtype=torch.float32, device=gpu_ctx.device)
        rows, n_rows = np.zeros((n_steps, 5)), ctypes.c_int32()
        code = nbmod.load().md_step(g.h, x.data_ptr(), v.data_ptr(), f.data_ptr(), 0.0002, n, nstlist, 1,
                                    rows.ctypes.data_as(ctypes.c_void_p), n_steps, ctypes.byref(n_rows))
        step = g.step
        g.close()
        return code, step, x, v, f, rows[:n_rows.value]

    code, step, x, v, f, rows = run(n_steps)
    assert code == nbmod.NB_ERR_CAPACITY and step == nstlist - 1
    code, _, xr, vr, fr, ref = run(nstlist - 1)
    assert code == nbmod.NB_OK
    assert np.array_equal(rows, ref)
    for a, b in ((x, xr), (v, vr), (f, fr)):
        assert torch.equal(a, b)
    assert float(f.abs().max()) > 0.0
