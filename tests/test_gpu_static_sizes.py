"""What dmb_step_static has room for at its largest particle counts: a galaxy whose kernels
are widened until its candidates fill the scratch, all particles active or only the
inner gas (few gas candidates, cut into many work items with their partial sums, beside
millions of DM candidates), and a uniform box with the finest items.  Each step is
accepted and gives the outputs of dmb_build_cells + dmb_interact_step bit for bit."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

N = 262144


@pytest.fixture(scope="module")
def galaxy():
    return workloads.galaxy(n_gas=N, n_dm=N, seed=(2, 19))


def _check(cfg, precision, scale, active=None):
    import torch
    import paper_2603_24688_amd as dmb
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    gas, dm = (dict(cfg[s], h=scale * cfg[s]["h"]) for s in ("gas", "dm"))
    if active is not None:
        r = np.linalg.norm(gas["pos"] - gas["pos"].mean(0), axis=1)
        gas["active"] = (r <= np.quantile(r, active)).astype(np.uint8)
    G, D, par = dmb.to_device(gas), dmb.to_device(dm), cfg["params"]
    a, b = dmb.alloc_out(N, N), dmb.alloc_out(N, N)
    ctx = dmb.Context(0)
    ctx.step_static(G, D, par, a, precision=precision)
    ctx.build_cells(G, D, par, precision=precision)
    ctx.interact_step(G, D, par, b, precision=precision)
    torch.cuda.synchronize()
    st = ctx.build_stats()
    ctx.close()
    print(f"[static sizes] precision {precision} h x {scale} active {active} {st}", flush=True)
    for k in a:
        assert torch.equal(a[k], b[k]), k
    assert int(a["counters"][0]) > 0
    return st


@pytest.mark.parametrize("precision,scale,active", [(0, 1.34, None), (1, 1.405, None), (0, 1.6, 0.2), (1, 1.66, 0.2),
                                                    (0, 1.66, 0.05), (1, 1.72, 0.05)])
def test_wide_kernels(galaxy, precision, scale, active):
    _check(galaxy, precision, scale, active)


@pytest.mark.parametrize("precision", [0, 1])
def test_finest_items(precision):
    cfg = workloads.box(n_gas=N, n_dm=N, seed=(19, 7), sigma0_cm2=3e-22, h_mode="density", n_ngb=8)
    st = _check(cfg, precision, 1.5)
    assert 300000 < st["cand_pairs_gas"] < 524288 and st["items_gas"] > 30000
