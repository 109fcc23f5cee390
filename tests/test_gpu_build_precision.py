"""A structure serves steps of both precisions: a step's outputs do not depend on the
precision that dmb_build_cells (or dmb_batch_build) was called with, bit for bit, in
problems small enough for the finest work items and larger ones."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

KEYS = ("dv_dm", "dp_gas", "de_gas", "partner", "p_sum", "p_max", "counters")


@pytest.mark.parametrize("n_gas,n_dm", [(1500, 1300), (3000, 12000), (30000, 120000)])
def test_step_is_independent_of_the_build_precision(n_gas, n_dm):
    import torch
    import paper_2603_24688_amd as dmb
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cfg = workloads.galaxy(n_gas=n_gas, n_dm=n_dm, seed=(3, n_gas))
    G, D, par = dmb.to_device(cfg["gas"]), dmb.to_device(cfg["dm"]), cfg["params"]
    ctx = dmb.Context(0)
    for prec in (0, 1):
        got = {}
        for built in (0, 1):
            single, batched = dmb.alloc_out(n_gas, n_dm), dmb.alloc_out(n_gas, n_dm)
            ctx.build_cells(G, D, par, precision=built)
            ctx.interact_step(G, D, par, single, precision=prec)
            ctx.batch_build([G], [D], [par], precision=built)
            ctx.batch_step([G], [D], [par], [batched], precision=prec)
            torch.cuda.synchronize()
            got[built] = [{k: o[k].cpu().numpy() for k in KEYS} for o in (single, batched)]
        for a, b in zip(got[0], got[1]):
            moved = {k: int(np.sum(a[k] != b[k])) for k in KEYS if not np.array_equal(a[k], b[k])}
            print(f"[build precision] {n_gas}+{n_dm} step precision {prec}: {moved}", flush=True)
            assert not moved
    ctx.close()
