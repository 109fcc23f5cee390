"""Batches whose boxes differ as much as they can: one box of 20 000 gas particles among
boxes of a few, sizes at the edges of tiles and blocks, boxes without one species or
without a pair.  Every launch of the step covers the boxes' own blocks laid end to end.
Each box has to come out the same bit for bit wherever it stands among the boxes, and
as it does alone: scatters and counts bit for bit, binary64 sums, whose work items a batch
shares out, to 1e-12 of the largest (P_i of a binary32 step is a sum of binary32 groups
that follow the items, so it is left to the comparison of the two orders)."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (64, 64), (0, 300), (65, 257), (20000, 20000), (256, 63), (300, 0), (255, 256), (1, 700), (513, 1)]


def _box(k, n_gas, n_dm):
    cfg = workloads.box(n_gas=max(n_gas, 600), n_dm=max(n_dm, 600), seed=(41, k), sigma0_cm2=3e-21, h_mode="density",
                        n_ngb=8)
    for s, n in (("gas", n_gas), ("dm", n_dm)):
        cfg[s] = {a: (v if v is None else np.ascontiguousarray(v[:n])) for a, v in cfg[s].items()}
    if (n_gas, n_dm) == (1, 1):       # apart: no candidates at all
        L = np.asarray(cfg["params"]["box"])
        cfg["gas"]["pos"][0], cfg["dm"]["pos"][0] = 0.1 * L, 0.6 * L
        cfg["gas"]["h"][0] = cfg["dm"]["h"][0] = 0.01 * L[0]
    return cfg


@pytest.mark.parametrize("precision,rates,sampling", [(0, 0, 0), (1, 0, 1), (1, 3, 0)])
def test_uneven_boxes(precision, rates, sampling):
    import torch
    import paper_2603_24688_amd as dmb
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    boxes = [_box(k, *n) for k, n in enumerate(SIZES)]
    G, D = ([dmb.to_device(b[k]) for b in boxes] for k in ("gas", "dm"))
    P = [dict(b["params"], rates=rates, dm_sampling=sampling) for b in boxes]

    def outs():
        o = [dmb.alloc_out(*n) for n in SIZES]
        for x in o:
            for v in x.values():
                v.fill_(7)     # stale values must be overwritten
        return o

    one, many, replayed, turned = outs(), outs(), outs(), outs()
    ctx = dmb.Context(0)
    for k in range(len(boxes)):
        ctx.build_cells(G[k], D[k], P[k], precision=precision)
        ctx.interact_step(G[k], D[k], P[k], one[k], precision=precision)
    ctx.batch_build(G, D, P, precision=precision)
    ctx.batch_step(G, D, P, many, precision=precision)
    ctx.batch_step(G, D, P, replayed, precision=precision, nsteps=1, graph=True)
    back = [x[::-1] for x in (G, D, P, turned)]
    ctx.batch_build(*back[:3], precision=precision)
    ctx.batch_step(*back, precision=precision)
    torch.cuda.synchronize()
    ctx.close()
    for k, n in enumerate(SIZES):
        a, b, c, d = ({q: v.cpu().numpy() for q, v in o[k].items()} for o in (one, many, replayed, turned))
        print(f"[uneven p={precision} rates={rates} sampling={sampling}] box {k} {n} counters {b['counters'].tolist()}", flush=True)
        for q in a:
            assert np.array_equal(b[q], c[q]) and np.array_equal(b[q], d[q]), (k, q)
        for q in ("partner", "dv_dm", "p_max", "counters"):
            assert np.array_equal(a[q], b[q]), (k, q)
        for q in ("dp_gas", "de_gas", "p_sum")[:3 if precision == 0 else 2]:
            scale = np.max(np.abs(a[q]), initial=0.0)
            assert np.max(np.abs(a[q] - b[q]), initial=0.0) <= 1e-12 * scale, (k, q)
    assert int(many[4]["counters"][2]) > 0
