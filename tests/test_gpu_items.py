"""Work items of the two passes over the range of their cuts: pieces of one to 64
candidate sub-tiles, and (DM pass) four, three, two and one slices of a piece.
Sampled owners against the oracle with the bars of the other parity tests (1e-12
in binary64; 1e-5 for the gas and 2e-5 for P_i in binary32)."""
import numpy as np
import pytest

import workloads
from parity_util import decision_report, mean_field_error, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_gas,n_dm", [(65, 130), (3000, 12000), (30000, 120000), (36000, 150000), (70000, 290000)])
def test_item_cuts(n_gas, n_dm):
    import oracle
    import torch
    import paper_2603_24688_amd as dmb
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = dmb.Context(0)
    cfg = workloads.galaxy(n_gas=n_gas, n_dm=n_dm, seed=(3, n_gas))
    r = np.random.default_rng(n_gas)
    gsel = np.sort(r.choice(n_gas, min(n_gas, 150), replace=False))
    dsel = np.sort(r.choice(n_dm, min(n_dm, 150), replace=False))
    ref = oracle.step(cfg["gas"], cfg["dm"], cfg["params"], gas_sel=gsel, dm_sel=dsel)
    for prec in (0, 1):
        gpu = run_gpu(ctx, cfg, prec)
        st = ctx.build_stats()
        ep, ee = mean_field_error(gpu, ref, gsel)
        ps = ref["p_sum"][dsel]
        pe = np.max(np.abs(gpu["p_sum"][dsel] - ps) / np.maximum(ps, 1e-9))
        dec = decision_report(gpu, ref, dsel)
        print(f"[items] {n_gas}+{n_dm} precision={prec} dp {ep:.1e} dE {ee:.1e} P {pe:.1e} {dec['mismatch']} of "
              f"{dec['compared']} items {st['items_gas']} {st['items_dm']} of {st['cand_pairs_gas']} {st['cand_pairs_dm']}",
              flush=True)
        assert max(ep, ee) <= (1e-12 if prec == 0 else 1e-5)
        assert pe <= (1e-12 if prec == 0 else 2e-5)
        assert dec["mismatch"] == 0
        assert gpu["counters"]["pairs_gas"] == gpu["counters"]["pairs_dm"]
    ctx.close()
