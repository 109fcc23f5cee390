"""The partner search at the edge of one block's cache: 8192 pairs per scattering
DM (the most it holds, and in a box of 8192 gas particles the most there are) and
8193, where the DM are handed to the whole chip, up to 256 of them, and the rest
are searched by their own block without the cache.  Partners and kicks as in the
other parity tests: equal to the oracle's away from thresholds, kicks to 1e-12 in
binary64 and 2e-5 in binary32; a batched step equals the single ones bit for bit."""
import numpy as np
import pytest

import workloads
from parity_util import decision_report, kick_error, run_gpu

pytestmark = pytest.mark.gpu


def _cloud(orc, n_gas, n_dm):
    """Every DM reaches every gas particle; timesteps that put P_i near 0.95."""
    cfg = workloads.galaxy(n_gas=n_gas, n_dm=n_dm, seed=(7, n_gas))
    r = np.random.default_rng(n_gas)
    cfg["gas"]["pos"] = r.normal(0.0, 1.0, (n_gas, 3))
    cfg["dm"]["pos"] = r.normal(0.0, 1.0, (n_dm, 3))
    cfg["dm"]["h"] = np.full(n_dm, 25.0)
    cfg["params"]["sigma0_cm2"] = 1e-21
    unit = orc.step(cfg["gas"], dict(cfg["dm"], dt=np.ones(n_dm)), cfg["params"], gas_sel=np.arange(1))
    cfg["dm"]["dt"] = 0.95 / unit["p_sum"]
    return cfg


@pytest.mark.parametrize("n_gas,n_dm", [(8192, 40), (8193, 300)])
@pytest.mark.parametrize("sampling", [0, 1])
def test_resolve_cache_edge(n_gas, n_dm, sampling):
    import oracle
    import torch
    import paper_2603_24688_amd as dmb
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = dmb.Context(0)
    cfg = _cloud(oracle, n_gas, n_dm)
    cfg["params"]["dm_sampling"] = sampling
    small = _cloud(oracle, 700, 60)
    small["params"]["dm_sampling"] = sampling
    ref = oracle.step(cfg["gas"], cfg["dm"], cfg["params"], gas_sel=np.arange(1))
    for prec in (0, 1):
        gpu = run_gpu(ctx, cfg, prec)
        dec, ke = decision_report(gpu, ref), kick_error(gpu, ref)
        print(f"[resolve edge] n_gas={n_gas} n_dm={n_dm} sampling={sampling} precision={prec} {dec} kick {ke:.1e}", flush=True)
        assert dec["scatters"] > 0.8 * n_dm
        assert dec["mismatch"] == 0
        assert ke <= (1e-12 if prec == 0 else 2e-5)
        one = [gpu, run_gpu(ctx, small, prec)]
        boxes = [cfg, small]
        G, D = ([dmb.to_device(b[k]) for b in boxes] for k in ("gas", "dm"))
        P = [b["params"] for b in boxes]
        O = [dmb.alloc_out(len(b["gas"]["mass"]), len(b["dm"]["mass"])) for b in boxes]
        ctx.batch_build(G, D, P, precision=prec)
        ctx.batch_step(G, D, P, O, precision=prec)
        torch.cuda.synchronize()
        for o, s in zip(O, one):
            for k in ("dv_dm", "partner", "p_sum", "p_max", "dp_gas", "de_gas"):
                assert np.array_equal(o[k].cpu().numpy(), s[k]), k
            assert dmb.counters_dict(o["counters"]) == s["counters"]
    ctx.close()
