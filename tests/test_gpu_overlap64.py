"""The binary64 overlap on every order its breakpoints can take: a support that
starts at 0 or at delta - eta, ends at 1 or at delta + eta, with the small
kernel's centre on either side of 1/2, and separations so small that a piece is
only 2 delta wide (where the two ends of the inner integral lie on different
branches).  Oracle: its own 6-point rule; the bar is the conditioning both
rules share, 1e-12 + 16 x 1.11e-16 (1/nu + 1/eta) with nu = 1 - d/(h_b + h_s)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eta", [1.0, 0.9, 0.51, 0.5, 0.3, 0.04, 1e-3])
def test_overlap_orders(orc, eta):
    import torch
    import paper_2603_24688_amd as dmb
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    edges = [0.0, 0.5 * eta, eta, 0.5 - eta, 0.5 - 0.5 * eta, 0.5, 0.5 + 0.5 * eta, 0.5 + eta, 1.0 - eta,
             1.0 - 0.5 * eta, 1.0, 1.0 + 0.5 * eta, 1.0 + eta]
    delta = []
    for e in edges:
        for s in (1e-13, 1e-9, 1e-5, 1e-2):
            delta += [e - s, e + s]
    delta = np.array([x for x in sorted(set(delta)) if 0.0 < x < 1.0 + eta * (1.0 - 1e-7)])
    hb = 0.05 + 0.1 * (np.arange(len(delta)) % 11)
    hs = eta * hb
    d = delta * hb
    ref = np.array([orc.overlap(a, b, c) for a, b, c in zip(d, hb, hs)])
    ctx = dmb.Context(0)
    for h1, h2 in ((hb, hs), (hs, hb)):     # either argument may be the larger kernel
        T = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (d, h1, h2)]
        got = ctx.overlap_eval(*T, precision=dmb.DMB_FP64).cpu().numpy()
        bar = 1e-12 + 16 * 1.11e-16 * (1.0 / (1.0 - d / (hb + hs)) + 1.0 / eta)
        err = np.abs(got / ref - 1.0) / bar
        print(f"[overlap orders eta {eta}] {len(d)} separations, {err.max():.2f} of the bar", flush=True)
        assert np.all(ref > 0.0)
        assert err.max() < 1.0
    ctx.close()
