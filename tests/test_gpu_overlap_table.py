"""The overlap table of the binary32 steps, word for word, at recorded lookups.

The table's binary32 coefficients are differences of nodes and carry the nodes'
rounding: another rule for the nodes, exact to rounding as well, moves a fifth of
them, by up to 1e-8 of the overlap, and with them a rare pair of every binary32
step by one or two units in the last place.  dmb_overlap_eval (DMB_FP32) looks the
table up; the recorded places, found among 8e8, are those where such a move passes a
rounding boundary of the looked-up value, so each value has to be the recorded one
bit for bit."""
import json
import os

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(__file__), "golden", "overlap_table_points.json")


def test_overlap_table_points():
    import torch
    import paper_2603_24688_amd as dmb
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    with open(GOLDEN) as f:
        rows = np.array([[float.fromhex(v) for v in r] for r in json.load(f)["points"]])
    T = [torch.from_numpy(np.ascontiguousarray(rows[:, k])).cuda() for k in range(3)]
    ctx = dmb.Context(0)
    got = ctx.overlap_eval(*T, precision=dmb.DMB_FP32).cpu().numpy()
    ctx.close()
    moved = int(np.sum(got != rows[:, 3]))
    print(f"[overlap table] {moved} of {len(rows)} recorded lookups moved, by up to "
          f"{np.max(np.abs(got / rows[:, 3] - 1.0)):.1e}", flush=True)
    assert moved == 0
