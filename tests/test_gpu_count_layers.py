"""Intercept counts through stacked sheets, each of them doubled or tripled:
around the number of hits that the first pass lists per segment (12 distinct t in
plain precision, 11 intervals in certified), against the number of sheets, the
binary tree's pass and the lane form.  Coincident triangles give one t: in plain
precision they take one place in the list, however many there are, so only
segments with more sheets than it holds go to the second pass."""
import numpy as np
import pytest

import paper_2305_01867_amd as rsi
from paper_2305_01867_amd import workloads
from gpu_helpers import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("copies", [1, 2, 3])
@pytest.mark.parametrize("layers", [1, 4, 11, 12, 13, 30])
def test_counts_through_stacked_sheets(layers, copies):
    V, F = workloads.heightfield(20, 3)
    Vs = [V + np.float32([0, 0, 2 * k]) for k in range(layers)] * copies
    Fs = [F + np.int32(k * len(V)) for k in range(layers * copies)]
    dV, dF = dev(np.concatenate(Vs)), dev(np.concatenate(Fs).astype(np.int32))
    rng = np.random.default_rng(layers)
    n = 5001
    # steep segments strictly inside the sheets' outline, through all of them
    O = rng.uniform(0.2, 0.8, (n, 3)).astype(np.float32)
    E = (O + rng.uniform(-0.02, 0.02, (n, 3))).astype(np.float32)
    O[:, 2], E[:, 2] = -1.5, 2 * layers - 0.5
    dO, dE = dev(O), dev(E)
    with rsi.rsi_build(dV, dF) as mesh:
        for precision in ("certified", "plain"):
            r = rsi.rsi_intersect(mesh, dO, dE, mode="intercept_count", precision=precision)
            got = host(r["count"])
            for other in (dict(node_width=2), dict(stack_depth=20)):
                want = rsi.rsi_intersect(mesh, dO, dE, mode="intercept_count", precision=precision, **other)
                assert np.array_equal(got, host(want["count"])), (precision, other)
            if precision == "certified" or layers <= 4:
                # (a steep segment may meet a sheet of noise in three places)
                assert np.all(got >= layers) and np.mean(got == layers) > 0.9, precision
            past = int(host(r["counters"])[3])
            if precision == "plain":
                assert past == int(np.sum(got > 12)), (past, int(np.sum(got > 12)))
            elif copies == 1:
                assert past <= int(np.sum(got > 11))
