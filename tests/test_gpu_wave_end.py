"""Segments that outgrow their lane's stack wait for the wave's end and share a
pool in the wave's stack memory there: more of them than that pool has room for,
and than a wave puts off (64), against the oracle in every mode, with flags at
aligned and unaligned addresses and in the proposal order.  Counter 1 names each
such segment once, whichever pass settles it."""
import os

import numpy as np
import pytest
import torch

import oracle
import paper_2305_01867_amd as rsi
from gpu_helpers import dev, host, say

pytestmark = pytest.mark.gpu

SHAPE = dict(block=64, waves_per_cu=1)  # few waves, so that each has many such segments


def _slivers(k, seed):
    """k needles across the unit cube: every box holds nearly all of it, so a
    segment that hits nothing visits the whole tree."""
    rng = np.random.default_rng(seed)
    e = rng.uniform(-1e-3, 1e-3, (k, 3, 3))
    V = np.concatenate([e[:, :1], e[:, 1:2] + 1.0, e[:, 2:] + 0.5], 1).reshape(-1, 3).astype(np.float32)
    return V, np.arange(3 * k, dtype=np.int32).reshape(-1, 3)


@pytest.mark.parametrize("depth", [11, 12])
@pytest.mark.parametrize("nodes", [None, "1"])
@pytest.mark.parametrize("proposal", [False, True])
def test_segments_that_outgrow_their_stack(depth, nodes, proposal, monkeypatch):
    V, F = _slivers(3000, 5)
    rng = np.random.default_rng(6)
    n = 4 * 64 * torch.cuda.get_device_properties(0).multi_processor_count // 3 + 1  # 85 a wave
    O, E = (rng.uniform(0.0, 1.0, (n, 3)).astype(np.float32) for _ in range(2))
    hit, ids, uvt, _ = oracle.intersect(V, F, O, E)
    dO, dE = dev(O), dev(E)
    with rsi.rsi_build(dev(V), dev(F), algorithm="restructured") as mesh:
        if proposal:
            rsi.rsi_proposal_train(mesh, dO, dE, epochs=1, batch=64)
        if nodes:
            monkeypatch.setenv("RSI_DEBUG_POOL_NODES", nodes)
        opts = dict(SHAPE, stack_depth=depth, proposal=proposal)
        for precision in ("certified", "plain"):
            for offset in (0, 1):
                buf = torch.full((n + 8,), 9, dtype=torch.uint8, device="cuda")
                r = rsi.rsi_intersect(mesh, dO, dE, mode="boolean", precision=precision,
                                      out={"hit": buf[offset:offset + n]}, **opts)
                b = host(buf)
                if precision == "certified":
                    assert np.array_equal(b[offset:offset + n], hit), offset
                assert np.all(b[:offset] == 9) and np.all(b[offset + n:] == 9), offset
                outgrew = int(host(r["counters"])[1])
                assert n // 2 < outgrew <= n, outgrew  # (a segment once; 0.4% of them hit something)
        for mode in ("first_hit", "barycentric"):
            r = rsi.rsi_intersect(mesh, dO, dE, mode=mode, precision="certified", **opts)
            assert np.array_equal(host(r["tri_id"]), ids), mode
            if mode == "barycentric":
                got, want = host(r["uvt"]).view(np.uint32), uvt.astype(np.float32).view(np.uint32)
                assert np.array_equal(got[ids >= 0], want[ids >= 0])
            outgrew = int(host(r["counters"])[1])
            assert n // 2 < outgrew <= n, (mode, outgrew)
    say(f"  depth {depth}, pool of {nodes or 'the wave'}, proposal {proposal}: {outgrew} of {n} outgrew their stack")
