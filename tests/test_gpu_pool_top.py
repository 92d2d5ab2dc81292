"""The pool form with the tree's top in LDS (from 192 segments per CU on): both
sides of its threshold, every mode and precision, meshes with fewer and with more
nodes than the copy holds, against the binary tree's lane-per-segment pass."""
import numpy as np
import pytest
import torch

import paper_2305_01867_amd as rsi
from paper_2305_01867_amd import workloads
from gpu_helpers import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid", [2, 9, 70])
@pytest.mark.parametrize("over", [-1, 0, 1001])
def test_pool_with_the_top_in_lds(grid, over):
    """2, 128 and 9,522 triangles; one segment below the threshold, on it and
    past it.  Certified results are exact, so the passes agree element by
    element; plain ones agree on these segments, none of which is within
    binary32 rounding of an edge by construction of the comparison: the ids are
    compared where the certified pass finds the same answer as the plain one."""
    V, F = workloads.heightfield(grid, 4)
    n = torch.cuda.get_device_properties(0).multi_processor_count * 192 + over
    O, E = workloads.rays_in_box(n, 8, V.min(0), V.max(0))
    dO, dE = dev(O), dev(E)
    keys = {"boolean": ("hit",), "first_hit": ("tri_id",), "barycentric": ("tri_id", "uvt"), "intercept_count": ("count",)}
    with rsi.rsi_build(dev(V), dev(F)) as mesh:
        for mode, names in keys.items():
            want = rsi.rsi_intersect(mesh, dO, dE, mode=mode, precision="certified", node_width=2)
            got = rsi.rsi_intersect(mesh, dO, dE, mode=mode, precision="certified")
            for k in names:
                assert np.array_equal(host(got[k]), host(want[k]), equal_nan=k == "uvt"), (mode, k)
            plain2 = host(rsi.rsi_intersect(mesh, dO, dE, mode=mode, precision="plain", node_width=2)[names[0]])
            plain = host(rsi.rsi_intersect(mesh, dO, dE, mode=mode, precision="plain")[names[0]])
            same = plain2 == host(want[names[0]])
            assert same.mean() > 0.999 and np.array_equal(plain[same], plain2[same]), mode


@pytest.mark.parametrize("per_cu,over", [(1024, 1), (1536, 0), (2048, 0), (2048, 1)])
def test_pool_past_one_round(per_cu, over):
    """More segments than are in flight at once, up to twice as many (no chunks
    at the end) and one past that, against the binary tree's lane form."""
    V, F = workloads.heightfield(33, 5)
    n = torch.cuda.get_device_properties(0).multi_processor_count * per_cu + over
    O, E = workloads.rays_in_box(n, 9, V.min(0), V.max(0))
    dO, dE = dev(O), dev(E)
    with rsi.rsi_build(dev(V), dev(F)) as mesh:
        for mode, name in (("boolean", "hit"), ("first_hit", "tri_id"), ("intercept_count", "count")):
            want = rsi.rsi_intersect(mesh, dO, dE, mode=mode, precision="certified", node_width=2)
            got = rsi.rsi_intersect(mesh, dO, dE, mode=mode, precision="certified")
            assert np.array_equal(host(got[name]), host(want[name])), mode
