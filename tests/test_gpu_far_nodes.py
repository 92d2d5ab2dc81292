"""Nodes past 4 GB: the 4-wide pass reaches them by 64-bit addresses (below
that by 32-bit offsets from the tree's first node)."""
import numpy as np
import pytest
import torch

import paper_2305_01867_amd as rsi
from gpu_helpers import host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid", [4096, 4097])
def test_four_wide_nodes_around_4_gb(grid):
    """33,538,050 triangles: (triangles + 512) x 128 bytes just below 2^32;
    33,554,432: just above.  The 4-wide pass (a lane per segment: the caller's
    stack depth keeps it out of the pool form) against the binary one."""
    assert ((2 * (grid - 1) ** 2 + 512) * 128 > 2 ** 32 - 1) == (grid == 4097)
    gen = torch.Generator("cuda").manual_seed(grid)
    g = torch.linspace(0.0, 1.0, grid, device="cuda")
    y, x = torch.meshgrid(g, g, indexing="ij")
    z = 0.2 * torch.sin(9.0 * x) * torch.cos(7.0 * y) + 1e-4 * torch.rand(grid, grid, generator=gen, device="cuda")
    V = torch.stack([x, y, z], 2).reshape(-1, 3).contiguous()
    i = torch.arange(grid - 1, device="cuda")
    v = (i[:, None] * grid + i[None, :]).reshape(-1)
    F = torch.stack([torch.stack([v, v + 1, v + grid + 1], 1), torch.stack([v, v + grid + 1, v + grid], 1)], 1)
    F = F.reshape(-1, 3).int().contiguous()
    n = 20000
    O = torch.rand(n, 3, generator=gen, device="cuda") * 1.2 - 0.1
    E = torch.rand(n, 3, generator=gen, device="cuda") * 1.2 - 0.1
    O[:, 2] = O[:, 2] - 0.5
    E[:, 2] = E[:, 2] - 0.5
    with rsi.rsi_build(V, F) as mesh:
        assert rsi.rsi_mesh_info_get(mesh)["node_width"] == 4
        for mode, key in (("boolean", "hit"), ("first_hit", "tri_id")):
            wide = rsi.rsi_intersect(mesh, O, E, mode=mode, precision="certified", stack_depth=20, node_width=4)
            narrow = rsi.rsi_intersect(mesh, O, E, mode=mode, precision="certified", stack_depth=20, node_width=2)
            assert np.array_equal(host(wide[key]), host(narrow[key]))
        assert int((narrow["tri_id"] >= 0).sum()) > n // 10
