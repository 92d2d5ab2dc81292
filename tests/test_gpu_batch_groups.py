"""The batched lane form's item groups (equal cost, meshes cut across them):
one mesh in every group, a few, and 64 uneven ones with an empty mesh and a mesh
without segments among them, against each mesh built and asked by itself."""
import numpy as np
import pytest
import torch

import paper_2305_01867_amd as rsi
from paper_2305_01867_amd import workloads
from gpu_helpers import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grids,rays", [
    ([40], [530_001]),
    ([70, 3, 25], [500_000, 40_001, 63]),
    ([6 + (7 * k) % 45 for k in range(62)] + [0, 30], [200 + (9973 * k * k) % 17_777 for k in range(62)] + [5, 0]),
])
def test_groups_of_equal_cost(grids, rays):
    Vs, Fs, Os, Es = [], [], [], []
    for k, (g, m) in enumerate(zip(grids, rays)):
        V, F = workloads.heightfield(g, 100 + k) if g else (np.zeros((0, 3), np.float32), np.zeros((0, 3), np.int32))
        box = (V.min(0), V.max(0)) if g else (np.zeros(3), np.ones(3))
        O, E = workloads.rays_in_box(m, 200 + k, *box) if m else (np.zeros((0, 3), np.float32),) * 2
        Vs.append(V), Fs.append(F), Os.append(O), Es.append(E)
    assert sum(rays) > 2 * 262_144  # past the pool form
    offs = [np.concatenate([[0], np.cumsum([len(x) for x in xs])]).astype(np.int64) for xs in (Vs, Fs, Os)]
    cat = lambda xs: dev(np.concatenate(xs))  # noqa: E731
    batch = rsi.rsi_batch_create(*offs)
    rsi.rsi_batch_build(batch, cat(Vs), cat(Fs))
    for mode, name in (("boolean", "hit"), ("first_hit", "tri_id")):
        got = host(rsi.rsi_batch_intersect(batch, cat(Os), cat(Es), mode=mode, precision="certified")[name])
        for k in range(len(grids)):
            mine = got[offs[2][k]:offs[2][k + 1]]
            if not len(Fs[k]):
                assert np.all(mine == (0 if mode == "boolean" else -1))
            elif len(mine):
                with rsi.rsi_build(dev(Vs[k]), dev(Fs[k])) as mesh:
                    want = host(rsi.rsi_intersect(mesh, dev(Os[k]), dev(Es[k]), mode=mode, precision="certified")[name])
                assert np.array_equal(mine, want), (mode, k)
    torch.cuda.synchronize()
