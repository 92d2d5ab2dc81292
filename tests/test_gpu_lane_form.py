"""The first pass with a lane per segment over 4-wide nodes, which large calls take
and a stack depth asks for: the calls that other tests make with the library's own
launch shape are small and take the pool form.  Flags staged per wave at every
alignment, meshes of every shape, batches in every order, replays of a captured
graph; and both forms around the number of segments at which the library changes
from one to the other, on meshes on both sides of the rule's size."""
import numpy as np
import pytest
import torch

import oracle
import paper_2305_01867_amd as rsi
from paper_2305_01867_amd import workloads
from gpu_helpers import dev, host, say
from test_gpu_batch import small_batch
from test_gpu_pool import KEYS, against_oracle, same
from test_gpu_stage import _slow_and_fast
from test_gpu_wide import mesh_case

pytestmark = pytest.mark.gpu
LANE = dict(stack_depth=20)  # the library's own shape, by name


@pytest.mark.parametrize("precision", ["certified", "plain"])
def test_staged_boolean_writes(precision):
    V, F = workloads.heightfield(80, 9)
    O, E = _slow_and_fast(200_000, 3)
    hit, _, _, _ = oracle.intersect(V, F, O, E)
    with rsi.rsi_build(dev(V), dev(F), algorithm="restructured") as mesh:
        for n in (1, 255, 256, 257, 4095, 70_001, 200_000):
            for offset in (0, 1, 4, 7):
                for shape in (LANE, dict(LANE, block=64, waves_per_cu=1)):  # (long ranges: windows written early)
                    buf = torch.full((n + 16,), 9, dtype=torch.uint8, device="cuda")
                    rsi.rsi_intersect(mesh, dev(O[:n]), dev(E[:n]), mode="boolean", precision=precision,
                                      out={"hit": buf[offset:offset + n]}, **shape)
                    b = host(buf)
                    assert np.array_equal(b[offset:offset + n], hit[:n]), (n, offset, shape)
                    assert np.all(b[:offset] == 9) and np.all(b[offset + n:] == 9), (n, offset, shape)


@pytest.mark.parametrize("case", ["scene", "soup2", "soup3", "soup1025", "soup2049", "duplicates", "hf128"])
@pytest.mark.parametrize("algorithm", ["radix_tree", "restructured"])
def test_every_mode_on_every_mesh(case, algorithm):
    V, F = mesh_case(case)
    O, E = workloads.rays_in_box(6000, 4, V.min(0), V.max(0))
    O[0, 1], E[1, 2] = np.nan, np.inf
    O[2] = E[2] = V[F[0, 0]]
    O[3], E[3] = V[F[0, 0]] - np.float32(0.25), V[F[0, 0]] + np.float32(0.25)  # through a vertex
    hit, ids, uvt, _ = oracle.intersect(V, F, O, E)
    count = oracle.intercept_count(V, F, O, E)
    dO, dE = dev(O), dev(E)
    with rsi.rsi_build(dev(V), dev(F), algorithm=algorithm) as mesh:
        for mode in KEYS:
            for order in ("input", "origin_octant"):
                r = rsi.rsi_intersect(mesh, dO, dE, mode=mode, precision="certified", ray_sort=order, **LANE)
                against_oracle(r, mode, hit, ids, uvt, count)
            same(rsi.rsi_intersect(mesh, dO, dE, mode=mode, precision="plain", **LANE),
                 rsi.rsi_intersect(mesh, dO, dE, mode=mode, precision="plain", node_width=2), mode)


def test_batches_in_every_order_and_from_a_graph():
    parts, V, F, O, E, vo, to, ro = small_batch()
    dV, dF, dO, dE = dev(V), dev(F), dev(O), dev(E)
    with rsi.rsi_batch_create(vo, to, ro) as b:
        rsi.rsi_batch_build(b, dV, dF)
        for mode in KEYS:
            for order in ("input", "midpoint", "origin_octant"):
                r = rsi.rsi_batch_intersect(b, dO, dE, mode=mode, precision="certified", ray_sort=order, **LANE)
                for m, (Vm, Fm, Om, Em) in enumerate(parts):
                    part = {k: r[k][ro[m]:ro[m + 1]] for k in KEYS[mode]}
                    if len(Om) and len(Fm):
                        hit, ids, uvt, _ = oracle.intersect(Vm, Fm, Om, Em)
                        against_oracle(part, mode, hit, ids, uvt, oracle.intercept_count(Vm, Fm, Om, Em))
        out = {"tri_id": torch.empty(O.shape[0], dtype=torch.int32, device="cuda"),
               "uvt": torch.empty((O.shape[0], 3), dtype=torch.float32, device="cuda"),
               "counters": torch.zeros(4, dtype=torch.int64, device="cuda")}
        call = lambda: rsi.rsi_batch_intersect(b, dO, dE, mode="barycentric", precision="certified", out=out, **LANE)
        call()
        want = {k: host(out[k]).copy() for k in ("tri_id", "uvt")}
        g, s = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(s):
            with torch.cuda.graph(g, stream=s, capture_error_mode="thread_local"):
                rsi.rsi_batch_build(b, dV, dF)
                call()
        torch.cuda.current_stream().wait_stream(s)
        for rep in range(4):
            out["tri_id"].fill_(-7)
            out["uvt"].fill_(5.0)
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            for k in want:
                assert np.array_equal(host(out[k]), want[k], equal_nan=True), (rep, k)
            rsi.rsi_batch_intersect(b, dO, dE, mode="boolean", **LANE)  # eager work between replays
            torch.cuda.synchronize()


# 65,522 and 66,248 triangles: below and above the size up to which the pool form
# takes twice the resident lanes
@pytest.mark.parametrize("grid,lanes", [(182, 2), (183, 1)])
@pytest.mark.parametrize("over", [0, 1])
def test_both_sides_of_the_switch(grid, lanes, over):
    V, F = workloads.heightfield(grid, 6)
    assert (len(F) <= 65536) == (lanes == 2)
    n = lanes * torch.cuda.get_device_properties(0).multi_processor_count * 1024 + over
    O, E = workloads.rays_in_box(n, 61, V.min(0), V.max(0))
    dO, dE = dev(O), dev(E)
    with rsi.rsi_build(dev(V), dev(F), algorithm="restructured") as mesh:
        for mode in KEYS:
            for precision in ("certified", "plain"):
                want = rsi.rsi_intersect(mesh, dO, dE, mode=mode, precision=precision, node_width=2)
                same(rsi.rsi_intersect(mesh, dO, dE, mode=mode, precision=precision), want, mode)
                same(rsi.rsi_intersect(mesh, dO, dE, mode=mode, precision=precision, **LANE), want, mode)
    say(f"  {len(F)} triangles, {n} segments: both forms equal the binary first pass")


@pytest.mark.parametrize("grid", [4096, 4097, 5793, 5794])
def test_pool_form_around_4_gb_and_its_largest_mesh(grid):
    """Pool form with nodes just below and just above 4 GB (33,538,050 and
    33,554,432 triangles), with 67,094,528 triangles, whose references nearly fill
    the 26 bits of a pool entry, and with 67,117,698, where the library takes the
    lane form; without and with the tree's top in LDS."""
    limit = (1 << 26) - 512
    assert (2 * (grid - 1) ** 2 <= limit) == (grid <= 5793)
    gen = torch.Generator("cuda").manual_seed(grid)
    g = torch.linspace(0.0, 1.0, grid, device="cuda")
    y, x = torch.meshgrid(g, g, indexing="ij")
    z = 0.2 * torch.sin(9.0 * x) * torch.cos(7.0 * y) + 1e-4 * torch.rand(grid, grid, generator=gen, device="cuda")
    V = torch.stack([x, y, z], 2).reshape(-1, 3).contiguous()
    i = torch.arange(grid - 1, device="cuda", dtype=torch.int32)
    v = (i[:, None] * grid + i[None, :]).reshape(-1)
    F = torch.stack([v, v + 1, v + grid + 1, v, v + grid + 1, v + grid], 1).reshape(-1, 3).contiguous()
    with rsi.rsi_build(V, F) as mesh:
        for n in (20_000, 60_000):
            O, E = (torch.rand(n, 3, generator=gen, device="cuda") * 1.2 - 0.1 for _ in range(2))
            O[:, 2] -= 0.5
            E[:, 2] -= 0.5
            for mode in KEYS:
                got = rsi.rsi_intersect(mesh, O, E, mode=mode, precision="certified")
                same(got, rsi.rsi_intersect(mesh, O, E, mode=mode, precision="certified", node_width=2), mode)
            assert int((got["count"] > 0).sum()) > n // 10
