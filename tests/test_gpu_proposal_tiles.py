"""The training pass at the edges of its tiles and row chunks: one row, one
short of / one past a 32-row tile, the last unsplit batch and the first split
one, and batches of up to 16 chunks of the shortest and of a longer length."""
import numpy as np
import pytest

from oracle import mlp_reference as ref
import paper_2305_01867_amd as rsi
from paper_2305_01867_amd import workloads
from gpu_helpers import dev, host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 31, 33, 256, 257])
def test_gradient_at_tile_and_chunk_edges(rows):
    """Gradient, loss and logits against the binary64 reference network.

    Both sides round activations and gradients to bf16 at the same points; the
    kernel accumulates in fp32, the reference in binary64, so a value within
    about 2^-20 of its size of a rounding boundary may land on the other bf16
    neighbour (2^-8 of its size): one in some thousand values.  One such value
    among a row's 256 moves that row's gradient by 2^-8 / 16 = 2.4e-4 of its
    norm, four of them by 1e-3, the bound taken (and fewer rows flip, on
    average over more rows).  ReLU masks that flip are not in this bound: with
    768 units a row and fp32 error 2^-20 there is none to expect below a
    thousand rows; larger batches are compared in the next test."""
    V, F = workloads.heightfield(24, 3)
    O, E = workloads.rays_in_box(rows, 5, V.min(0), V.max(0))
    with rsi.rsi_build(dev(V), dev(F)) as mesh:
        rng = np.random.default_rng(rows)
        P = np.concatenate([(rng.uniform(-1, 1, (o, i)) * np.sqrt(6.0 / i) *
                             (np.arange(i) < ref.FEAT if i == ref.INPUTS else 1.0)).ravel()
                            for o, i in ref.LAYER_SHAPES] + [rng.normal(0, 0.05, 4 * ref.HIDDEN)]).astype(np.float32)
        rsi.rsi_proposal_params(mesh, dev(P))
        nb = len(host(rsi.rsi_proposal_frontier(mesh)[0]))
        labels = rng.integers(0, nb, rows).astype(np.int32)
        grad, logits, loss = rsi.rsi_proposal_gradient(mesh, dev(O), dev(E), dev(labels))
        X0 = host(rsi.rsi_proposal_features(mesh, dev(O), dev(E)).float()).astype(np.float64)
    want_loss, want_logits, want_grad = ref.forward_backward(X0, labels, P.astype(np.float64), nb)
    norm = np.linalg.norm
    assert abs(float(host(loss)[0]) - want_loss) <= 1e-3 * abs(want_loss)
    assert norm(host(logits) - want_logits) <= 1e-3 * norm(want_logits)
    off = 0
    for size in [o * i for o, i in ref.LAYER_SHAPES] + [ref.HIDDEN] * 4:
        a, b = host(grad)[off:off + size].astype(np.float64), want_grad[off:off + size]
        off += size
        say(f"  {rows} rows: {size} parameters, relative error {norm(a - b) / norm(b):.2e}")
        assert norm(a - b) <= 1e-3 * norm(b)


@pytest.mark.parametrize("tiles", [8, 16, 128, 256])
def test_gradient_of_a_repeated_tile(tiles):
    """One 32-row tile repeated 8, 16, 128 and 256 times (one chunk, two, 16 of
    256 rows, 16 of 512): the mean gradient is the tile's own.

    The counts are powers of two, so 1 / rows scales every gradient exactly
    and only the order of the fp32 sums differs.  A chunk adds its tile sums T
    one after the other, at most 16 of them, then at most 16 chunks are added:
    each partial sum j T rounds by at most j T 2^-24, together 8.5 ulp of the
    sum for each of the two levels, and 32 more for the products within a tile;
    with sum |terms| at most 20 times the sum in norm, 2^-14 of it.  A tile
    left out or taken twice would be 2^-8."""
    V, F = workloads.heightfield(24, 3)
    O, E = workloads.rays_in_box(32, 6, V.min(0), V.max(0))
    with rsi.rsi_build(dev(V), dev(F)) as mesh:
        rng = np.random.default_rng(9)
        P = np.concatenate([(rng.uniform(-1, 1, (o, i)) * np.sqrt(6.0 / i) *
                             (np.arange(i) < ref.FEAT if i == ref.INPUTS else 1.0)).ravel()
                            for o, i in ref.LAYER_SHAPES] + [rng.normal(0, 0.05, 4 * ref.HIDDEN)]).astype(np.float32)
        rsi.rsi_proposal_params(mesh, dev(P))
        nb = len(host(rsi.rsi_proposal_frontier(mesh)[0]))
        labels = rng.integers(0, nb, 32).astype(np.int32)
        one, _, loss1 = rsi.rsi_proposal_gradient(mesh, dev(O), dev(E), dev(labels))
        many, _, loss = rsi.rsi_proposal_gradient(mesh, dev(np.tile(O, (tiles, 1))), dev(np.tile(E, (tiles, 1))),
                                                  dev(np.tile(labels, tiles)))
    a, b = host(many).astype(np.float64), host(one).astype(np.float64)
    off = 0
    for size in [o * i for o, i in ref.LAYER_SHAPES] + [ref.HIDDEN] * 4:
        x, y = a[off:off + size], b[off:off + size]
        off += size
        say(f"  {tiles} tiles: {size} parameters, relative difference {np.linalg.norm(x - y) / np.linalg.norm(y):.2e}")
        assert np.linalg.norm(x - y) <= 2.0 ** -14 * np.linalg.norm(y)
    assert abs(float(host(loss)[0]) - float(host(loss1)[0])) <= 2.0 ** -14 * float(host(loss1)[0])
