"""Which workgroup computes which owner tile: batch order (many short sequences), ranking in registers (up to 64
sequences) and by histogram (more), over both owner tile heights of the d = 64 forward pass and both passes of the
joint backward launch.  Every output is NaN-poisoned before the call, so a tile that no workgroup took shows;
tolerances are those of the parity tests."""
import numpy as np
import pytest

from paper_2604_27124_amd import workloads as W
from gpu_util import Dev, check_against_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,N,H,d", [
    (64, 300, 4, 64),      # batch order: runs of a multiple of 8 ids per sequence, three 128-row tiles
    (70, 257, 3, 64),      # batch order: ids per sequence not a multiple of 8, one row in the last tile
    (90, 100, 5, 64),      # batch order, one tile per head
    (33, 513, 8, 128),     # batch order at d = 128
    (64, 130, 1, 64),      # ranked in registers, every lane in use
    (65, 300, 1, 64),      # ranked by histogram
    (65, 250, 2, 128),     # ranked by histogram, d = 128
    (44, 257, 3, 64),      # forward: 264 workgroups of 256 rows (two owner blocks a wave), ranked in registers
    (42, 257, 3, 64),      # forward: 252 of them, so 128-row tiles
])
def test_every_tile_is_taken_once(B, N, H, d):
    rng = np.random.default_rng(B * N + H)
    lens = rng.integers(0, N + 1, size=B)
    edges = [v for v in (0, 1, 127, 128, 129, 255, 256, 257, N) if v <= N]
    lens[:len(edges)] = edges
    w = W.make(B, N, H, d, lens, seed=B + N)
    slices = [(z, (z + k) % H) for z in list(range(len(edges))) + [B // 2, B - 1] for k in range(min(H, 2))]
    dev = Dev(w)
    print("mapping", (B, N, H, d), check_against_oracle(w, slices=slices, dev=dev), flush=True)
    for t in [dev.fwd()] + list(dev.bwd()):
        got = t.float()
        assert bool(got.isfinite().all())
        nonzero = (got != 0).any(dim=3).any(dim=2).cpu().numpy()        # [B, N]; a valid row is never all zero
        assert np.array_equal(nonzero, np.arange(N)[None, :] < lens[:, None])
