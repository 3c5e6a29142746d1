"""The backward pass of d = 64 in one pass over the scores: the path that sigmoid_attn_bwd takes on large batches of long
heads with a workspace.  dK and dV have to be the bits of the two-pass kernels (the same arithmetic); dQ, whose scores
round the scaled key where the two-pass kernel rounds the scaled query, is held to the oracle like theirs."""
import numpy as np
import pytest
import torch

from paper_2604_27124_amd import binding as A
from paper_2604_27124_amd import workloads as W
from gpu_util import BWD_TOL, Dev, check_against_oracle

pytestmark = pytest.mark.gpu

EDGES = (0, 1, 31, 32, 33, 63, 64, 65, 128, 129, 192, 255, 256, 257, 320, 511, 512, 513)
bits = lambda t: t.view(torch.int16)


def inputs(B, N, H, lens, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    q, k, v, g = (torch.empty(B, N, H, 64, dtype=torch.bfloat16, device="cuda").normal_(generator=gen) for _ in range(4))
    n = torch.from_numpy(np.asarray(lens, dtype=np.int32)).cuda()
    return q, k, v, g, n, torch.full((B,), -5.0, device="cuda")


def lengths(B, N, seed):
    lens = np.random.default_rng(seed).integers(0, N + 1, size=B)
    lens[:min(B, len(EDGES))] = EDGES[:B]
    lens[B - 1] = N
    return lens


@pytest.mark.parametrize("B,N,H", [
    (20, 1030, 8),       # ranked; one query row in the last of 17 tiles, 6 keys in the last of five
    (70, 1024, 3),       # more sequences than lanes, ranked
    (260, 650, 2),       # batch order, groups of sequences, the last one smaller
    (384, 449, 4),       # two tiles a head
    (5, 4100, 10),       # a few sequences a group, long chains
    (1, 16500, 12),      # more tiles of a head than lanes
])
def test_against_the_two_pass_kernels(B, N, H):
    args = inputs(B, N, H, lengths(B, N, B), seed=N)
    n = args[4]
    assert A.sigmoid_attn_bwd_onepass_workspace_bytes(B, N, H, 64) > 0
    seven = lambda: [torch.full_like(args[0], 7.0) for _ in range(3)]
    pad = (torch.arange(N, device="cuda")[None, :] >= n[:, None])[:, :, None, None]
    bad = [t.masked_fill(pad, x) for t, x in zip(args[:4], (float("nan"), float("inf"), float("-inf"), float("nan")))]
    first = A.sigmoid_attn_bwd(*args, 0.125, *seven())
    dk, dv = A.sigmoid_attn_bwd_dkdv(*args, 0.125)
    dq = A.sigmoid_attn_bwd_dq(*args, 0.125)
    assert torch.equal(bits(first[1]), bits(dk)) and torch.equal(bits(first[2]), bits(dv))
    worst = (first[0].float() - dq.float()).abs().amax(dim=(1, 3)) / dq.float().abs().amax(dim=(1, 3)).clamp_min(1e-30)
    print("dQ of one pass against two, worst slice", B, N, H, float(worst.max()), flush=True)
    assert float(worst.max()) <= BWD_TOL
    assert not bool((first[0] * pad).any())
    assert not torch.equal(bits(first[0]), bits(dq))                   # another kernel made it
    for inp in (args[:4], bad):                                        # same bits in every run, whatever the padding holds
        again = A.sigmoid_attn_bwd(*inp, *args[4:], 0.125, *seven())
        for x, y in zip(first, again):
            assert torch.equal(bits(x), bits(y))


def test_against_the_oracle():
    lens = lengths(20, 1030, 3)
    w = W.make(20, 1030, 8, 64, lens, seed=7)
    slices = [(z, (3 * z + k) % 8) for z in range(20) for k in range(2)]
    print("one pass", check_against_oracle(w, slices=slices, fwd=False), flush=True)


def test_infinite_inputs():
    """An Inf in a query or key row saturates its weights: the NaNs are those of the two-pass kernels, no others."""
    args = inputs(20, 1030, 8, lengths(20, 1030, 5), seed=8)
    for z, n in enumerate(args[4].tolist()):
        if n:
            args[0][z, n // 2, 0, z] = float("inf")
            args[1][z, n - 1, 1, 7] = float("-inf")
            args[3][z, n // 3, 2, 9] = float("inf")
    one = A.sigmoid_attn_bwd(*args, 0.125)
    two = (A.sigmoid_attn_bwd_dq(*args, 0.125), *A.sigmoid_attn_bwd_dkdv(*args, 0.125))
    for name, x, y in zip(("dQ", "dK", "dV"), one, two):
        assert torch.equal(x.isnan(), y.isnan()) and torch.equal(x.isinf(), y.isinf()), name
        x, y = (t.float().nan_to_num(0, 0, 0) for t in (x, y))
        top = y.abs().amax(dim=(1, 3)).clamp_min(1e-30)
        assert bool(((x - y).abs().amax(dim=(1, 3)) <= BWD_TOL * top).all()), name


def test_slices_of_a_batch():
    """More sums than the workspace may hold: the batch goes through it in slices."""
    B, N, H = 150, 2048, 16
    need = A.sigmoid_attn_bwd_onepass_workspace_bytes(B, N, H, 64)
    assert need <= 1 << 29 and need < A.sigmoid_attn_bwd_onepass_workspace_bytes(100, N, H, 64) * 1.5
    args = inputs(B, N, H, np.random.default_rng(1).integers(1, 400, size=B), seed=4)
    one = A.sigmoid_attn_bwd(*args, 0.125)
    dk, dv = A.sigmoid_attn_bwd_dkdv(*args, 0.125)
    dq = A.sigmoid_attn_bwd_dq(*args, 0.125)
    assert torch.equal(bits(one[1]), bits(dk)) and torch.equal(bits(one[2]), bits(dv))
    assert bool(((one[0].float() - dq.float()).abs().amax(dim=(1, 3)) <= BWD_TOL * dq.float().abs().amax(dim=(1, 3))).all())


def test_workspaces_and_streams():
    args = inputs(20, 1030, 8, lengths(20, 1030, 6), seed=9)
    need = A.sigmoid_attn_bwd_onepass_workspace_bytes(20, 1030, 8, 64)
    ref = A.sigmoid_attn_bwd(*args, 0.125)
    ws = torch.full((need,), 0x7f, dtype=torch.uint8, device="cuda")   # contents irrelevant on entry
    for x, y in zip(ref, A.sigmoid_attn_bwd(*args, 0.125, workspace=ws)):
        assert torch.equal(bits(x), bits(y))
    ws = torch.full((need + 64,), 0x7f, dtype=torch.uint8, device="cuda")
    for start in (16, 48):                                             # aligned to 16 bytes and no further
        for x, y in zip(ref, A.sigmoid_attn_bwd(*args, 0.125, workspace=ws[start:start + need])):
            assert torch.equal(bits(x), bits(y))
        assert bool((ws[:start] == 0x7f).all()) and bool((ws[start + need:] == 0x7f).all())
    ws = ws[:need]
    dq = A.sigmoid_attn_bwd(*args, 0.125, workspace=ws[:need - 1])[0]  # too small for one pass: two
    assert torch.equal(bits(dq), bits(A.sigmoid_attn_bwd_dq(*args, 0.125)))
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    outs = [[torch.empty_like(args[0]) for _ in range(3)] for _ in range(2)]
    for _ in range(3):                                                 # two streams at once, scratch of their own
        A.sigmoid_attn_bwd(*args, 0.125, *outs[0], stream=side)
        torch.empty(need, dtype=torch.uint8, device="cuda").fill_(0x55)
        A.sigmoid_attn_bwd(*args, 0.125, *outs[1])
    torch.cuda.synchronize()
    for got in outs:
        for x, y in zip(ref, got):
            assert torch.equal(bits(x), bits(y))


@pytest.mark.parametrize("B,N", [(40, 1030), (300, 1030), (40, 2100), (150, 1500)])     # ranked, batch order, other padding, slices
def test_a_sequence_has_the_same_bits_in_every_batch(B, N):
    """One pass: what surrounds a sequence (other sequences, padding, slices of the batch) reaches none of its bits."""
    base = inputs(20, 1030, 16, lengths(20, 1030, 9), seed=12)
    ref = A.sigmoid_attn_bwd(*base, 0.125)
    args = inputs(B, N, 16, lengths(B, N, 10), seed=13)
    at = [(7 * z + 3) % B for z in range(20)]
    for z, to in enumerate(at):
        for whole, part in zip(args[:4], base[:4]):
            whole[to, :1030] = part[z]
        args[4][to] = base[4][z]
    assert A.sigmoid_attn_bwd_onepass_workspace_bytes(B, N, 16, 64) > 0
    for one, many in zip(ref, A.sigmoid_attn_bwd(*args, 0.125)):
        for z, to in enumerate(at):
            assert torch.equal(bits(one[z]), bits(many[to, :1030])), z


def test_where_no_workspace_can_be_had(monkeypatch):
    """Without memory for it the call is the two-pass one, bit for bit, and so is one with an empty workspace."""
    args = inputs(20, 1030, 8, lengths(20, 1030, 4), seed=14)
    two = (A.sigmoid_attn_bwd_dq(*args, 0.125), *A.sigmoid_attn_bwd_dkdv(*args, 0.125))
    empty = A.sigmoid_attn_bwd(*args, 0.125, workspace=torch.empty(0, dtype=torch.uint8, device="cuda"))
    monkeypatch.setattr(A, "_fast", A._NoFastCalls)
    monkeypatch.setattr(A, "_scratch", lambda *a: None)
    for got in (empty, A.sigmoid_attn_bwd(*args, 0.125)):
        for x, y in zip(got, two):
            assert torch.equal(bits(x), bits(y))


def test_overlapping_launches_with_heads_across_xcds():
    """Two streams, heads whose key tiles lie on several XCDs (12 heads, 33 links of a chain): a tile waits only for one that has
    been started, so both end with the bits of a launch on its own."""
    args = inputs(3, 8448, 12, (8448, 8200, 7000), seed=11)
    ref = A.sigmoid_attn_bwd(*args, 0.125)
    outs = [[torch.empty_like(args[0]) for _ in range(3)] for _ in range(2)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    for _ in range(2):
        for side, out in zip(streams, outs):
            A.sigmoid_attn_bwd(*args, 0.125, *out, stream=side)
    torch.cuda.synchronize()
    for got in outs:
        for x, y in zip(ref, got):
            assert torch.equal(bits(x), bits(y))


def test_in_a_hip_graph():
    args = inputs(20, 1030, 8, lengths(20, 1030, 2), seed=3)
    eager = A.sigmoid_attn_bwd(*args, 0.125)
    outs = [torch.empty_like(args[0]) for _ in range(3)]
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        A.sigmoid_attn_bwd(*args, 0.125, *outs, stream=side)
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            A.sigmoid_attn_bwd(*args, 0.125, *outs, stream=torch.cuda.current_stream())
    torch.cuda.synchronize()
    for replay in range(3):
        for t in outs:
            t.fill_(float("nan"))
        A.sigmoid_attn_bwd(*args, 0.125)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for x, y in zip(outs, eager):
            assert torch.equal(bits(x), bits(y)), replay
