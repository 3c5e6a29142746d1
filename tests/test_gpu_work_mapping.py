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
    (33, 513, 8, 128),     # d = 128: dK/dV in batch order, forward and dQ ranked in registers
    (48, 513, 8, 128),     # batch order at d = 128
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


@pytest.mark.parametrize("B,Lq,Lk,H,d", [
    (400, 257, 257, 4, 64),      # several owner tiles a workgroup in every launch, three or two tiles a head
    (300, 100, 100, 12, 64),     # one tile a head: workgroups go on with the next head
    (240, 300, 300, 4, 128),     # d = 128, 128- and 256-row owner tiles
    (200, 130, 700, 8, 64),      # cross-attention: more key tiles than query tiles (forward: one tile a workgroup)
    (40, 4096, 4096, 16, 64),    # long sequences: two tiles a workgroup in the backward pass
    (2, 130, 130, 16384, 64),    # more owner tiles per sequence than workgroups are dealt to one
])
def test_workgroups_of_several_tiles(B, Lq, Lk, H, d):
    """The joint calls of a large batch against calls on single sequences (or, for one long list of heads, on a part of
    them), where every workgroup has one tile: the same arithmetic, so the same bits.  The first sequences hold an Inf
    or NaN: it may not reach the tiles of another sequence or head."""
    import torch
    from paper_2604_27124_amd import binding as A
    gen = torch.Generator(device="cuda").manual_seed(B + H)
    normal = lambda n: torch.empty(B, n, H, d, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    q, k, v, g = normal(Lq), normal(Lk), normal(Lk), normal(Lq)
    rng = np.random.default_rng(B + d)
    nq, nk = rng.integers(0, Lq + 1, size=B), rng.integers(0, Lk + 1, size=B)
    if B > 2:
        edges = (0, 1, 127, 128, 129, 255, 256, 257)
        nq[:8], nk[4:12] = np.minimum(edges, Lq), np.minimum(edges, Lk)
        if Lq > 1000:                                            # all edges on both sides, and a few full tiles more
            nq[8:16] = (511, 512, 513, 768, 769, Lq - 1, Lq, 1024)
        v[1, 0, 1, 3], k[3, 0, 0, 5], g[6, 0, 2, 1] = float("inf"), float("nan"), float("-inf")
    else:
        nq[:], nk[:] = (130, 70), (130, 70)
        v[0, 5, 7, 3] = float("inf")
    if Lq == Lk:
        nk = nq
    dev = lambda a: torch.from_numpy(a.astype(np.int32)).cuda()
    nq, nk, bias = dev(nq), dev(nk), torch.full((B,), -5.0, device="cuda")
    scale = d ** -0.5

    def calls(q, k, v, g, nq, nk, bias):
        poison = lambda t: torch.full_like(t, 7.0)
        o = A.sigmoid_attn_cross_fwd(q, k, v, nq, nk, bias, scale, out=poison(q))
        grads = A.sigmoid_attn_cross_bwd(q, k, v, g, nq, nk, bias, scale, dq=poison(q), dk=poison(k), dv=poison(v))
        dq, db = A.sigmoid_attn_cross_bwd_dq_dbias(q, k, v, g, nq, nk, bias, scale, dq=poison(q))
        return (o, *grads, dq), db

    bits = lambda t: t.view(torch.int16)
    whole, db = calls(q, k, v, g, nq, nk, bias)
    if B == 2:
        for h0 in (0, 7, 8190, 16376):
            part, _ = calls(*(t[:, :, h0:h0 + 8].contiguous() for t in (q, k, v, g)), nq, nk, bias)
            for got, want in zip(whole, part):
                assert torch.equal(bits(got[:, :, h0:h0 + 8].contiguous()), bits(want)), (h0, "heads")
        for got in whole:       # heads that were not compared: every row written, zeros exactly in the padding
            nonzero = (got != 0).any(dim=3)
            assert bool(nonzero[0, :130].all()) and bool(nonzero[1, :70].all()) and not bool(nonzero[1, 70:].any())
        return
    for z in list(range(16)) + list(range(16, B, 7)) + [B - 1]:
        part, db1 = calls(*(t[z:z + 1] for t in (q, k, v, g, nq, nk, bias)))
        for i, (got, want) in enumerate(zip(whole, part)):
            assert torch.equal(bits(got[z:z + 1]), bits(want)), (z, i)
        assert torch.allclose(db[z:z + 1], db1, rtol=1e-4, atol=1e-4, equal_nan=True), z   # fp32 sums in another order


@pytest.mark.parametrize("B,Lk,d", [
    (300, 3000, 64),       # two passes of 256 threads over the sequences
    (520, 6000, 64),       # three passes
    (520, 6000, 128),      # two passes of 512 threads
])
def test_ranking_of_more_sequences_than_threads(B, Lk, d):
    """Few query rows against many keys, one head: the forward pass and dQ + dbias rank these batches (by histogram, the
    sequences of a class in several passes of the workgroup over the batch).  Against calls on single sequences, bit
    for bit; the outputs hold 7 before the call, so an owner tile that no workgroup took shows."""
    import torch
    from paper_2604_27124_amd import binding as A
    Lq = 100
    gen = torch.Generator(device="cuda").manual_seed(B + d)
    normal = lambda n: torch.empty(B, n, 1, d, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    q, k, v, g = normal(Lq), normal(Lk), normal(Lk), normal(Lq)
    rng = np.random.default_rng(B)
    nq, nk = rng.integers(0, Lq + 1, size=B), rng.integers(0, 200, size=B)
    nq[[0, 255, 256, 257, B - 1]] = (0, 1, 100, 0, 33)
    nk[[5, 256, B - 1]] = (0, Lk, 64)
    dev = lambda a: torch.from_numpy(a.astype(np.int32)).cuda()
    sq, sk, bias = dev(nq), dev(nk), torch.full((B,), -4.0, device="cuda")
    seven = lambda t: torch.full_like(t, 7.0)
    bits = lambda t: t.view(torch.int16)
    o = A.sigmoid_attn_cross_fwd(q, k, v, sq, sk, bias, d ** -0.5, out=seven(q))
    dq, db = A.sigmoid_attn_cross_bwd_dq_dbias(q, k, v, g, sq, sk, bias, d ** -0.5, dq=seven(q))
    for z in range(B):
        one = [t[z:z + 1] for t in (q, k, v, g, sq, sk, bias)]
        o1 = A.sigmoid_attn_cross_fwd(*one[:3], *one[4:], d ** -0.5)
        dq1, db1 = A.sigmoid_attn_cross_bwd_dq_dbias(*one, d ** -0.5)
        assert torch.equal(bits(o[z:z + 1]), bits(o1)), (z, "o")
        assert torch.equal(bits(dq[z:z + 1]), bits(dq1)) and torch.equal(db[z:z + 1], db1), (z, "dq, dbias")


@pytest.mark.parametrize("B,Lq,Lk,H,d", [
    (3, 333, 333, 50, 64),       # forward: 300 workgroups of 256 rows (two owner blocks a wave), one tile each
    (3, 100, 77, 3, 64),         # fewer rows than one pass over a tile or one owner block
    (300, 300, 300, 12, 64),     # several owner tiles a workgroup, two owner blocks a wave in the forward pass
    (240, 300, 140, 4, 128),     # several owner tiles a workgroup, d = 128
])
def test_padding_is_never_read_or_written(B, Lq, Lk, H, d):
    """Padded rows hold NaN and Inf: every load ends with the last valid row of its tile and every store with the last
    row of its sequence, in each pass over a tile and each owner block (the bits are those of zeros in the padding)."""
    import torch
    from paper_2604_27124_amd import binding as A
    gen = torch.Generator(device="cuda").manual_seed(B * H + d)
    rng = np.random.default_rng(B + Lq)
    nq, nk = rng.integers(0, Lq + 1, size=B), rng.integers(0, Lk + 1, size=B)
    edges = (Lq, 1, 33, 257, 270, 288, 289, 0)[:B]
    nq[:len(edges)] = np.minimum(edges, Lq)
    nk[B - len(edges):] = np.minimum(edges, Lk)
    if Lq == Lk:
        nk = nq
    dev = lambda a: torch.from_numpy(a.astype(np.int32)).cuda()
    sq, sk, bias = dev(nq), dev(nk), torch.full((B,), -4.0, device="cuda")

    def tensor(L, n, bad):
        clean = torch.empty(B, L, H, d, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
        pad = (torch.arange(L, device="cuda")[None, :] >= n[:, None])[:, :, None, None]
        return clean.masked_fill(pad, 0.0), clean.masked_fill(pad, bad)

    inf, nan = float("inf"), float("nan")
    pairs = [tensor(L, n, bad) for L, n, bad in ((Lq, sq, nan), (Lk, sk, inf), (Lk, sk, -inf), (Lq, sq, nan))]
    results = []
    for q, k, v, g in zip(*pairs):
        poison = lambda t: torch.full_like(t, 7.0)
        o = A.sigmoid_attn_cross_fwd(q, k, v, sq, sk, bias, d ** -0.5, out=poison(q))
        grads = A.sigmoid_attn_cross_bwd(q, k, v, g, sq, sk, bias, d ** -0.5, dq=poison(q), dk=poison(k), dv=poison(v))
        dq, db = A.sigmoid_attn_cross_bwd_dq_dbias(q, k, v, g, sq, sk, bias, d ** -0.5, dq=poison(q))
        results.append((o, *grads, dq, db))
    for n, clean, bad in zip((sq, sq, sk, sk, sq, None), *results):
        assert bool(bad.isfinite().all())
        assert torch.equal(clean, bad)
        if n is not None:
            nonzero = (bad != 0).any(dim=3).any(dim=2)
            other = sk if n is sq else sq                       # a row with nothing to stream is zero
            valid = (torch.arange(bad.shape[1], device="cuda")[None, :] < n[:, None]) & (other > 0)[:, None]
            assert torch.equal(nonzero, valid)


def test_rows_behind_a_tile_span_more_than_2_gib():
    """1100 rows of 16384 heads: from a head's first tile to its last valid row it is more than 2^31 bytes."""
    import torch
    from paper_2604_27124_amd import binding as A
    gen = torch.Generator(device="cuda").manual_seed(5)
    q, k, v, g = (torch.empty(1, 1100, 16384, 64, dtype=torch.bfloat16, device="cuda").normal_(generator=gen) for _ in range(4))
    n, bias = torch.tensor([1090], dtype=torch.int32, device="cuda"), torch.tensor([-7.0], device="cuda")
    whole = (A.sigmoid_attn_fwd(q, k, v, n, bias, 0.125), *A.sigmoid_attn_bwd(q, k, v, g, n, bias, 0.125))
    for h in (0, 9000, 16380):
        q1, k1, v1, g1 = (t[:, :, h:h + 4].contiguous() for t in (q, k, v, g))
        part = (A.sigmoid_attn_fwd(q1, k1, v1, n, bias, 0.125), *A.sigmoid_attn_bwd(q1, k1, v1, g1, n, bias, 0.125))
        for got, want in zip(whole, part):
            assert bool(want[0, :1090].any()) and not bool(want[0, 1090:].any())
            assert torch.equal(got[:, :, h:h + 4].contiguous().view(torch.int16), want.view(torch.int16)), h
