"""Small launches (d = 64: two waves share 32 owner rows; d = 128: four waves a workgroup, one backward launch) against the kernels of larger launches: the same
sequences with others beside them in the batch.  Every sum has the same order, so the bits are the same."""
import numpy as np
import pytest
import torch

from paper_2604_27124_amd import binding as A

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq,nk,Lq,Lk", [
    ((1, 64), (1, 64), 64, 64),            # one tile, one row
    ((31, 65), (33, 128), 65, 130),        # blocks and tiles just missed, two tiles
    ((192, 129), (192, 129), 200, 200),    # three tiles; the halves of the backward on their own
    ((256, 255), (256, 225), 257, 256),    # four: every slot of the ring
    ((300, 0), (257, 300), 300, 320),      # five and a row; a sequence without queries
    ((100, 37), (0, 1000), 100, 1000),     # without keys; sixteen tiles against two
])
@pytest.mark.parametrize("d", [64, 128])
def test_same_bits_as_larger_launches(nq, nk, Lq, Lk, d):
    H, copies = 2, 512                     # more than 1024 tiles with the copies, at most 64 without
    gen = torch.Generator(device="cuda").manual_seed(Lq * Lk)
    normal = lambda n: torch.empty(2, n, H, d, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    q, k, v, g = normal(Lq), normal(Lk), normal(Lk), normal(Lq)
    sq, sk = (torch.tensor(n, dtype=torch.int32, device="cuda") for n in (nq, nk))
    q[1, 0, 1, 3] = float("inf")           # saturates one row's scores; may not reach others
    for t, n in ((q, nq), (k, nk), (v, nk), (g, nq)):
        for z in range(2):
            t[z, n[z]:] = float("nan")     # padding is not read
    args = (q, k, v, g, sq, sk, torch.tensor([-3.0, -5.0], device="cuda"))
    many = [t.repeat(copies, *[1] * (t.dim() - 1)) for t in args]

    def calls(q, k, v, g, sq, sk, b):
        seven = lambda t: torch.full_like(t, 7.0)
        o = A.sigmoid_attn_cross_fwd(q, k, v, sq, sk, b, 0.125, out=seven(q))
        grads = A.sigmoid_attn_cross_bwd(q, k, v, g, sq, sk, b, 0.125, dq=seven(q), dk=seven(k), dv=seven(v))
        halves = ()
        if q.shape == k.shape and nq == nk:
            halves = (A.sigmoid_attn_bwd_dq(q, k, v, g, sq, b, 0.125, dq=seven(q)), *A.sigmoid_attn_bwd_dkdv(q, k, v, g, sq, b, 0.125, seven(k), seven(v)))
        return (o, *grads, *halves)

    for few, all_ in zip(calls(*args), calls(*many)):
        for z in (0, 2 * copies - 2):
            assert torch.equal(few.view(torch.int16), all_[z:z + 2].view(torch.int16))
        assert not bool((few == 7).all(dim=3).any())


@pytest.mark.parametrize("B,Lq,Lk,H,d", [
    (128, 64, 64, 1, 64),          # batch order: forward, dQ, dK/dV, joint backward
    (65, 100, 100, 1, 64),         # two tiles a head: forward and halves in batch order
    (256, 64, 64, 1, 64),          # a workgroup to every CU
    (66, 64, 128, 1, 64),          # joint backward of passes of different lengths, two of three workgroups to a head in the first
    (128, 128, 128, 1, 128),       # d = 128: all in batch order
    (65, 250, 250, 1, 128),        # joint backward of 260, ranked by histogram
    (100, 129, 129, 1, 128),
])
def test_more_sequences_than_lanes(B, Lq, Lk, H, d):
    """Every tile is taken once, and every sequence has the bits it has in a larger launch."""
    gen = torch.Generator(device="cuda").manual_seed(B * Lq + d)
    normal = lambda n: torch.empty(B, n, H, d, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    q, k, v, g = normal(Lq), normal(Lk), normal(Lk), normal(Lq)
    rng = np.random.default_rng(B + Lq)
    nq, nk = rng.integers(0, Lq + 1, size=B), rng.integers(0, Lk + 1, size=B)
    nq[:5], nk[:5] = (Lq, 0, 1, min(63, Lq), Lq), (Lk, 1, Lk, 0, min(129, Lk))
    if Lq == Lk:
        nk = nq
    sq, sk = (torch.from_numpy(n.astype(np.int32)).cuda() for n in (nq, nk))
    args = (q, k, v, g, sq, sk, torch.full((B,), -4.0, device="cuda"))
    copies = 2 + 1100 // B
    many = [t.repeat(copies, *[1] * (t.dim() - 1)) for t in args]

    def calls(q, k, v, g, sq, sk, b):
        seven = lambda t: torch.full_like(t, 7.0)
        out = [A.sigmoid_attn_cross_fwd(q, k, v, sq, sk, b, 0.125, out=seven(q))]
        out += A.sigmoid_attn_cross_bwd(q, k, v, g, sq, sk, b, 0.125, dq=seven(q), dk=seven(k), dv=seven(v))
        if Lq == Lk:
            out += [A.sigmoid_attn_bwd_dq(q, k, v, g, sq, b, 0.125, dq=seven(q)), *A.sigmoid_attn_bwd_dkdv(q, k, v, g, sq, b, 0.125, seven(k), seven(v))]
        return out

    for i, (few, all_) in enumerate(zip(calls(*args), calls(*many))):
        for z in (0, (copies - 1) * B):
            assert torch.equal(few.view(torch.int16), all_[z:z + B].view(torch.int16)), i
