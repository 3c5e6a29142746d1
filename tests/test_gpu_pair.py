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
