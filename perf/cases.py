"""What the framework's users run, as cases that can be timed and compared between two builds.

A case is one pass through the public entry points of `paper_2604_27124_amd.binding` on a seeded synthetic
batch: a forward pass (embedding extraction), a training step (forward and backward), its backward half
alone, a cross-attention step (queries and keys of different lengths) or a step with a learnable bias
(dQ and the bias gradient in one call).  Head shapes, lengths, padding and spreads are those of the named
workloads (`workloads.py`), of the benchmark grid (`grid.py`) and of the tests.
"""
import math
import random

import torch

from paper_2604_27124_amd import binding as A


def listed():
    return [
        # the smoke-test step: two short sequences, a few workgroups; launches and latency are everything
        dict(name="tiny_step", kind="step", B=2, H=2, d=64, N=256, Nk=0, lens="uniform", lo=173, hi=256, std=1.0),
        # one cell embedded on its own (interactive use): a single ragged sequence, forward only
        dict(name="one_cell_fwd", kind="fwd", B=1, H=12, d=64, N=1000, Nk=0, lens="full", lo=0, hi=0, std=1.0),
        # embedding extraction over a batch of an odd padded length, wide heads
        dict(name="embed_d128_fwd", kind="fwd", B=12, H=16, d=128, N=1537, Nk=0, lens="uniform", lo=400, hi=1537, std=1.0),
        # training on many short cells (more sequences than fit one ranking pass)
        dict(name="short_cells_step", kind="step", B=512, H=12, d=64, N=512, Nk=0, lens="lognormal", lo=16, hi=512, std=1.0),
        # the short end of the benchmark grid: 16384 tokens as 32 sequences, 25 % padding, backward
        dict(name="grid512_bwd", kind="bwd", B=32, H=32, d=64, N=512, Nk=0, lens="uniform", lo=384, hi=384, std=1.0),
        # training without padding, 160M-model head shape
        dict(name="unpadded_step", kind="step", B=8, H=12, d=64, N=2048, Nk=0, lens="full", lo=0, hi=0, std=1.0),
        # training on jagged cells, right-padded to the batch maximum
        dict(name="jagged_step", kind="step", B=16, H=12, d=64, N=4096, Nk=0, lens="lognormal", lo=64, hi=4096, std=1.0),
        # the headline workload: long jagged sequences, scores of a larger spread
        dict(name="long_step", kind="step", B=4, H=12, d=64, N=8192, Nk=0, lens="uniform", lo=1024, hi=8192, std=math.sqrt(2.0)),
        # the middle of the grid at the wide head shape, 25 % padding
        dict(name="grid2048_d128_step", kind="step", B=8, H=16, d=128, N=2048, Nk=0, lens="uniform", lo=1536, hi=1536, std=1.0),
        # the largest: very long sequences, wide heads
        dict(name="wide_step", kind="step", B=2, H=16, d=128, N=16384, Nk=0, lens="uniform", lo=12000, hi=16384, std=1.0),
        # cross-attention: a short query side against longer, ragged keys
        dict(name="cross_step", kind="cross", B=6, H=12, d=64, N=513, Nk=3001, lens="uniform", lo=200, hi=513, std=1.0),
        # training with a learnable bias
        dict(name="bias_step", kind="dbias", B=8, H=12, d=64, N=1500, Nk=0, lens="uniform", lo=500, hi=1500, std=1.0),
    ]


def draw(rng):
    """Kinds, head shapes, lengths and paddings as above, sizes spread over the logarithm of their range."""
    while True:
        kind = rng.choice(["fwd", "step", "step", "bwd", "cross", "dbias"])
        d = rng.choice([64, 64, 128])
        H = rng.choice([2, 4, 8, 12, 16, 32] if d == 64 else [2, 4, 8, 16])
        N = int(round(math.exp(rng.uniform(math.log(64), math.log(16384)))))
        most = max(1, min(512, 131072 // N))            # sequences of a batch of at most 131072 padded tokens
        B = int(round(math.exp(rng.uniform(0.0, math.log(most)))))
        Nk = int(round(math.exp(rng.uniform(math.log(64), math.log(8192))))) if kind == "cross" else 0
        lens = rng.choice(["full", "uniform", "uniform", "lognormal"])
        lo = max(1, int(N * rng.uniform(0.1, 0.9)))
        case = dict(kind=kind, B=B, H=H, d=d, N=N, Nk=Nk, lens=lens, lo=lo, hi=N, std=rng.choice([1.0, 1.0, math.sqrt(2.0)]))
        w = work(case)
        if w["flops"] <= 4.0e12 and w["bytes"] <= 2.0e9:   # no more than the largest listed one
            return case


def _lengths(case, N, salt):
    """Valid lengths of the batch, fixed by the case (their order within the batch is the seed's)."""
    if case["lens"] == "full":
        return [N] * case["B"]
    rng = random.Random("%d %d %d %d %s" % (salt, case["B"], N, case["lo"], case["lens"]))
    lo = max(1, min(N, round(case["lo"] * N / case["N"])))
    hi = max(lo, min(N, round(case["hi"] * N / case["N"])))
    if case["lens"] == "uniform":
        return [rng.randint(lo, hi) for _ in range(case["B"])]
    median = 0.38 * hi                                   # lognormal, median 1500 of 4096 and 200 of 512
    return [min(hi, max(lo, round(median * math.exp(0.8 * rng.gauss(0.0, 1.0))))) for _ in range(case["B"])]


def prepare(case, seed):
    """The tensors a training loop or an encoder has on the GPU before the call."""
    B, H, d, N, Nk = case["B"], case["H"], case["d"], case["N"], case["Nk"] or case["N"]
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(n, std):
        x = torch.empty(B, n, H, d, dtype=torch.bfloat16, device="cuda")
        return x.normal_(0.0, std, generator=gen)

    nq, nk = _lengths(case, N, 1), _lengths(case, Nk, 2 if case["Nk"] else 1)
    order = random.Random(seed).sample(range(B), B)
    nq, nk = [nq[i] for i in order], [nk[i] for i in order]
    s = dict(kind=case["kind"], scale=1.0 / math.sqrt(d), q=normal(N, case["std"]), k=normal(Nk, case["std"]),
             v=normal(Nk, case["std"]), nq=torch.tensor(nq, dtype=torch.int32, device="cuda"),
             nk=torch.tensor(nk, dtype=torch.int32, device="cuda"),
             bias=torch.tensor([-math.log(n) for n in nk], dtype=torch.float32, device="cuda"))
    if case["kind"] != "fwd":
        s["do"] = normal(N, 1.0)
    return s


def run(s):
    """One pass, as a user's program calls it: outputs are allocated by the call."""
    kind, q, k, v, n, bias, scale = s["kind"], s["q"], s["k"], s["v"], s["nq"], s["bias"], s["scale"]
    if kind == "fwd":
        return A.sigmoid_attn_fwd(q, k, v, n, bias, scale)
    if kind == "bwd":
        return A.sigmoid_attn_bwd(q, k, v, s["do"], n, bias, scale)
    if kind == "step":
        o = A.sigmoid_attn_fwd(q, k, v, n, bias, scale)
        return (o, *A.sigmoid_attn_bwd(q, k, v, s["do"], n, bias, scale))
    if kind == "cross":
        o = A.sigmoid_attn_cross_fwd(q, k, v, n, s["nk"], bias, scale)
        return (o, *A.sigmoid_attn_cross_bwd(q, k, v, s["do"], n, s["nk"], bias, scale))
    o = A.sigmoid_attn_fwd(q, k, v, n, bias, scale)      # "dbias": the bias is a trained parameter
    dk, dv = A.sigmoid_attn_bwd_dkdv(q, k, v, s["do"], n, bias, scale)
    dq, db = A.sigmoid_attn_bwd_dq_dbias(q, k, v, s["do"], n, bias, scale)
    return o, dq, dk, dv, db


def work(case):
    """4 d FLOP per valid (query, key) pair and head forward, 10 d backward (scores recomputed once); every
    valid input row read once per direction, every output row (padded ones as zeros) written once."""
    H, d, N, Nk = case["H"], case["d"], case["N"], case["Nk"] or case["N"]
    nq, nk = _lengths(case, N, 1), _lengths(case, Nk, 2 if case["Nk"] else 1)
    pairs = sum(a * b for a, b in zip(nq, nk))
    row = 2 * H * d
    fwd = case["kind"] != "bwd"
    bwd = case["kind"] != "fwd"
    flops = H * d * pairs * (4 * fwd + 10 * bwd)
    rows = fwd * (sum(nq) + 2 * sum(nk) + case["B"] * N) + bwd * (2 * sum(nq) + 2 * sum(nk) + case["B"] * (N + 2 * Nk))
    return {"bytes": rows * row, "flops": flops}


def tolerance(case):
    """Against the same formulas in 64-bit floats every output differs by 2.6e-3 to 3.9e-3 (2-norm) over these
    cases and draws: the bf16 roundings of P, dS, the scaled owner rows and the result.  Four times that."""
    return {"rel": 1.5e-2}
