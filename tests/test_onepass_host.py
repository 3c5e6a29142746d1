"""The one-pass backward on the host: which shapes take it, what the compiled kernel has to hold to, and that its work
mapping gives every tile once and in the order the chain of a head needs."""
import os
import random
import re
import subprocess

import pytest

from paper_2604_27124_amd import binding as A
from paper_2604_27124_amd import build as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_workspace_size():
    f = A.sigmoid_attn_bwd_onepass_workspace_bytes
    assert f(4, 8192, 12, 64) == 48 * (128 * 64 * 64 * 4 + 32 * 8 * 4)
    assert f(8, 2048, 12, 64) > 0 and f(7, 2048, 12, 64) == 0          # 768 tiles of 256 keys
    assert f(16, 1024, 12, 64) > 0 and f(64, 1023, 12, 64) == 0
    assert f(4, 8192, 12, 128) == 0 and f(0, 8192, 12, 64) == 0
    assert 0 < f(1000, 4096, 16, 64) <= 1 << 30                        # in slices
    assert f(1, 1100, 16384, 64) == 0                                  # one sequence that no slice can hold


def test_compiled_kernel(tmp_path):
    """No spills and two waves a SIMD (the loop has no register to spare); every tile barrier waits for all LDS work; the
    sums between workgroups are stored and read at agent scope, and each count follows a full wait for them."""
    out = tmp_path / "api.s"
    flags = [f for f in B.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([B.hipcc(), *flags, "-I", os.path.join(ROOT, "include"), "-S", "--cuda-device-only", "-o", str(out),
                    os.path.join(B.CSRC, "sigattn_api.hip")], check=True, capture_output=True)
    text = out.read_text()
    text = text[re.search(r"^_ZN7sigattn7onepass15sigattn_onepass\w+:", text, re.M).start():]
    end = text.index(".Lfunc_end")
    meta = dict(re.findall(r"^; (NumVgprs|ScratchSize|Occupancy): (\d+)", text[end:end + 6000], re.M)[:3])
    assert meta["ScratchSize"] == "0" and meta["Occupancy"] == "2"
    body = [l.split(";")[0].strip() for l in text[:end].split("\n")]
    body = [l for l in body if l and not l.startswith(".")]
    assert not any(re.match(r"v_pk_(add|mul|fma)_f32", l) for l in body)
    waits = [re.search(r"s_waitcnt .*lgkmcnt\((\d+)\)", body[i - 1]) for i, l in enumerate(body) if l == "s_barrier"]
    assert len(waits) == 10 and all(m and m.group(1) == "0" for m in waits)
    counts = [i for i, l in enumerate(body) if l.startswith("global_store_dword ")]
    assert counts
    for i in counts:
        assert body[i].endswith("sc1")
        sums = max(j for j in range(i) if body[j].startswith("buffer_store"))
        assert "s_waitcnt vmcnt(0)" in body[sums:i], body[sums:i]


def map_work(wg, nq, nk, H, T, group):
    """The device's mapping of a ranked launch, step by step (lists stand for the lanes of a wave)."""
    n = len(nq)
    tiles_of = [(k + 255) // 256 for k in nk]
    if wg >= sum(tiles_of) * H:                                        # padded tiles
        lo = sum(tiles_of)
        for z in range(n):
            if lo * H <= wg < (lo + T - tiles_of[z]) * H:
                e = wg - lo * H
                return z, e % H, tiles_of[z] + e // H
            lo += T - tiles_of[z]
    rank = [sum(nq[u] >= nq[l] + (l <= u) for u in range(n)) for l in range(n)]
    seq = sorted(range(n), key=lambda l: rank[l])
    tiles = [tiles_of[z] for z in seq]
    start = [sum(tiles[:l]) * H for l in range(n)]
    lo = max(l for l in range(0, n, group) if start[l] <= wg)
    hi, e = min(n, lo + group), wg - start[lo]
    for j in range(T):
        before, here = sum(min(t, j) for t in tiles[lo:hi]), sum(t > j for t in tiles[lo:hi])
        if before * H <= e < (before + here) * H:
            r = e - before * H
            return seq[[l for l in range(lo, hi) if tiles[l] > j][r // H]], r % H, j


@pytest.mark.parametrize("seed", range(20))
def test_mapping_is_complete_and_ordered(seed):
    rng = random.Random(seed)
    n, H, L = rng.choice((1, 2, 5, 16, 64)), rng.choice((1, 2, 12)), rng.choice((200, 256, 300, 4096))
    nk = [rng.randint(0, L) for _ in range(n)]
    nq = nk if seed % 2 else [rng.randint(0, 700) for _ in range(n)]
    T, seen, last = (L + 255) // 256, set(), {}
    for wg in range(n * H * T):
        z, h, j = map_work(wg, nq, nk, H, T, min(n, 1 + seed % 5))
        seen.add((z, h, j))
        if j * 256 < nk[z]:
            assert last.get((z, h), -1) == j - 1                       # a tile's predecessor has a smaller id
            last[z, h] = j
    assert len(seen) == n * H * T
