"""The one-pass backward on the host: which shapes take it, what the compiled kernel (and those of the pairs) has to hold
to, that its plan (its own functions, run on the CPU) gives every tile once and in the order the chain of a head needs, and that
two launches at once end."""
import ctypes
import os
import random
import re
import subprocess

import numpy as np
import pytest

from paper_2604_27124_amd import binding as A
from paper_2604_27124_amd import build as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_workspace_size():
    f = A.sigmoid_attn_bwd_onepass_workspace_bytes
    assert f(4, 8192, 12, 64) == 48 * (128 * 64 * 64 * 4 + 32 * (8 * 4 + 32))
    assert f(8, 2048, 12, 64) > 0 and f(7, 2048, 12, 64) == 0          # 768 tiles of 256 keys
    assert f(128, 449, 12, 64) > 0 and f(128, 512, 12, 64) > 0 and f(500, 448, 12, 64) == 0
    assert f(127, 449, 12, 64) == 0 and f(127, 512, 12, 64) == 0 and f(32, 513, 12, 64) > 0    # two tiles a head: 3072
    assert f(32, 512, 32, 64) == 0
    assert f(4, 8192, 12, 128) == 0 and f(0, 8192, 12, 64) == 0
    assert 0 < f(1000, 4096, 16, 64) <= 1 << 29                        # in slices
    assert f(1, 1100, 16384, 64) == 0                                  # one sequence that no slice can hold


def test_plan_needs_no_more_alignment_than_a_workspace_has(tmp_path):
    src = tmp_path / "align.hip"
    src.write_text('#include "sigattn_onepass.hpp"\n'
                   "static_assert(alignof(sigattn::onepass::TileWork) <= 16 && alignof(sigattn::u32x4) <= 16, \"aligned to 16 bytes\");\n")
    flags = [f for f in B.HIPCC_FLAGS if f not in ("-shared", "-fPIC", "-O3")]
    r = subprocess.run([B.hipcc(), *flags, "-I", B.CSRC, "-fsyntax-only", "--cuda-device-only", str(src)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out = tmp_path_factory.mktemp("isa") / "api.s"
    flags = [f for f in B.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([B.hipcc(), *flags, "-I", os.path.join(ROOT, "include"), "-S", "--cuda-device-only", "-o", str(out),
                    os.path.join(B.CSRC, "sigattn_api.hip")], check=True, capture_output=True)
    return out.read_text()


@pytest.mark.parametrize("kernel", ["7onepass15sigattn_onepassE", "4pair12sigattn_pairILi0E", "4pair12sigattn_pairILi1E",
                                    "4pair12sigattn_pairILi2E", "4pair16sigattn_pair_bwdE", "7half12812sigattn_halfILi0E",
                                    "7half12812sigattn_halfILi1E", "7half12816sigattn_half_bwdE"])
def test_compiled_kernels(assembly, kernel):
    """No spills, and two waves a SIMD where one is not all there is; in the kernels with loops of their own every barrier
    waits for all LDS work (the partial waits of the d = 128 ones are looked at with those of the large kernels, whose loop
    they run).  One pass: the sums between workgroups are stored and read at agent scope, and between the last of them and each
    count stands a full wait."""
    text = assembly[re.search(rf"^_ZN7sigattn{kernel}\w+:", assembly, re.M).start():]
    end = text.index(".Lfunc_end")
    meta = dict(re.findall(r"^; (NumVgprs|ScratchSize|Occupancy): (\d+)", text[end:end + 6000], re.M)[:3])
    alone = kernel.endswith(("halfILi1E", "half_bwdE"))                # one wave a SIMD with all its registers
    assert meta["ScratchSize"] == "0" and meta["Occupancy"] == ("1" if alone else "2")
    body = [l.split(";")[0].strip() for l in text[:end].split("\n")]
    body = [l for l in body if l and not l.startswith(".")]
    assert not any(re.match(r"v_pk_(add|mul|fma)_f32", l) for l in body)
    if "half" in kernel:
        return
    barriers = [i for i, l in enumerate(body) if l == "s_barrier"]
    assert len(barriers) >= 10
    for i in barriers:                                                 # the wait may stand a few plain instructions before
        j = next(j for j in range(i - 1, i - 9, -1) if not re.match(r"(v_|s_)(?!waitcnt|load|buffer_load|barrier)", body[j]))
        assert re.match(r"s_waitcnt .*lgkmcnt\(0\)", body[j]), body[j:i + 1]
    if "onepass" not in kernel:
        return
    counts = [i for i, l in enumerate(body) if l.startswith("global_store_dword ")]
    assert counts and all(body[i].endswith("sc1") for i in counts)
    for i in counts:
        wait = next(j for j in range(i - 1, -1, -1) if body[j].startswith(("s_waitcnt vmcnt(0)", "buffer_", "global_", "ds_", "v_mfma")))
        assert body[wait].startswith("s_waitcnt vmcnt(0)"), body[wait:i + 1]     # before any other memory or matrix work
    sums = [l for l in body if l.startswith("buffer_store_dwordx4") and l.endswith("sc1")]
    assert len(sums) >= 4 * len(counts) and len(sums) % 4 == 0


def test_key_tiles_are_taken_from_a_counter(assembly):
    """Which key tile of its head a workgroup works on is how many of the head have been taken before: one atomic addition that
    returns, by one lane, handed to the others by a barrier before anything of the tile is read."""
    text = assembly[re.search(r"^_ZN7sigattn7onepass15sigattn_onepassE\w+:", assembly, re.M).start():]
    body = [l.split(";")[0].strip() for l in text[:text.index(".Lfunc_end")].split("\n")]
    atomics = [i for i, l in enumerate(body) if "_atomic_" in l]
    assert len(atomics) == 1 and re.match(r"global_atomic_add v\d+, .* sc0$", body[atomics[0]])
    handed = next(i for i in range(atomics[0], len(body)) if body[i] == "s_barrier")
    loads = [i for i, l in enumerate(body) if l.startswith("buffer_load")]
    assert [i for i in loads if i < handed] == loads[:2]              # those of queries and dO, which do not depend on the tile


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    """The ids [B, H, key tiles] that the plan kernel's own functions give, compiled for the host."""
    out = tmp_path_factory.mktemp("plan") / "plan.so"
    flags = [f for f in B.HIPCC_FLAGS if f != "-O3"]
    subprocess.run([B.hipcc(), *flags, "--offload-host-only", "-I", B.CSRC, "-o", str(out),
                    os.path.join(os.path.dirname(__file__), "onepass_plan.hip")], check=True, capture_output=True)
    lib = ctypes.CDLL(str(out))

    def ids(nq, nk, H, L_q, L_k, group=None):
        n, T = len(nq), (L_k + 255) // 256
        group = lib.group_of(n, H, (L_q + 63) // 64) if group is None else group
        assert 1 <= group <= n
        q, k, got = np.array(nq, dtype=np.int32), np.array(nk, dtype=np.int32), np.full((n, H, T), -1, dtype=np.int32)
        at = lambda a: a.ctypes.data_as(ctypes.c_void_p)
        assert lib.plan_ids(at(q), at(k), n, H, L_q, L_k, group, at(got)) == T
        return got, group

    return ids


def place(z, h, j, nq, nk, H, T, group):
    """The id of a tile, step by step from what the plan is to be."""
    n, tiles = len(nq), [(k + 255) // 256 for k in nk]
    if n > 256:                                                        # batch order
        z0 = z - z % group
        return z0 * H * T + (j * min(group, n - z0) + z - z0) * H + h
    rank = [sum(nq[u] > nq[v] or (nq[u] == nq[v] and u < v) for u in range(n)) for v in range(n)]
    ranked = [tiles[v] for v in sorted(range(n), key=lambda v: rank[v])]
    r, lo = rank[z], rank[z] - rank[z] % group
    if j < tiles[z]:
        at = sum(ranked[:lo]) + sum(min(t, j) + (k < r and t > j) for k, t in list(enumerate(ranked))[lo:lo + group])
    else:
        at = sum(ranked) + sum(T - t for t in tiles[:z]) + j - tiles[z]
    return at * H + h


@pytest.mark.parametrize("n,H,L,group", [
    (1, 1, 200, None), (1, 12, 16500, None), (2, 3, 256, 1), (5, 10, 4100, None), (16, 2, 300, 3), (64, 3, 1500, 7), (70, 3, 1024, None),
    (255, 1, 600, 255), (256, 1, 600, None), (256, 2, 449, 100), (257, 1, 600, None), (260, 2, 650, 9), (600, 3, 513, None),
])
@pytest.mark.parametrize("seed", range(4))
def test_plan_is_complete_and_ordered(plan, n, H, L, group, seed):
    """Every tile has an id and every id a tile; a head's tiles have rising ids; tiles with valid keys come before those
    without (more than 256 sequences: in batch order).  Lengths out of range are clamped, and empty sides have no tiles."""
    rng = random.Random(f"{n} {H} {L} {seed}")
    nk = [rng.choice((rng.randint(0, L), rng.randint(0, L), 0, L, L + 5, -3)) for _ in range(n)]
    nq = nk if seed % 2 else [rng.choice((rng.randint(0, 700), 0, 64)) for _ in range(n)]      # queries of their own: also none where there are keys
    L_q = L if seed % 2 else 700
    ids, group = plan(nq, nk, H, L_q, L, group)
    clamp = lambda v, top: max(0, min(v, top))
    cq, ck = [clamp(v, L_q) for v in nq], [clamp(v, L) for v in nk]
    assert sorted(ids.ravel()) == list(range(ids.size))
    assert (np.diff(ids, axis=2) > 0).all()
    T = ids.shape[2]
    for z in rng.sample(range(n), min(n, 12)):
        for h in {0, H - 1}:
            for j in {0, T // 2, T - 1}:
                assert ids[z, h, j] == place(z, h, j, cq, ck, H, T, group), (z, h, j)
    if n <= 256:
        valid = np.arange(T)[None, None, :] < np.array([(k + 255) // 256 for k in ck])[:, None, None]
        valid = np.broadcast_to(valid, ids.shape)
        assert not valid.any() or valid.all() or ids[valid].max() < ids[~valid].min()
        order = [z for z in sorted(range(n), key=lambda z: (-cq[z], z)) if ck[z] > 0]          # groups of ranks: longest first
        first = [ids[z, 0, 0] for z in order]
        assert group > 1 or first == sorted(first)


def finishes(launches, by_start, first, cus=4):
    """Two launches of one-pass workgroups on a GPU of eight XCDs of `cus` CUs, a workgroup to a CU.  Ids go to the XCDs in turn,
    and each XCD starts its ids of a launch in order, those of launch first[xcd] before the other's.  A launch is the plan: the
    (head, key tile) of each id.  A workgroup takes that tile, or (by_start) the next one of that head, and ends when the
    tile before its own has.  True if both launches end."""
    queues = [[[i for i in range(len(t)) if i % 8 == x] for t in launches] for x in range(8)]
    taken, running, done = [{}, {}], [[] for _ in range(8)], [set(), set()]
    moved = True
    while moved:
        moved = False
        for x in range(8):
            for l in (first[x], 1 - first[x]):
                while queues[x][l] and len(running[x]) < cus:
                    head, j = launches[l][queues[x][l].pop(0)]
                    taken[l][head] = taken[l].get(head, 0) + 1
                    running[x].append((l, head, taken[l][head] - 1 if by_start else j))
                    moved = True
        for x in range(8):
            for l, head, j in list(running[x]):
                if j == 0 or (head, j - 1) in done[l]:
                    running[x].remove((l, head, j))
                    done[l].add((head, j))
                    moved = True
    return all(len(d) == len(t) for d, t in zip(done, launches))


@pytest.mark.parametrize("H,sequences,T", [(12, 5, 6), (3, 20, 5), (8, 4, 6)])
def test_overlapping_launches_end(plan, H, sequences, T):
    """With tiles taken by start both launches end, whichever each XCD starts first; with tiles by id they can wait for each other
    for ever (not where the number of heads keeps a head on one XCD)."""
    n = [256 * T] * sequences
    ids, _ = plan(n, n, H, 256 * T, 256 * T, sequences)
    launch = [(i // T, i % T) for i in np.argsort(ids.ravel())]
    orders = [[m >> x & 1 for x in range(8)] for m in range(256)]
    assert all(finishes([launch, launch], True, first) for first in orders)
    assert all(finishes([launch, launch], False, first) for first in orders) == (H % 8 == 0)
