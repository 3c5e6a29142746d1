"""Properties of the compiled gfx950 code that the kernels' synchronisation relies on, checked on the
assembly hipcc emits (cross-compiled here, no GPU needed).

The barrier that closes a streamed tile waits with `s_waitcnt lgkmcnt(k)` only until the tile's LDS
writes have completed, letting the k operand reads issued behind them stay in flight.  That is correct
only if (a) exactly k LDS reads, and nothing else that counts on that counter (no scalar loads), lie
between the writes and the barrier in the emitted code, and (b) the packed-fp32 forms stay switched off.
"""
import os
import re
import subprocess
import tempfile

import pytest

from paper_2604_27124_amd import build as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


FWD, DQ, DKDV = 0, 1, 2


@pytest.fixture(scope="module")
def kernels():
    """name -> instruction lines of its body and its register figures, one entry per attention kernel of the library
    (the second stage of the bias gradient has neither matrix work nor a ring of tiles)."""
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "api.s")
        flags = [f for f in B.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
        cmd = [B.hipcc(), *flags, "-I", os.path.join(ROOT, "include"), "-S", "--cuda-device-only", "-o", out,
               os.path.join(B.CSRC, "sigattn_api.hip")]
        subprocess.run(cmd, check=True, capture_output=True)
        text = open(out).read()
    result, name, in_body = {}, None, False
    for line in text.split("\n"):
        m = re.match(r"^(_Z\w+):", line)                  # any function: what follows belongs to it, not to the one before
        if m:
            name = m.group(1) if re.match(r"_ZN7sigattn(7half128)?\d+sigattn_((bwd_)?kernel|half)", m.group(1)) else None
            in_body = name is not None
            if in_body:
                result[name] = {"body": [], "meta": {}}
            continue
        if name is None:
            continue
        if line.startswith(".Lfunc_end"):
            in_body = False
        m = re.match(r"^; (NumVgprs|ScratchSize|Occupancy): (\d+)", line)     # behind the function's end
        if m:
            assert not in_body and m.group(1) not in result[name]["meta"], name
            result[name]["meta"][m.group(1)] = int(m.group(2))
        ins = line.split(";")[0].strip()
        if in_body and ins and not ins.startswith("."):
            result[name]["body"].append(ins)
    return result


def passes_and_d(name):
    """The passes a kernel holds, and its head dimension."""
    if "half128" in name:                                 # the same loops in four-wave workgroups, d = 128
        m = re.search(r"sigattn_halfILi(\d)E", name)
        return ((int(m.group(1)),) if m else (DKDV, DQ)), 128
    m = re.search(r"sigattn_bwd_kernelILi(\d+)E", name)
    if m:
        return (DKDV, DQ), int(m.group(1))
    m = re.search(r"sigattn_kernelILi(\d)ELi(\d+)E", name)
    return (int(m.group(1)),), int(m.group(2))


def test_every_kernel_is_looked_at(kernels):
    shapes = sorted((d, p) for p, d in map(passes_and_d, kernels))
    assert shapes == sorted([(64, (FWD,))] * 2 + [(64, (DKDV,)), (64, (DQ,)), (64, (DQ,)), (64, (DKDV, DQ)),
                            (128, (FWD,)), (128, (DKDV,)), (128, (DQ,)), (128, (DQ,)),
                            (128, (FWD,)), (128, (DQ,)), (128, (DKDV, DQ))])             # the last three: half128
    for name, k in kernels.items():
        assert set(k["meta"]) == {"NumVgprs", "ScratchSize", "Occupancy"}, name
        assert any(ins.startswith("s_endpgm") for ins in k["body"]), name


def test_tile_barrier_counts_its_reads(kernels):
    for name, k in kernels.items():
        body = k["body"]
        partial = []                              # barriers that end a tile, in the order of the code
        for i, ins in enumerate(body):
            if ins != "s_barrier":
                continue
            # the LDS wait that belongs to the barrier: the nearest instruction before it that is not plain
            # ALU work (the compiler may slip a few such instructions in between; no LDS or scalar-memory
            # instruction may sit there)
            w = i - 1
            while w >= 0 and re.match(r"(v_|s_)(?!waitcnt|load|buffer_load|barrier)", body[w]) and i - w < 8:
                w -= 1
            m = re.match(r"s_waitcnt (?:vmcnt\(\d+\) )?lgkmcnt\((\d+)\)$", body[w])
            assert m, f"{name}: barrier without an LDS wait in front of it ({body[w]!r})"
            allowed = int(m.group(1))
            if allowed == 0:
                continue                      # a full wait is always safe
            assert w == i - 1, f"{name}: instructions between a partial LDS wait and its barrier"
            reads, j = 0, i - 2
            while j >= 0 and not body[j].startswith("ds_write"):
                assert not body[j].startswith(("s_load", "s_buffer_load", "s_barrier")), \
                    f"{name}: {body[j]!r} between the tile store and its barrier"
                if body[j].startswith("ds_read"):
                    reads += 1
                j -= 1
            assert j >= 0, f"{name}: partial LDS wait with no tile store before it"
            assert reads == allowed, f"{name}: lgkmcnt({allowed}) but {reads} LDS reads follow the tile store"
            partial.append(i)
        loops = len(passes_and_d(name)[0])
        assert len(partial) == 4 * loops, f"{name}: {len(partial)} tile barriers"    # four unrolled ring slots a pass
        # registers parked in scratch may come and go per owner tile, never from tile to tile
        for first, last in ((partial[4 * l], partial[4 * l + 3]) for l in range(loops)):
            spills = [ins for ins in body[first:last] if ins.startswith("scratch_")]
            assert not spills, f"{name}: {spills} between the tiles of one pass"


def test_no_packed_fp32_and_next_to_no_spills(kernels):
    for name, k in kernels.items():
        for ins in k["body"]:
            assert not re.match(r"v_pk_(add|mul|fma)_f32", ins), f"{name}: packed fp32 instruction {ins!r}"
        # two registers a lane: what the four-wave joint backward and the d = 128 dQ + dbias kernel park today
        assert k["meta"]["ScratchSize"] <= 8, f"{name}: register spills"
        alone = passes_and_d(name) == ((DKDV,), 128) or ("half128" in name and passes_and_d(name)[0] != (FWD,))
        assert k["meta"]["Occupancy"] >= (1 if alone else 2), f"{name}: waves per SIMD"


def test_hot_loops_use_the_matrix_and_transcendental_pipes(kernels):
    for name, k in kernels.items():
        ops = [ins.split()[0] for ins in k["body"]]
        loops = len(passes_and_d(name)[0])
        assert ops.count("v_mfma_f32_32x32x16_bf16") > 64 * loops, name
        assert any(o.startswith("v_exp_f32") for o in ops) and any(o.startswith("v_rcp_f32") for o in ops), name
        assert any(o == "ds_read_b64_tr_b16" for o in ops), name


@pytest.mark.parametrize("rows,compiles", [(64, True), (128, False)])
def test_only_tiles_of_two_blocks_compile(tmp_path, rows, compiles):
    """At the last tile of an owner tile the next owner rows are loaded behind the first 32-row block: with more than two
    blocks the scores of the later ones would be computed from them, so such a shape must not compile."""
    src = tmp_path / "shape.hip"
    src.write_text('#include "sigattn_kernels.hpp"\n'
                   f"template __global__ void sigattn::sigattn_kernel<sigattn::FWD, 64, 1, 8, {rows}, 72, 72, 1, 4>(const sigattn::Params);\n")
    flags = [f for f in B.HIPCC_FLAGS if f not in ("-shared", "-fPIC", "-O3")]
    r = subprocess.run([B.hipcc(), *flags, "-I", B.CSRC, "-fsyntax-only", "--cuda-device-only", str(src)],
                       capture_output=True, text=True)
    assert (r.returncode == 0) == compiles, r.stderr[-2000:]
    assert compiles or "two 32-row blocks" in r.stderr
