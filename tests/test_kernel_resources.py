"""Register and scratch budget of the gfx950 kernels, read from the compiler's code-object
metadata (no GPU needed).

A producer wave holds 256 accumulation registers plus its vector registers; in a shared-CU
run two consumer waves must fit beside it on each SIMD (512 registers), and no kernel may
spill to scratch (a spill in the MFMA loop costs an order of magnitude).
"""
import ctypes
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_19539_amd", "csrc")
SOURCES = ["kernels.hip", "combine.hip", "plan_device.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
SIMD_REGISTERS = 512
CONSUMER_WAVES_BESIDE_PRODUCER = 2


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    found = {}
    for src in SOURCES:
        out = tmp_path_factory.mktemp("dev") / (src + ".s")
        subprocess.run([HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-x", "hip", "--cuda-device-only",
                        "-S", os.path.join(CSRC, src), f"-I{os.path.join(ROOT, 'include')}", f"-I{CSRC}", "-o", str(out),
                        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"],
                       check=True, capture_output=True)
        out_text = out.read_text()
        meta = out_text.split("amdhsa.kernels:", 1)[1]
        for block in re.split(r"\n  - ", meta)[1:]:
            fields = dict(re.findall(r"^\s*\.(\w+):\s+(\S+)", block, re.M))
            if "name" in fields:
                found[fields["name"]] = fields
                body = out_text.split("\n" + fields["name"] + ":", 1)[1].split(".Lfunc_end", 1)[0]
                found[fields["name"]]["body"] = body
    return found


def by_name(kernels, fragment):
    hits = {n: f for n, f in kernels.items() if fragment in n}
    assert hits, fragment
    return hits


def test_no_kernel_spills(kernels):
    for name, f in kernels.items():
        assert int(f["private_segment_fixed_size"]) == 0, name
        assert int(f["vgpr_spill_count"]) == 0, name


def test_consumer_fits_beside_a_producer_wave(kernels):
    """The shared-CU consumer variant (kOwn = false) leaves a producer wave its registers; the
    variant for compute units of its own keeps four waves per SIMD."""
    (cons,) = by_name(kernels, "consumer_kernelILb0ELb0E").values()   # the MOE_WRITE_COUNTS
    (own,) = by_name(kernels, "consumer_kernelILb1ELb0E").values()    # variants are outside it
    assert int(own["vgpr_count"]) <= 128
    granule = 8  # registers are allocated to a wave in blocks of 8
    cons_alloc = -(-int(cons["vgpr_count"]) // granule) * granule
    budget = SIMD_REGISTERS - CONSUMER_WAVES_BESIDE_PRODUCER * cons_alloc
    # The launches taken by default (split 1 to 4 parts) must leave that room.
    for name, f in by_name(kernels, "producer_kernel").items():
        tag = re.search(r"ILb[01]ELi(n?\d+)E", name).group(1)
        split = -int(tag[1:]) if tag.startswith("n") else int(tag)
        if split in (-1, 1, 2, 3, 4):
            assert int(f["vgpr_count"]) <= budget, (name, f["vgpr_count"], budget)
        assert int(f["agpr_count"]) == 256, name


def _registers(text):
    """Vector ('v'), accumulation ('a') and scalar ('s') registers that an instruction names."""
    out = {(b, int(n)) for b, n in re.findall(r"\b([vas])(\d+)\b", text)}
    for b, lo, hi in re.findall(r"\b([vas])\[(\d+):(\d+)\]", text):
        out |= {(b, i) for i in range(int(lo), int(hi) + 1)}
    return out


def test_producer_assembly_keeps_its_distances(kernels):
    """The matrix instructions and the LDS DMAs are assembly statements, which the compiler's own wait
    states do not cover.  In the emitted order of each kernel: no vector instruction writes an operand
    within two wait states before a matrix instruction reads it, none but a matrix instruction touches an
    accumulator within 11 of its product, and no lane read writes a DMA's scalar base within 5."""
    for name, f in by_name(kernels, "producer_kernel").items():
        ins = [line.split(";")[0].strip() for line in f["body"].split("\n")
               if line.startswith("\t") and not line.strip().startswith((".", ";"))]
        states = [int(i.split()[1]) + 1 if i.startswith("s_nop") else 1 for i in ins]
        n_mfma = 0

        def before(i, limit):
            ws = 0
            while i > 0 and ws < limit:
                i -= 1
                yield ins[i]
                ws += states[i]

        for i, op in enumerate(ins):
            if op.startswith("v_mfma"):
                n_mfma += 1
                reads = {r for r in _registers(op) if r[0] in "va"}
                for p in before(i, 2):
                    if p.startswith("v_") and not p.startswith(("v_mfma", "v_cmp")):
                        assert not _registers(p.split(None, 1)[1].split(",")[0]) & reads, (name, p, op)
                acc = {r for r in _registers(op) if r[0] == "a"}
                ws = 0
                for k in range(i + 1, len(ins)):
                    if ws >= 11 or ins[k].startswith(("s_cbranch", "s_branch", "s_endpgm")):
                        break
                    assert ins[k].startswith("v_mfma") or not _registers(ins[k]) & acc, (name, op, ins[k])
                    ws += 4 if ins[k].startswith("v_mfma") else states[k]
            elif op.startswith("global_load_lds"):
                base = {r for r in _registers(op) if r[0] == "s"}
                for p in before(i, 5):
                    if p.startswith(("v_readlane", "v_readfirstlane")):
                        assert not _registers(p.split(None, 1)[1].split(",")[0]) & base, (name, p, op)
        assert n_mfma > 100, name


def test_every_split_variant_is_instantiated(kernels):
    names = set(by_name(kernels, "producer_kernel"))
    for down, split in ((0, 1), (1, 1), (1, 2), (1, 3), (1, 4), (1, 0), (1, "n1")):
        assert any(f"ILb{down}ELi{split}E" in n for n in names), (down, split)


def test_combine_variants_present(kernels):
    names = set(by_name(kernels, "combine_kernel"))
    assert len(names) == 3, names


def test_combine_rows_of_a_batch_are_in_flight_together(kernels):
    """The combine's time with few tokens is a chain of loads: between the row loads of a batch of four
    choices nothing may wait for a vector load (three choices' loads in a row here: the compiler may lay
    the last one's out elsewhere)."""
    for name, f in by_name(kernels, "combine_kernel").items():
        vec = int(re.search(r"combine_kernelILi(\d)E", name).group(1))
        ops = re.findall(r"^\s(global_load_dwordx4|s_waitcnt vmcnt\(\d+\))", f["body"], re.M)
        longest = run = 0
        for op in ops:
            run = run + 1 if op.startswith("global_load") else 0
            longest = max(longest, run)
        assert longest >= 3 * vec, (name, ops)


@pytest.mark.parametrize("H,T,k,vec", [
    # A vector per thread as long as the longer ones leave compute units idle.
    (7168, 48, 8, 1), (7168, 256, 2, 1), (4096, 256, 6, 1), (7168, 512, 8, 1), (16384, 128, 5, 1), (8, 1, 1, 1),
    # Past that; a row with a nearly empty second part was spread up to 511 tokens before, 1.3 times slower.
    (2056, 257, 6, 2), (2056, 257, 8, 2), (4096, 4096, 2, 2), (7168, 257, 7, 4), (7168, 513, 9, 4), (16384, 129, 5, 4),
    # Rows of one vector per thread are never split further.
    (2048, 1, 8, 1), (2048, 8192, 8, 1),
])
def test_combine_split_at_its_lines(combine_vec, H, T, k, vec):
    assert combine_vec(T, k, H) == vec


@pytest.fixture(scope="module")
def combine_vec(tmp_path_factory):
    d = tmp_path_factory.mktemp("split")
    (d / "split.cpp").write_text('#include "combine_split.hpp"\n'
                                 'extern "C" int f(long T, int k, int H) { return moe::combine_vec(T, k, H); }\n')
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", f"-I{CSRC}", str(d / "split.cpp"), "-o",
                    str(d / "split.so")], check=True, capture_output=True)
    fn = ctypes.CDLL(str(d / "split.so")).f
    fn.argtypes = [ctypes.c_long, ctypes.c_int, ctypes.c_int]
    return fn


def test_consumer_leaves_lds_to_the_producer(kernels):
    """A producer workgroup takes all of a CU's LDS; a consumer workgroup holding any LDS would
    keep producer workgroups off the compute units the two are meant to share."""
    for cons in by_name(kernels, "consumer_kernel").values():
        assert int(cons["group_segment_fixed_size"]) == 0
    for name, f in by_name(kernels, "producer_kernel").items():
        assert int(f["group_segment_fixed_size"]) == 160 * 1024, name


def test_tail_kernel_fits_beside_the_polling_consumer(kernels):
    """The tail kernel runs while the consumer polls on shared CUs: it holds no LDS (so no
    workgroup waits for LDS it holds) and at most 128 vector registers per wave."""
    (tail,) = by_name(kernels, "tail_kernel").values()
    assert int(tail["group_segment_fixed_size"]) == 0
    assert int(tail["vgpr_count"]) <= 128


def test_device_planner_kernels_present_and_small(kernels):
    """The planner kernels, the four phases and the one for small plans: single-workgroup ones stay within the 160 KiB of LDS a workgroup
    may hold on gfx950, grid ones use little."""
    names = {n.split("_kernel")[0].rsplit("plan_", 1)[1]: f for n, f in by_name(kernels, "plan_").items()
             if "_kernel" in n}
    assert set(names) == {"rows", "layout", "fill", "segs", "small"}, names
    for part, f in names.items():
        lds = int(f["group_segment_fixed_size"])
        assert lds <= 160 * 1024, (part, lds)
        if part in ("rows", "fill"):
            assert lds <= 32 * 1024, (part, lds)
