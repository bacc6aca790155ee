"""Static check of the generated gfx950 assembly (CPU only, needs hipcc).

The pipelined and the decode kernels issue their MFMAs through inline assembly, so the compiler
does not add the wait states the hardware needs between a vector instruction
that writes a VGPR/AccVGPR and an MFMA that reads it (two wait states on this
family), nor does it know that a vector instruction which reads an MFMA's result
has to wait until the MFMA has finished.  This test compiles the kernels to assembly
and verifies (1) that none of the two instructions in front of any MFMA is a
vector-ALU write to one of the MFMA's source registers, and (2) that no instruction
other than an MFMA reads an MFMA's destination registers within kResultWait wait
states after it, along every path of the control flow.  Both kernels address LDS with absolute byte addresses, so
they must not own any static LDS either.
"""
import os
import re
import shutil
import subprocess

import pytest

from paper_2512_10411_amd import build

# source file, substring of the kernel that addresses LDS absolutely, fewest MFMAs expected
CASES = [("swaa_fwd_pipelined.hip", "pipelined", 60), ("swaa_decode.hip", "decode_split", 16), ("swaa_fwd_short.hip", "fwd_short", 16),
         ("swaa_bwd_dq_pipelined.hip", "dq_pipelined", 100)]


def reg_set(tok):
    """'v[4:7]' -> {('v',4),...}; 'a12' -> {('a',12)}; others -> empty."""
    m = re.fullmatch(r"([va])\[(\d+):(\d+)\]", tok)
    if m:
        return {(m.group(1), i) for i in range(int(m.group(2)), int(m.group(3)) + 1)}
    m = re.fullmatch(r"([va])(\d+)", tok)
    if m:
        return {(m.group(1), int(m.group(2)))}
    return set()


def parse(line):
    line = line.split(";")[0].strip()
    if not line or line.endswith(":") or line.startswith("."):
        return None
    parts = line.split(None, 1)
    op = parts[0]
    ops = [t.strip() for t in parts[1].split(",")] if len(parts) > 1 else []
    return op, ops


# wait states after an MFMA before its result may be touched (the 8-pass MFMAs used here
# need 11; the kernels wait 24); an MFMA in between counts as kMfmaIssue, since the matrix
# pipe takes MFMAs in order and finishes each before the one after next starts
kResultWait = 18
kMfmaIssue = 8


def reads_and_writes(op, ops):
    """(registers read, registers written) of a non-MFMA instruction, conservatively."""
    if not ops:
        return set(), set()
    all_regs = set().union(*[reg_set(t) for t in ops])
    store_like = op.startswith(("ds_write", "global_store", "buffer_store", "scratch_store", "v_cmp", "global_load_lds",
                                "v_readfirstlane", "v_readlane"))
    read_modify_write = op.startswith(("v_fmac", "v_mac", "v_permlane", "v_pk_fmac", "v_dot2c", "v_writelane"))
    if store_like:
        return all_regs, set()
    dst = reg_set(ops[0])
    if read_modify_write:
        return all_regs, dst
    return set().union(*[reg_set(t) for t in ops[1:]]) if len(ops) > 1 else set(), dst


def result_hazards(insts, labels):
    """Rule (2): [(mfma, offender)] over all paths within the wait window.  A register that
    another instruction overwrites first no longer holds the MFMA's result and is dropped."""
    problems = []

    def walk(j, dst, ws, mfma, depth):
        dst = set(dst)
        while ws < kResultWait and j < len(insts) and dst:
            op, ops = insts[j]
            if op == "s_endpgm":
                return
            if op.startswith("v_mfma"):
                ws += kMfmaIssue
            elif op == "s_nop":
                ws += int(ops[0]) + 1
            elif op == "s_branch":
                j = labels[ops[0]]
                ws += 1
                continue
            elif op.startswith("s_cbranch"):
                if depth < 4:
                    walk(labels[ops[0]], dst, ws + 1, mfma, depth + 1)
                ws += 1
            else:
                reads, writes = reads_and_writes(op, ops)
                if reads & dst:
                    problems.append((mfma, insts[j]))
                    return
                dst -= writes
                ws += 1
            j += 1

    for i, (op, ops) in enumerate(insts):
        if op.startswith("v_mfma"):
            walk(i + 1, reg_set(ops[0]), 0, insts[i], 0)
    return problems


def is_valu_write(op):
    return op.startswith("v_") and not op.startswith("v_mfma") and not op.startswith("v_cmp") and \
        not op.startswith("v_nop")


@pytest.mark.skipif(shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"),
                    reason="hipcc not available")
@pytest.mark.parametrize("src,kernel,min_mfma", CASES)
def test_no_vector_write_within_two_instructions_of_an_mfma_that_reads_it(tmp_path, src, kernel, min_mfma):
    SRC = os.path.join(build.CSRC, src)
    out = tmp_path / "k.s"
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    cmd = [build.hipcc_path(), *flags, "--cuda-device-only", "-S", "-o", str(out), SRC]
    subprocess.run(cmd, check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    text = open(out).read()
    # the kernel addresses LDS absolutely, so its dynamic LDS must start at address 0
    sizes = re.findall(r"\.amdhsa_group_segment_fixed_size\s+(\d+)", text)
    names = re.findall(r"\.amdhsa_kernel\s+(\S+)", text)
    assert names and len(sizes) == len(names)
    for name, size in zip(names, sizes):
        if kernel in name:
            assert int(size) == 0, (name, size)
    assert any(kernel in name for name in names)
    insts, labels = [], {}
    for ln in text.splitlines():
        m = re.match(r"^(\.LBB\d+_\d+):", ln)
        if m:
            labels[m.group(1)] = len(insts)
        p = parse(ln)
        if p:
            insts.append(p)
    n_mfma = 0
    problems = []
    for i, (op, ops) in enumerate(insts):
        if not op.startswith("v_mfma"):
            continue
        n_mfma += 1
        srcs = set().union(*[reg_set(t) for t in ops[1:]])
        wait_states = 0
        for back in (1, 2, 3):
            if i - back < 0 or wait_states >= 2:
                break
            pop, pops = insts[i - back]
            if pop == "s_nop":
                wait_states += int(pops[0]) + 1
                continue
            if is_valu_write(pop) and pops and (reg_set(pops[0]) & srcs):
                problems.append((insts[i - back], insts[i]))
            wait_states += 1
    assert n_mfma >= min_mfma, "expected the MFMA kernel in the assembly"
    assert not problems, problems[:5]
    late = result_hazards(insts, labels)
    assert not late, late[:5]


@pytest.mark.skipif(shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"),
                    reason="hipcc not available")
@pytest.mark.parametrize("src,kernels", [
    ("swaa_bwd.hip", ("dkv_dma_kernel", "dkv_dma_short", "bwd_dkv_kernelILi64", "bwd_dq_kernel", "bwd_dq64_short")),
    ("swaa_fwd_d64.hip", ("fwd_d64_kernel", "fwd_d64_short")), ("swaa_bwd_dq_pipelined.hip", ("bwd_dq_pipelined", "bwd_dq_short")),
    ("swaa_fwd_short.hip", ("fwd_short",))])
def test_lds_dma_kernels_own_all_lds(tmp_path, src, kernels):
    """These LDS-DMA kernels address LDS with plain byte addresses from 0, too.  (The MFMAs of swaa_bwd.hip but dkv_dma_kernel's, which
    the next test looks at, and of swaa_fwd_d64.hip go through compiler builtins: the wait-state rules above are the compiler's there.)"""
    out = tmp_path / "b.s"
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    cmd = [build.hipcc_path(), *flags, "--cuda-device-only", "-S", "-o", str(out), os.path.join(build.CSRC, src)]
    subprocess.run(cmd, check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    text = open(out).read()
    sizes = re.findall(r"\.amdhsa_group_segment_fixed_size\s+(\d+)", text)
    spills = re.findall(r"\.amdhsa_private_segment_fixed_size\s+(\d+)", text)
    names = re.findall(r"\.amdhsa_kernel\s+(\S+)", text)
    assert names and len(sizes) == len(names) == len(spills)
    seen = set()
    for name, size, spill in zip(names, sizes, spills):
        for k in kernels:
            if k in name:
                seen.add(k)
                assert int(size) == 0, (name, size)
                # and no spills (their reloads would wait for the copies, inside the loop)
                assert int(spill) == 0, (name, spill)
    assert seen == set(kernels)


@pytest.mark.skipif(shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"),
                    reason="hipcc not available")
def test_dkv_kernel_of_head_dimension_128_keeps_the_wait_states_and_its_accumulators(tmp_path):
    """swaa_bwd_dkv_dma_kernel names its 256 accumulator registers in the instructions: nothing else may live
    there (not even for a moment), and the two rules above hold for its MFMAs."""
    out = tmp_path / "b.s"
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    cmd = [build.hipcc_path(), *flags, "--cuda-device-only", "-S", "-o", str(out), os.path.join(build.CSRC, "swaa_bwd.hip")]
    subprocess.run(cmd, check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    lines = open(out).read().splitlines()
    first = next(i for i, ln in enumerate(lines) if re.match(r"_Z\S*dkv_dma_kernel\S*:", ln))
    insts, labels, written_out = [], {}, []  # written_out: does the instruction come from inline assembly?
    inside = False
    for ln in lines[first:next(i for i in range(first, len(lines)) if lines[i].startswith(".Lfunc_end"))]:
        inside = (inside or "#ASMSTART" in ln) and "#ASMEND" not in ln
        m = re.match(r"^(\.LBB\d+_\d+):", ln)
        if m:
            labels[m.group(1)] = len(insts)
        p = parse(ln)
        if p:
            insts.append(p)
            written_out.append(inside)
    mfmas = [i for i, (op, _) in enumerate(insts) if op.startswith("v_mfma")]
    assert len(mfmas) >= 140  # a prologue of 16 and two versions of a step
    for i, (op, ops) in enumerate(insts):
        if written_out[i]:
            continue
        assert not any(r[0] == "a" for t in ops for r in reg_set(t)), insts[i]
        assert not op.startswith("scratch_"), insts[i]
    for i in mfmas:
        srcs = set().union(*[reg_set(t) for t in insts[i][1][1:]])
        wait_states = 0
        for pop, pops in reversed(insts[max(0, i - 3):i]):
            if wait_states >= 2:
                break
            assert not (is_valu_write(pop) and pops and reg_set(pops[0]) & srcs), ((pop, pops), insts[i])
            wait_states += int(pops[0]) + 1 if pop == "s_nop" else 1
    late = result_hazards(insts, labels)
    assert not late, late[:5]


@pytest.mark.skipif(shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"),
                    reason="hipcc not available")
def test_dkv_kernel_of_head_dimension_64_keeps_the_wait_states(tmp_path):
    """The two rules above for swaa_bwd_dkv_kernel<64>, whose file holds kernels of compiler builtins as well."""
    out = tmp_path / "b.s"
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    cmd = [build.hipcc_path(), *flags, "--cuda-device-only", "-S", "-o", str(out), os.path.join(build.CSRC, "swaa_bwd.hip")]
    subprocess.run(cmd, check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    lines = open(out).read().splitlines()
    first = next(i for i, ln in enumerate(lines) if re.match(r"_Z\S*bwd_dkv_kernelILi64\S*:", ln))
    insts, labels = [], {}
    for ln in lines[first:next(i for i in range(first, len(lines)) if lines[i].startswith(".Lfunc_end"))]:
        m = re.match(r"^(\.LBB\d+_\d+):", ln)
        if m:
            labels[m.group(1)] = len(insts)
        p = parse(ln)
        if p:
            insts.append(p)
    mfmas = [i for i, (op, _) in enumerate(insts) if op.startswith("v_mfma")]
    assert len(mfmas) == 48  # the first block's scores, two sub-steps, the last block's sums
    for i in mfmas:
        srcs = set().union(*[reg_set(t) for t in insts[i][1][1:]])
        wait_states = 0
        for pop, pops in reversed(insts[max(0, i - 3):i]):
            if wait_states >= 2:
                break
            assert not (is_valu_write(pop) and pops and reg_set(pops[0]) & srcs), ((pop, pops), insts[i])
            wait_states += int(pops[0]) + 1 if pop == "s_nop" else 1
    late = result_hazards(insts, labels)
    assert not late, late[:5]


@pytest.mark.skipif(shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"),
                    reason="hipcc not available")
@pytest.mark.parametrize("src,kernel", [("swaa_bwd.hip", "bwd_dq_kernel"), ("swaa_fwd_d64.hip", "fwd_d64_kernel")])
def test_tile_buffers_are_reused_behind_a_wait_for_their_reads(tmp_path, src, kernel):
    """Two buffers, one barrier per tile: behind it the buffer of the tile before is copied into.  A wave's copies must have
    landed in front of that barrier (vmcnt), and so must its reads of that buffer (lgkmcnt): their MFMAs are compiler builtins,
    which the barrier does not hold back."""
    out = tmp_path / "k.s"
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    cmd = [build.hipcc_path(), *flags, "--cuda-device-only", "-S", "-o", str(out), os.path.join(build.CSRC, src)]
    subprocess.run(cmd, check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    lines = open(out).read().splitlines()
    starts = [i for i, ln in enumerate(lines) if re.match(r"_Z\S*" + kernel + r"\S*:", ln)]
    assert starts
    for first in starts:
        insts = [parse(ln) for ln in lines[first:next(i for i in range(first, len(lines)) if lines[i].startswith(".Lfunc_end"))]]
        insts = [(op, " ".join(ops)) for op, ops in filter(None, insts)]
        barriers = [i for i, (op, _) in enumerate(insts) if op == "s_barrier"]
        assert len(barriers) == 1  # the one at the top of the loop over the tiles
        op, counters = insts[barriers[0] - 1]
        assert op == "s_waitcnt" and "vmcnt(0)" in counters and "lgkmcnt(0)" in counters, (op, counters)


@pytest.mark.parametrize("src", sorted(f for f in os.listdir(build.CSRC) if f.endswith((".hip", ".h"))))
def test_loads_written_in_assembly_are_waited_for_and_taken(src):
    """A load in inline assembly writes its register whenever it arrives, and the compiler thinks it written at once: the same block has
    to wait for it, and a statement has to take what it loads.  (Copies straight to LDS have no register to write.)"""
    text = open(os.path.join(build.CSRC, src)).read()
    for m in re.finditer(r"\basm\b(?: volatile)?\s*\((.*?)\);", text, re.S):
        block = m.group(1)
        loads = re.findall(r"\b(?:s_load|s_buffer_load|global_load|flat_load|buffer_load|scratch_load|ds_read|ds_load)_(?!lds)\w+", block)
        if not loads:
            continue
        assert "s_waitcnt" in block.split(loads[-1])[-1], (src, block)
        outputs = re.findall(r'"=&?[svagr]+"\((\w+)\)', block)
        assert outputs and all(re.search(r'\(' + name + r'\)', text[m.end():m.end() + 400]) for name in outputs), (src, block)
