"""Distances that the chain kernels' inline assembly has to keep by itself.

gfx950 does not wait for them and the compiler, which adds waits between its own
instructions, does not see into an asm block: a vector instruction that reads
VCC (an addition with carry) needs two instructions or wait states after the
vector instruction that wrote it, and one with a DPP operand needs two after
the one that wrote the operand.  The kernels are compiled to assembly and every
such pair is looked at, in the order the code lies in, the compiler's own
instructions included.

The chain kernels' rounds are also placed on purpose (8-byte instructions from
an 8-byte boundary on, see place_code in the sources), which is checked here on
the encodings."""
import os
import re
import subprocess

import pytest

from paper_2510_23938_amd import build as B

MC = os.path.join(os.path.dirname(os.path.realpath(B.HIPCC)), "..", "llvm", "bin", "llvm-mc")
WAIT_STATES = 2


def registers(operand):
    """VGPR numbers an operand names."""
    m = re.fullmatch(r"v(\d+)", operand)
    if m:
        return {int(m.group(1))}
    m = re.fullmatch(r"v\[(\d+):(\d+)\]", operand)
    return set(range(int(m.group(1)), int(m.group(2)) + 1)) if m else set()


def operands(text):
    return [x.strip() for x in text.split(None, 1)[1].split(" quad_perm")[0].split(",")] if " " in text else []


def writes_vcc(name, ops):
    return "vcc" in ops[:2] or (name.startswith("v_cmp") and name.endswith("_e32"))


def reads_vcc(name, ops):
    return "vcc" in ops[2:] or (name.startswith("v_cndmask") and not name.endswith("_e64"))


def short_distances(lines):
    """(line number, text) of every vector instruction too close behind what it depends on."""
    found, checked = [], 0
    vcc_age, age = 99, {}  # wait states since VCC, and each VGPR, was written by a vector instruction
    for number, (text, _) in enumerate(lines):
        name = text.split()[0]
        ops = operands(text)
        if name.startswith("v_"):
            if reads_vcc(name, ops):
                checked += 1
                if vcc_age < WAIT_STATES:
                    found.append((number, text))
            if "quad_perm" in text or "row_" in text:
                checked += 1
                source = ops[2] if "vcc" in ops[:2] else ops[1]  # the first source is the DPP one
                assert registers(source), text
                if any(age.get(r, 99) < WAIT_STATES for r in registers(source)):
                    found.append((number, text))
        passed = int(text.split()[1]) + 1 if name == "s_nop" else 1
        vcc_age += passed
        age = {r: a + passed for r, a in age.items() if a + passed < WAIT_STATES}
        if name.startswith("v_"):
            if writes_vcc(name, ops):
                vcc_age = 0
            for r in registers(ops[0]):
                age[r] = 0
    return found, checked


def functions(listing):
    """{name: [(text, bytes)]} of an llvm-mc listing; an alignment to 8 bytes inside a function is (".p2align", 0)."""
    out, name = {}, None
    for line in listing.splitlines():
        m = re.match(r"(_Z\w+):", line)
        if m:
            name = m.group(1)
            out[name] = []
        text = line.split("; encoding:")[0].strip()
        m = re.search(r"; encoding: \[(.*)\]", line)
        if name and m:
            out[name].append((text, m.group(1).count(",") + 1))
        elif name and re.fullmatch(r"\.p2align\s+3", text):
            out[name].append((".p2align", 0))
        elif text.startswith(".amdhsa_kernel"):
            name = None
    return out


@pytest.fixture(scope="module", params=["sha256_split.hip", "sha384_split.hip"])
def kernels(request, tmp_path_factory):
    asm = tmp_path_factory.mktemp("isa") / "kernels.txt"
    src = os.path.join(B.CSRC, request.param)
    subprocess.run([B.HIPCC, *[f for f in B.FLAGS if f != "-fPIC"], "-x", "hip", "-S", "--cuda-device-only", src,
                    "-o", str(asm)], check=True, capture_output=True)
    listing = subprocess.run([MC, "-triple=amdgcn-amd-amdhsa", "-mcpu=gfx950", "-show-encoding", str(asm)], check=True,
                             capture_output=True, text=True).stdout
    return {k: v for k, v in functions(listing).items() if v}


def test_distances(kernels):
    checked = 0
    for name, lines in kernels.items():
        found, n = short_distances([x for x in lines if x[1]])
        assert not found, (name, len(found), found[:5])
        checked += n
    assert checked > 100  # the rounds' additions were among them


def test_rounds_keep_their_place(kernels):
    runs = 0
    for name, lines in kernels.items():
        if "chain_kernel" not in name:
            continue
        marks = [i for i, (text, _) in enumerate(lines) if text == ".p2align"]
        for start, end in zip(marks, marks[1:] + [len(lines)]):
            run = lines[start + 1:end]
            stop = next((i for i, (text, _) in enumerate(run) if text.startswith(("s_cbranch", "s_branch"))), len(run))
            run = run[:stop]
            while run and run[0][0] == "s_nop 0":  # off the boundary on purpose
                run = run[1:]
            if len(run) < 200:
                continue
            runs += 1
            body = run[:len(run) - 25]  # the last step meets the next block's reads and counters
            assert all(size == 8 for _, size in body), (name, [x for x in body if x[1] != 8][:5])
    assert runs >= 4


def test_the_distances_are_seen():
    """The checks themselves, on a few lines each."""
    write = "v_add_co_u32_dpp v1, vcc, v2, v3 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf"
    read = "v_addc_co_u32_dpp v4, vcc, v5, v6, vcc quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf"
    other = "v_xor_b32_e32 v9, v10, v11"

    def bad(*texts):
        return [t for _, t in short_distances([(t, 8) for t in texts])[0]]

    assert bad(write, read) == [read]
    assert bad(write, other, read) == [read]
    assert bad(write, "s_nop 0", read) == [read]
    assert bad(write, "s_nop 1", read) == [] and bad(write, other, other, read) == []
    assert bad("v_mov_b32_e32 v2, v8", write) == [write]
    assert bad("v_lshl_add_u64 v[2:3], v[4:5], 0, v[6:7]", other, write) == [write]
    assert bad("v_mov_b32_e32 v2, v8", other, other, write) == []
    assert bad("v_mov_b32_e32 v3, v8", write) == []  # the second source is no DPP operand
    assert bad("v_cmp_lt_u32_e32 vcc, s3, v7", "v_cndmask_b32_e32 v1, v2, v3, vcc") != []
