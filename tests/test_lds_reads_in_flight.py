"""The GEMM kernels issue their LDS reads and MFMAs as asm statements, which the compiler takes to be done at once.  What it places between such a
statement and the wait for it -- a copy of a fragment at a loop's head, another value in the register of a fragment that is not used any more -- is
wrong only now and then on the GPU, so it is looked for here, in the compiled code: data flow over each kernel's control-flow graph of the registers that LDS
reads are still to write, and of the accumulators that an MFMA is still to write.  (CPU only.)"""
import os
import re
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2203_10991_amd import build

SOURCES = ["gemm_conv", "gemm_dense", "gemm_f32_split", "gemm_smfmac", "gemm_smfmac_q8", "gemm_smfmac_small"]
REGISTER = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)")
MFMA_WAIT_STATES = 20                # instructions (s_nop n: n + 1) behind the longest MFMA, of 16 passes, until its result may be read or overwritten


def _registers(text):
    out = set()
    for kind, first, last, one in REGISTER.findall(text):
        out |= {(kind, int(one))} if one else {(kind, i) for i in range(int(first), int(last) + 1)}
    return out


def _blocks(lines):
    """basic blocks of (line number, instruction, written as asm), and the numbers of their successors"""
    blocks, label, asm = [[]], {}, False
    for number, line in lines:
        asm = (asm or "#ASMSTART" in line) and "#ASMEND" not in line
        target = re.match(r"(\.L\w+):", line)
        text = line.split(";")[0].strip()
        if target:
            blocks.append([])
            label[target.group(1)] = len(blocks) - 1
        elif text and not text.startswith(".") and not text.endswith(":"):
            blocks[-1].append((number, text, asm))
            if text.startswith(("s_branch", "s_cbranch", "s_endpgm")):
                blocks.append([])
    after = []
    for i, b in enumerate(blocks):
        last = b[-1][1] if b else ""
        # (where a block has not changed the mask of its lanes, some are there: a way round uniform code that the compiler could as well have left out)
        lanes = "s_cbranch_exec" in last and not any("exec" in text for _, text, _ in b[:-1])
        jumps, falls = last.startswith(("s_branch", "s_cbranch")), not last.startswith(("s_branch", "s_endpgm"))
        if lanes:
            jumps, falls = "execnz" in last, "execz" in last
        to = [label[last.split()[1]]] if jumps else []
        if falls and i + 1 < len(blocks):
            to.append(i + 1)
        after.append(to)
    return blocks, after


def _through(block, reads, sums, found=None):
    """reads: register -> LDS operations issued behind the one that writes it; sums: register -> wait states behind its MFMA"""
    reads, sums = dict(reads), dict(sums)
    for number, text, asm in block:
        op = text.split()[0]
        touched = _registers(text)
        states = int(text.split()[1], 0) + 1 if op == "s_nop" else 1
        if op.startswith("s_waitcnt"):
            left = re.search(r"lgkmcnt\((\d+)\)", text)
            if left:
                reads = {r: n for r, n in reads.items() if n < int(left.group(1))}
        mfma, read = "mfma" in op or "smfmac" in op, asm and op.startswith("ds_read")
        written = _registers(text.split(",")[0]) if mfma or read else set()
        if found is not None:
            if not asm and touched & (reads.keys() | (set() if mfma else sums.keys())):
                found.append((number, text))
        if op.startswith("ds_"):
            reads = {r: n + 1 for r, n in reads.items()}
        sums = {r: n + states for r, n in sums.items() if n + states < MFMA_WAIT_STATES}
        if read:
            reads.update(dict.fromkeys(written, 0))
        if mfma and asm:
            sums.update(dict.fromkeys(written, 0))
    return reads, sums


def _touched_too_early(lines):
    blocks, after = _blocks(lines)
    entry, work = {0: ({}, {})}, [0]
    while work:
        i = work.pop()
        left = _through(blocks[i], *entry[i])
        for j in after[i]:
            known = entry.setdefault(j, None)
            if known is None:
                entry[j] = tuple(dict(x) for x in left)
                work.append(j)
                continue
            changed = False
            for have, new in zip(known, left):
                for r, n in new.items():
                    if n < have.get(r, 64):
                        have[r] = n
                        changed = True
            if changed:
                work.append(j)
    found = []
    for i, state in entry.items():
        _through(blocks[i], *state, found)
    return found


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc) and shutil.which(hipcc) is None:
        pytest.skip("needs hipcc")
    to = tmp_path_factory.mktemp("asm")

    def one(name):
        r = subprocess.run([hipcc, *build.HIPCC_FLAGS, "-S", "--cuda-device-only", os.path.join(build.CSRC, f"{name}.hip"),
                            "-o", str(to / f"{name}.s")], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        return (to / f"{name}.s").read_text().split("\n")
    with ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        return dict(zip(SOURCES, ex.map(one, SOURCES)))


@pytest.mark.parametrize("name", SOURCES)
def test_nothing_touches_a_register_before_its_asm_read_or_mfma_is_done(assembly, name):
    kernels, current = {}, None
    for number, line in enumerate(assembly[name], 1):
        start = re.match(r"(_Z\w+):", line)
        if start:
            current = kernels.setdefault(start.group(1), [])
        elif line.startswith(".Lfunc_end"):
            current = None
        elif current is not None:
            current.append((number, line))
    issued = [k for k, lines in kernels.items() if any("ds_read" in line for _, line in lines) and any("mfma" in line or "smfmac" in line for _, line in lines)]
    assert issued
    for k in issued:
        found = _touched_too_early(kernels[k])
        assert not found, f"{k}: {len(found)} instructions, first {found[:4]}"
