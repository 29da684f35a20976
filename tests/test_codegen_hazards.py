"""Orderings that the compiler does not keep by itself, checked in the assembly of the kernels that rely on them.

Matrix instructions written as inline assembly are opaque to the compiler's hazard bookkeeping: the code keeps the distance to
the instructions that touch their accumulators, and the compiler may move those unless something ties them down.  A bare
s_barrier does not wait for LDS writes: the code puts the wait in front of it.  Neither shows in a result reliably, so the
instruction streams are walked instead (every path, a few wait states deep).
"""
import concurrent.futures
import os
import re
import subprocess

import pytest

from paper_2601_17261_amd import build as B

SOURCES = ["gemm_bf16_aligned.hip", "gemm_bf16_mid.hip", "gemm_bf16_few.hip", "skinny.hip", "glue.hip", "probe.hip"]
# wait states this compiler keeps on gfx950 around v_mfma_f32_16x16x32_bf16 when it knows the instruction (through the
# builtin): 8 from the instruction to anything else that reads or writes its result, 2 from a vector instruction's result to it
AFTER_MFMA, BEFORE_MFMA = 8, 2
REG = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)")


def registers(operand):
    out = set()
    for kind, lo, hi, one in REG.findall(operand):
        out.update((kind, i) for i in (range(int(lo), int(hi) + 1) if lo else (int(one),)))
    return out


class Instr:
    def __init__(self, text, in_asm):
        self.text = text
        parts = text.split(None, 1)
        self.op = parts[0]
        ops = [o.strip() for o in parts[1].split(",")] if len(parts) > 1 else []
        self.in_asm = in_asm
        self.mfma = self.op.startswith("v_mfma")
        self.first = registers(ops[0]) if ops else set()
        self.all = registers(parts[1]) if len(parts) > 1 else set()
        self.rest = set().union(*(registers(o) for o in ops[1:])) if len(ops) > 1 else set()
        self.states = int(ops[0], 0) + 1 if self.op == "s_nop" else 1
        self.target = ops[-1] if self.op.startswith(("s_branch", "s_cbranch")) else None


def functions(asm):
    """{kernel name: (instructions, successors of each)}"""
    out = {}
    name, body, labels, in_asm = None, [], {}, False
    for raw in asm.splitlines():
        line = raw.split("//")[0].strip()
        if line.startswith((";;#ASMSTART", ";APP", ";#APP")):
            in_asm = True
        elif line.startswith((";;#ASMEND", ";NO_APP", ";#NO_APP")):
            in_asm = False
        line = line.split(";")[0].strip()
        m = re.match(r"^([\w.$]+):$", line)
        if m:
            if m.group(1).startswith("_Z"):
                name, body, labels = m.group(1), [], {}
            elif m.group(1).startswith(".Lfunc_end") and name:
                succ = []
                for i, ins in enumerate(body):
                    s = [] if ins.op in ("s_endpgm", "s_branch", "s_setpc_b64") or i + 1 == len(body) else [i + 1]
                    if ins.target:
                        s.append(labels[ins.target])
                    succ.append([t for t in s if t < len(body)])
                out[name] = (body, succ)
                name = None
            else:
                labels[m.group(1)] = len(body)
        elif name and line and not line.startswith("."):
            body.append(Instr(line, in_asm))
    return out


def reached(succ, body, start, limit):
    """instructions fewer than `limit` wait states behind `start`, on any path"""
    best, todo = {}, [(t, 0) for t in succ[start]]
    while todo:
        i, gap = todo.pop()
        if gap >= limit or best.get(i, limit) <= gap:
            continue
        best[i] = gap
        todo += [(t, gap + body[i].states) for t in succ[i]]
    return best


def wait_state_faults(body, succ):
    faults = []
    for i, ins in enumerate(body):
        if ins.mfma and ins.in_asm:
            for j, gap in reached(succ, body, i, AFTER_MFMA).items():
                if not body[j].mfma and body[j].all & ins.first:
                    faults.append("%s  --%d-->  %s" % (ins.text, gap, body[j].text))
        elif ins.op.startswith("v_") and not ins.mfma and ins.first:
            for j, gap in reached(succ, body, i, BEFORE_MFMA).items():
                if body[j].mfma and body[j].in_asm and body[j].rest & ins.first:
                    faults.append("%s  --%d-->  %s" % (ins.text, gap, body[j].text))
    return faults


def barrier_faults(body, succ):
    """LDS writes that may be under way at an s_barrier (no wait for them on some path between)"""
    faults, seen = [], set()
    todo = [(t, i) for i, ins in enumerate(body) if ins.op.startswith(("ds_write", "ds_add")) for t in succ[i]]
    while todo:
        i, src = todo.pop()
        if i in seen:
            continue
        seen.add(i)
        if body[i].op == "s_barrier":
            faults.append("%s  -->  s_barrier (instruction %d)" % (body[src].text, i))
            continue
        if body[i].op == "s_waitcnt" and "lgkmcnt(0)" in body[i].text:
            continue
        todo += [(t, src) for t in succ[i]]
    return faults


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    d = tmp_path_factory.mktemp("asm")

    def one(src):
        out = os.path.join(str(d), src.replace(".hip", ".s"))
        subprocess.run([B.HIPCC] + B.FLAGS + ["-S", "--cuda-device-only", os.path.join(B.CSRC, src), "-o", out], check=True, capture_output=True)
        with open(out) as f:
            return f.read()
    with concurrent.futures.ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        return dict(zip(SOURCES, ex.map(one, SOURCES)))


@pytest.fixture(scope="module")
def kernels(assembly):
    return {src: functions(text) for src, text in assembly.items()}


@pytest.mark.parametrize("src", SOURCES)
def test_results_of_written_out_matrix_instructions(kernels, src):
    found = {name: wait_state_faults(*f) for name, f in kernels[src].items()}
    written = any(ins.mfma and ins.in_asm for body, _ in kernels[src].values() for ins in body)
    assert written == (src in ("gemm_bf16_aligned.hip", "gemm_bf16_mid.hip", "probe.hip"))
    assert not any(found.values()), "\n".join("%s: %d, e.g. %s" % (n, len(v), v[0]) for n, v in found.items() if v)


@pytest.mark.parametrize("src", SOURCES)
def test_lds_writes_are_complete_at_barriers(kernels, src):
    found = {name: barrier_faults(*f) for name, f in kernels[src].items()}
    assert found
    assert not any(found.values()), "\n".join("%s: %s" % (n, v[0]) for n, v in found.items() if v)


def test_accumulators_stay_in_place(kernels):
    """X Q up to 32 columns: no moves between the halves of the register file in a loop over slices (a block of matrix instructions that
    branches back to its own start)"""
    found = 0
    for name, (body, succ) in kernels["skinny.hip"].items():
        if "xq_bf16_many_kernel" not in name:
            continue
        loops = [body[t:i + 1] for i, s in enumerate(succ) for t in s if t <= i]
        inner = [l for l in loops if sum(ins.mfma for ins in l) in (6, 12) and not any(ins.target for ins in l[:-1])]
        assert inner, name
        found += 1
        assert not [ins.text for l in inner for ins in l if ins.op.startswith("v_accvgpr")], name
    assert found == 12


def test_registers_of_the_persistent_kernel(assembly):
    """What the forms of gemm_bf16_aligned_kernel<OUT, T_F32, PHASES, RAGGED, CAP> spill: nothing for one evaluation, but for half an fp32
    tile of a ragged layer, whose 128 registers wait beside the next tile's first fragments"""
    limit = {("0", "1", "1", "1"): 118, ("0", "0", "3", "0"): 16, ("0", "1", "3", "0"): 16, ("0", "0", "3", "1"): 90, ("0", "1", "3", "1"): 90}
    found = re.findall(r"\.name:\s+\S*gemm_bf16_aligned_kernelILi(\d)ELb(\d)ELi(\d)ELb(\d)ELi\d+E\S*$.*?\.vgpr_spill_count:\s+(\d+)", assembly["gemm_bf16_aligned.hip"],
                       re.M | re.S)
    assert len(found) == 18
    for *form, spilled in found:
        assert int(spilled) <= limit.get(tuple(form), 0), (form, spilled)


def test_the_walk_finds_planted_faults():
    head, tail = "_Zk:\n", "\ts_endpgm\n.Lfunc_end0:\n"
    mfma = "\t;;#ASMSTART\n\tv_mfma_f32_16x16x32_bf16 a[0:3], v[4:7], v[8:11], a[0:3]\n\t;;#ASMEND\n"

    def walk(text, check):
        (f,) = functions(head + text + tail).values()
        return check(*f)
    read = "\tv_accvgpr_read_b32 v20, a2\n"
    assert len(walk(mfma + read, wait_state_faults)) == 1
    assert len(walk(mfma + "\ts_nop 6\n" + read, wait_state_faults)) == 1
    assert not walk(mfma + "\ts_nop 7\n" + read, wait_state_faults)
    assert len(walk(mfma + "\ts_cbranch_scc1 .LBB0_2\n\ts_nop 7\n.LBB0_2:\n" + read, wait_state_faults)) == 1      # by the branch
    assert not walk(mfma + "\tv_accvgpr_read_b32 v20, a4\n", wait_state_faults)
    assert len(walk("\tv_accvgpr_write_b32 a1, v3\n" + mfma, wait_state_faults)) == 1
    assert len(walk("\tds_write_b16 v1, v2\n\ts_waitcnt vmcnt(8)\n\ts_barrier\n", barrier_faults)) == 1
    assert not walk("\tds_write_b16 v1, v2\n\ts_waitcnt vmcnt(8) lgkmcnt(0)\n\ts_barrier\n", barrier_faults)
