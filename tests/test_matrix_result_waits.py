"""The waits between the matrix instructions of the built library and their neighbours.

A matrix instruction delivers its result a fixed number of issue slots later, and nothing but
the distance to the next use of those registers makes that use wait.  The compiler keeps the
distance for its own matrix instructions but does not look into inline assembly, where most of
the ones here are written; it also puts register copies wherever it needs them.  So the distance
is checked in the code that was built: every path of every kernel, from each bf16 matrix
instruction to the next use of its result, and from each vector instruction to the matrix
instruction (or, behind a transcendental, the vector instruction) that reads its result.
The distances are the ones the compiler keeps for its own: 8 slots behind 16x16x32, 12 behind
32x32x16, 2 in front of a matrix instruction, 1 behind a transcendental.
"""

import os
import re
import shutil
import subprocess

import pytest

from paper_2602_02579_amd import api

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
RESULT = {"v_mfma_f32_16x16x32_bf16": 8, "v_mfma_f32_32x32x16_bf16": 12}
TRANSCENDENTAL = ("v_exp_", "v_log_", "v_rcp_", "v_rsq_", "v_sqrt_", "v_sin_", "v_cos_")
REG = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)")
LINE = re.compile(r"^\t(\S+)\s*(.*?)\s*// ([0-9A-F]+):[ 0-9A-F]*(?:<[^>+]*(?:\+0x([0-9a-f]+))?>)?")


def registers(text):
    out = []
    for kind, lo, hi, one in REG.findall(text):
        out += [(kind, i) for i in range(int(lo), int(hi) + 1)] if lo else [(kind, int(one))]
    return out


def kernels(listing):
    """name -> [(address, opcode, operands, branch target or None)]"""
    out, name, base = {}, None, 0
    for line in listing.splitlines():
        head = re.match(r"^([0-9a-f]+) <(.+)>:$", line)
        if head:
            base, name = int(head[1], 16), head[2]
            out[name] = []
            continue
        m = LINE.match(line)
        if not m or name is None:
            continue
        target = None
        if m[1] == "s_branch" or m[1].startswith("s_cbranch"):
            target = base + int(m[4] or "0", 16)
        out[name].append((int(m[3], 16), m[1], m[2], target))
    return out


def decode(op, operands):
    """(registers read, registers written, operands are matrix A and B, slots it takes)"""
    parts = [p.strip() for p in re.split(r",(?![^\[]*\])", operands)]
    if op == "s_nop":
        return [], [], int(operands, 0) + 1
    if not op.startswith(("v_", "ds_", "global_", "buffer_", "flat_", "scratch_")):
        return [], [], 1
    if op.startswith("v_mfma"):
        # the accumulator operand may be the running result of another matrix instruction
        return registers(parts[1]) + registers(parts[2]), registers(parts[0]), 1
    if "store" in op or "write" in op or "lds" in op or "atomic" in op or op.startswith("ds_add"):
        if not op.startswith("v_"):
            return registers(operands), [], 1
    return registers(",".join(parts[1:])), registers(parts[0]), 1


def too_close(code):
    """[(address, instruction, register, slots there, slots needed)] of one kernel"""
    at = {a: i for i, (a, _, _, _) in enumerate(code)}
    steps = [decode(op, ops) for _, op, ops, _ in code]
    leaders = {0} | {at[t] for _, _, _, t in code if t in at}
    # state: (register, who wrote it) -> slots since; who: "matrix", "vector", "trans"
    seen, work, bad = {0: {}}, [0], {}
    while work:
        i = start = work.pop()
        clock = 0
        state = {k: (-age, need) for k, (age, need) in seen[start].items()}   # time written

        def leave(to):
            new = {k: (min(clock - t, 16), n) for k, (t, n) in state.items() if clock - t < 16}
            old = seen.get(to)
            if old is None:
                seen[to] = new
            else:
                closer = {k: v for k, v in new.items() if k not in old or old[k][0] > v[0]}
                if not closer:
                    return
                old.update(closer)
            work.append(to)
        while i < len(code):
            if i in leaders and i != start:
                leave(i)
                break
            addr, op, ops, target = code[i]
            reads, writes, slots = steps[i]
            matrix, vector = op.startswith("v_mfma"), op.startswith("v_")
            trans = op.startswith(TRANSCENDENTAL)

            def check(reg, who):
                hit = state.get((reg, who))
                if hit and clock - hit[0] < hit[1]:
                    bad[addr, reg] = (addr, f"{op} {ops}", reg, clock - hit[0], hit[1])
            for r in reads:
                check(r, "matrix")
                if matrix:
                    check(r, "vector")
                elif vector and not trans:
                    check(r, "trans")
            if matrix:
                for r in registers(ops.rsplit(",", 1)[-1] if "]" not in ops else
                                   re.split(r",(?![^\[]*\])", ops)[3]):
                    check(r, "vector")
            else:
                for r in writes:
                    check(r, "matrix")
            clock += slots
            for r in writes:
                for who in ("matrix", "vector", "trans"):
                    state.pop((r, who), None)
                if matrix:
                    if op in RESULT:
                        state[r, "matrix"] = (clock, RESULT[op])
                elif vector:
                    state[r, "vector"] = (clock, 2)
                    if trans:
                        state[r, "trans"] = (clock, 1)
            if target is not None and target in at:
                leave(at[target])
            if op in ("s_branch", "s_endpgm", "s_setpc_b64"):
                break
            i += 1
    return list(bad.values())


def test_checker_finds_a_read_that_comes_too_early():
    lines = ["v_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]", "s_nop 5",
             "v_accvgpr_read_b32 v8, a3", "v_exp_f32_e32 v9, v8", "v_add_f32_e32 v10, v9, v9",
             "v_mov_b32_e32 v0, v10", "s_nop 0",
             "v_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]", "s_endpgm"]
    code = [(4 * i, *line.split(" ", 1), None) if " " in line else (4 * i, line, "", None)
            for i, line in enumerate(lines)]
    assert [(b[0], b[3], b[4]) for b in too_close(code)] == [(8, 6, 8), (16, 0, 1), (28, 1, 2)]


def test_matrix_results_are_not_used_too_early(tmp_path):
    if not os.path.exists(api.library_path()):
        pytest.skip("libpkv.so not built")
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    lib = shutil.copy(api.library_path(), tmp_path)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, capture_output=True)
    with_matrix, bad = 0, []
    for part in sorted(os.listdir(tmp_path)):
        if not part.endswith("gfx950"):
            continue
        listing = subprocess.run([OBJDUMP, "-d", str(tmp_path / part)], check=True,
                                 capture_output=True, text=True).stdout
        for name, code in kernels(listing).items():
            if any(op in RESULT for _, op, _, _ in code):
                with_matrix += 1
                bad += [(name, *b) for b in too_close(code)]
    assert with_matrix >= 20
    assert not bad, "\n".join(f"{n} {a:x}: {t}: {r[0]}{r[1]} after {d} of {w} slots"
                              for n, a, t, r, d, w in bad[:20])
