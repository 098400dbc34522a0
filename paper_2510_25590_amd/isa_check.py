"""Static checks of the GEMM and attention kernels' machine code, run by every build.

The kernels issue global-to-LDS copies as inline assembly and wait for them by hand with `s_waitcnt vmcnt(N)`: the compiler
neither knows what the counts stand for nor waits itself.  `check_asm` proves on the generated code that (1) the K loops hold
no vector-memory instruction besides the counted copies and no kernel with such copies spills to scratch memory (spills share
the counter); (2) no wide store's data registers are overwritten by the next instruction; (3) registers that are the
destination of an assembly load are left alone until a wait covers them (`check_function`).  The kernels' assembly copies write LDS
only; (3) guards the step back to loads into registers, whose destinations the compiler takes as written at once.

Model of (3): loads complete in issue order.  Every destination register of an asm load is "pending" with an age = number
of vector-memory loads issued after it.  `s_waitcnt vmcnt(N)` lands every register whose age is at least N.  At a
join the state is the union of the predecessors' pending sets with the smaller age.  Any instruction that names a
pending register is a violation (the load's own address operand excepted).
"""
from __future__ import annotations

import os
import re
import subprocess
import tempfile

_REG_RANGE = re.compile(r"\bv\[(\d+):(\d+)\]")
_REG_ONE = re.compile(r"\bv(\d+)\b")
_LABEL = re.compile(r"^(\.LBB\d+_\d+):")
_VMCNT = re.compile(r"vmcnt\((\d+)\)")


def _regs(text: str) -> set[int]:
    out: set[int] = set()
    for a, b in _REG_RANGE.findall(text):
        out.update(range(int(a), int(b) + 1))
    for a in _REG_ONE.findall(text):
        out.add(int(a))
    return out


def _kernel_bodies(asm: str, name_part: str):
    """Yields (mangled name, lines) of every function whose name contains name_part."""
    lines = asm.splitlines()
    i = 0
    while i < len(lines):
        m = re.match(r"^(_Z\w+):", lines[i])
        if m and name_part in m.group(1):
            j = i + 1
            while j < len(lines) and not lines[j].startswith(".Lfunc_end"):
                j += 1
            yield m.group(1), lines[i + 1:j]
            i = j
        i += 1


def _blocks(lines):
    """Splits a function into basic blocks: list of (label or None, [(instr, in_asm)], successors by label / fallthrough)."""
    blocks, cur, label, in_asm = [], [], None, False
    for raw in lines:
        s = raw.strip()
        if not s or s.startswith(";") and not s.startswith(";;#ASM"):
            continue
        if s.startswith(";;#ASMSTART"):
            in_asm = True
            continue
        if s.startswith(";;#ASMEND"):
            in_asm = False
            continue
        m = _LABEL.match(s)
        if m:
            if cur or label is not None:
                blocks.append([label, cur, None])
            label, cur = m.group(1), []
            continue
        if s.startswith("."):
            continue
        instr = s.split(";")[0].strip()
        if not instr:
            continue
        cur.append((instr, in_asm))
        op = instr.split()[0]
        if op.startswith("s_cbranch") or op == "s_branch" or op == "s_endpgm":
            blocks.append([label, cur, None])
            label, cur = None, []
    if cur or label is not None:
        blocks.append([label, cur, None])
    index = {b[0]: k for k, b in enumerate(blocks) if b[0] is not None}
    for k, b in enumerate(blocks):
        succ = []
        last = b[1][-1][0] if b[1] else ""
        op = last.split()[0] if last else ""
        if op == "s_endpgm":
            pass
        elif op == "s_branch":
            succ.append(index[last.split()[1]])
        else:
            if op.startswith("s_cbranch"):
                succ.append(index[last.split()[1]])
            if k + 1 < len(blocks):
                succ.append(k + 1)
        b[2] = succ
    return blocks


def _transfer(state: dict[int, int], block, where: str, errors: list[str]) -> dict[int, int]:
    st = dict(state)
    for instr, in_asm in block[1]:
        op = instr.split()[0]
        if op == "s_waitcnt":
            m = _VMCNT.search(instr)
            if m:
                n = int(m.group(1))
                st = {r: a for r, a in st.items() if a < n}
            continue
        is_vmem_load = op.startswith("global_load") or op.startswith("buffer_load") or op.startswith("flat_load") or op.startswith("scratch_load")
        named = _regs(instr)
        if in_asm and op == "global_load_dwordx4":
            operands = instr[len(op):].split(",")
            dest, rest = _regs(operands[0]), _regs(",".join(operands[1:]))
            bad = (rest - dest) & st.keys() | dest & st.keys()
            if bad:
                errors.append(f"{where}: '{instr}' names registers of loads still in flight: v{sorted(bad)}")
            st = {r: a + 1 for r, a in st.items()}
            for r in dest:
                st[r] = 0
            continue
        bad = named & st.keys()
        if bad:
            errors.append(f"{where}: '{instr}' names registers of loads still in flight: v{sorted(bad)}")
            for r in bad:          # report once
                st.pop(r)
        if is_vmem_load:
            st = {r: a + 1 for r, a in st.items()}
    return st


def check_function(name: str, lines, unroll: int = 0) -> list[str]:
    """Data flow over (block, last step run).
    unroll = 0: every path of the control-flow graph is followed.
    unroll = n: the K loop is unrolled n times and its step blocks (those that hold both asm loads and MFMAs) run
    in their order in the text, step 0 first, when the source guarantees that.  Block merging by the compiler can
    leave edges in the graph that would skip or repeat a step; a path that enters a step block out of order cannot
    run and is not followed."""
    blocks = _blocks(lines)
    if not blocks:
        return [f"{name}: no code found"]
    short = name[:60]

    def has(b, pred):
        return any(pred(i, a) for i, a in b[1])
    steps = [k for k, b in enumerate(blocks)
             if has(b, lambda i, a: a and i.startswith("global_load_dwordx4")) and has(b, lambda i, a: i.startswith("v_mfma"))]
    if unroll and len(steps) != unroll:
        return [f"{short}: expected {unroll} K-step blocks (asm loads and MFMAs), found {len(steps)}: the check does not know this shape"]
    step_id = {k: n for n, k in enumerate(steps)} if unroll else {}

    errors: list[str] = []
    seen_err: set[str] = set()
    entry: dict[tuple[int, int], dict[int, int]] = {(0, -1): {}}
    work = [(0, -1)]
    rounds = 0
    reached_steps: set[int] = set()
    while work:
        rounds += 1
        if rounds > 200000:
            return [f"{short}: analysis did not converge"]
        k, tag = work.pop()
        errs: list[str] = []
        out = _transfer(entry[(k, tag)], blocks[k], f"{short} block {blocks[k][0] or k} (after step {tag})", errs)
        for e in errs:
            if e not in seen_err:
                seen_err.add(e)
                errors.append(e)
        out_tag = step_id.get(k, tag)
        if k in step_id:
            reached_steps.add(k)
        last = blocks[k][1][-1][0].split()[0] if blocks[k][1] else ""
        if last == "s_endpgm" and out:
            e = f"{short}: loads into v{sorted(out)} may still be in flight at s_endpgm"
            if e not in seen_err:
                seen_err.add(e)
                errors.append(e)
        for s in blocks[k][2]:
            if unroll and s in step_id and step_id[s] != (out_tag + 1) % unroll:
                continue   # out of order: not a path of the program
            old = entry.get((s, out_tag))
            if old is None:
                new = dict(out)
            else:
                new = dict(old)
                for r, a in out.items():
                    new[r] = min(a, old[r]) if r in old else a
            if new != old:
                entry[(s, out_tag)] = new
                work.append((s, out_tag))
    if unroll and len(reached_steps) != unroll:
        errors.append(f"{short}: only {len(reached_steps)} of {unroll} K-step blocks are reachable in order")
    return errors


_COPY = "global_load_lds_dwordx4"
_WIDE_STORE = re.compile(r"^(buffer|global)_store_dwordx[34]\b")


def check_copies(name: str, lines) -> list[str]:
    """The two-group kernels count their global-to-LDS copies by hand: inside a K loop (every basic block that runs MFMAs or
    such copies and is reached again from itself) no other vector-memory instruction may stand, or the counts are off."""
    blocks = _blocks(lines)
    short = name[:70]
    errors = []
    reach: list[set[int]] = []
    for k in range(len(blocks)):
        seen, work = set(), list(blocks[k][2])
        while work:
            b = work.pop()
            if b not in seen:
                seen.add(b)
                work += blocks[b][2]
        reach.append(seen)
    for k, b in enumerate(blocks):
        if k not in reach[k] or not any(i.startswith(_COPY) or i.startswith("v_mfma") for i, _ in b[1]):
            continue
        for instr, in_asm in b[1]:
            op = instr.split()[0]
            if re.match(r"^(global|buffer|flat|scratch)_(load|store|atomic)", op) and not (in_asm and op == _COPY):
                errors.append(f"{short} block {b[0] or k}: '{instr}' among the counted copies")
    return errors


def check_wide_stores(name: str, lines) -> list[str]:
    """A vector-memory store of more than eight bytes reads its data registers one wait state late; with a scalar offset
    register the compiler does not keep that distance.  No such store may be followed by a write of its data."""
    instrs = [i for b in _blocks(lines) for i, _ in b[1]]
    errors = []
    for cur, nxt in zip(instrs, instrs[1:]):
        if not _WIDE_STORE.match(cur) or not nxt.startswith("v_"):
            continue
        operands = cur.split(None, 1)[1].split(",")
        data = _regs(operands[0] if cur.startswith("buffer") else operands[1])
        if data & _regs(nxt.split(None, 1)[1].split(",")[0]):
            errors.append(f"{name[:70]}: '{nxt}' overwrites the data of '{cur}'")
    return errors


def check_asm(asm: str) -> None:
    """Checks every GEMM kernel of one translation unit's assembly; raises RuntimeError on a violation."""
    n = 0
    problems: list[str] = []
    for name, lines in _kernel_bodies(asm, "gemm_"):
        n += 1
        text = "\n".join(lines)
        if _COPY in text:
            m = re.search(r"; ScratchSize: (\d+)", asm[asm.index(name + ":"):])
            if m and int(m.group(1)) != 0:
                problems.append(f"{name[:70]}: uses {m.group(1)} bytes of scratch memory (its accesses share the copies' counter)")
            problems += check_copies(name, lines)
        problems += check_wide_stores(name, lines)
        problems += check_function(name, lines)
    if n == 0:
        problems.append("no GEMM kernel found in the assembly")
    if problems:
        raise RuntimeError("GEMM machine-code check failed:\n  " + "\n  ".join(problems[:20]))


def check_rounds(name: str, lines) -> list[str]:
    """The full rounds of the attention's two wave groups: basic blocks that run MFMAs and issue copies of key tiles.  What they wait for is counted by hand; spills and
    further loads share the counter and would make the waits stricter, never laxer, but a round with them is not the one that was measured.  So: no
    scratch access; no vector-memory access besides the copies but single index entries; and no wait that leaves more in flight than the
    copies of one round (the loop may be rotated, so that a round's wait opens the next block)."""
    short = name[:70]
    errors, rounds = [], 0
    for k, b in enumerate(_blocks(lines)):
        instrs = [i for i, _ in b[1]]
        copies = sum(i.startswith(_COPY) for i in instrs)
        if not copies or sum(i.startswith("v_mfma") for i in instrs) < 32:
            continue
        rounds += 1
        for instr in instrs:
            op = instr.split()[0]
            if re.match(r"^(global|buffer|flat|scratch)_(load|store|atomic)", op) and op not in (_COPY, "global_load_dword"):
                errors.append(f"{short} block {b[0] or k}: '{instr}' in a full round")
        left = [int(m.group(1)) for m in (_VMCNT.search(i) for i in instrs if i.startswith("s_waitcnt")) if m]
        if not left or max(left) > copies:
            errors.append(f"{short} block {b[0] or k}: {copies} copies, and waits that leave {left} in flight")
    if rounds == 0:
        errors.append(f"{short}: no full round found")
    return errors


def check_attention_asm(asm: str) -> None:
    """Checks every attention kernel of one translation unit's assembly; raises RuntimeError on a violation."""
    n = 0
    problems: list[str] = []
    for name, lines in _kernel_bodies(asm, "attn_"):
        n += 1
        problems += check_wide_stores(name, lines)
        if "attn_kvcache_kernel" in name:
            problems += check_rounds(name, lines)
    if n == 0:
        problems.append("no attention kernel found in the assembly")
    if problems:
        raise RuntimeError("attention machine-code check failed:\n  " + "\n  ".join(problems[:20]))


def check_gemm(hipcc: str, flags: list[str], source: str) -> None:
    """Compiles `source` to gfx950 assembly and checks its GEMM kernels."""
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "gemm.s")
        proc = subprocess.run([hipcc, *flags, "--cuda-device-only", "-S", source, "-o", out], capture_output=True, text=True)
        if proc.returncode != 0:
            raise RuntimeError("hipcc failed emitting assembly for the check:\n" + proc.stderr)
        check_asm(open(out).read())
