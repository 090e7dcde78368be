"""Static check of this package's own gfx950 code: scalar registers that a vector-memory instruction reads.

On this architecture a vector-memory instruction that takes a scalar register (its base address) reads a stale
value if a vector-ALU instruction wrote that register fewer than five wait states before it; the hardware does
not interlock the case.  The compiler pads the loads it emits itself, but it does not look into an `asm`
statement, and it restores spilled scalars with `v_readlane` right in front of their use.  The kernels here issue
their streaming loads from `asm` statements, so every build is checked:

  * `compile_to_isa` turns one of the package's device sources into ISA text (`hipcc -S`, the device pass only);
  * `hazards` walks that text backwards from every vector-memory instruction with scalar operands, over all
    control-flow predecessors, and reports each vector-ALU write of one of those scalars within five wait states.

A second rule has the same root: the destination registers of a load issued from an `asm` statement hold nothing
until the hand-written wait, so they must not be copied in between.  The compiler keeps to that as long as it has
registers; once it spills vector registers to scratch it may save exactly such a register, and the kernel computes
with what was there before the load (seen once with a tighter occupancy bound: wrong numbers, no fault).
`spilled_asm_kernels` lists the kernels that spill a vector register straight after one of their `asm` loads wrote it.
A register move does the same without a spill: a branch inside a loop with loads in flight (around a rare step, say) made
the compiler give values new registers ahead of the wait.  `copied_asm_kernels` lists the kernels with such a move.

A third rule is about asm statements that hold a matrix instruction (which the compiler does not see as one, so that its accumulators
stay where they are put) or a store of 16 bytes: it pads neither, and `asm_matrix_hazards` looks for vector writes
too close before or behind them and for results touched too early.

`build()` runs the checks on every device source and fails on a finding; tests call them too.
"""
from __future__ import annotations

import os
import re
import subprocess
from typing import Dict, List, Tuple

WAIT_STATES = 5

_VMEM = ("global_", "buffer_", "flat_", "scratch_")
_LABEL = re.compile(r"^([A-Za-z_.$][\w.$]*):$")
_SREG = re.compile(r"\bs\[(\d+):(\d+)\]|\bs(\d+)\b")


def _sregs(text: str) -> set:
    out = set()
    for m in _SREG.finditer(text):
        if m.group(1):
            out |= set(range(int(m.group(1)), int(m.group(2)) + 1))
        else:
            out.add(int(m.group(3)))
    return out


def _operands(text: str) -> List[str]:
    parts = text.split(None, 1)
    return [o.strip() for o in parts[1].split(",")] if len(parts) > 1 else []


def _valu_scalar_writes(text: str) -> set:
    """Scalar registers a vector-ALU instruction writes (lane reads, compares into a scalar pair, carry outputs)."""
    op = text.split()[0]
    if not op.startswith("v_"):
        return set()
    ops = _operands(text)
    out = set()
    if ops and re.fullmatch(r"s\[\d+:\d+\]|s\d+", ops[0]):
        out |= _sregs(ops[0])
    carry = ("_co_" in op or op.startswith(("v_addc", "v_subb", "v_subbrev", "v_div_scale", "v_mad_u64_u32", "v_mad_i64_i32")))
    if carry and len(ops) > 1 and re.fullmatch(r"s\[\d+:\d+\]|s\d+", ops[1]):
        out |= _sregs(ops[1])
    return out


def _wait_states(text: str) -> int:
    if text.startswith("s_nop"):
        return int(text.split()[1], 0) + 1
    return 1


def _flow(isa_text: str) -> Tuple[List[Tuple[int, str, bool]], List[List[int]]]:
    """The instructions as (line, text, inside an asm statement), and the predecessors of each."""
    ins: List[Tuple[int, str, bool]] = []
    labels: Dict[str, int] = {}
    in_asm = False
    for n, raw in enumerate(isa_text.splitlines(), 1):
        if raw.strip().startswith(";;#ASM"):
            in_asm = raw.strip().startswith(";;#ASMSTART")
            continue
        s = raw.split(";")[0].strip()
        if not s:
            continue
        m = _LABEL.match(s)
        if m:
            labels[m.group(1)] = len(ins)
            continue
        if s.startswith("."):
            continue
        ins.append((n, s, in_asm))
    preds: List[List[int]] = [[] for _ in ins]
    for i, (_, s, _) in enumerate(ins):
        op = s.split()[0]
        falls = op not in ("s_branch", "s_endpgm", "s_setpc_b64")
        if op == "s_branch" or op.startswith("s_cbranch"):
            tgt = labels.get(s.split()[1])
            if tgt is not None and tgt < len(ins):
                preds[tgt].append(i)
        if falls and i + 1 < len(ins):
            preds[i + 1].append(i)
    return ins, preds


def hazards(isa_text: str) -> List[Tuple[int, str, int, str, int]]:
    """Findings as (line of the write, write, line of the memory instruction, memory instruction, wait states between)."""
    ins, preds = _flow(isa_text)
    found = []
    for i, (ln, s, _) in enumerate(ins):
        op = s.split()[0]
        if not op.startswith(_VMEM):
            continue
        need = set()
        for o in _operands(s):
            if re.fullmatch(r"s\[\d+:\d+\]|s\d+", o.split()[0] if o else ""):
                need |= _sregs(o.split()[0])
        if not need:
            continue
        # backwards over every path, until five wait states lie between
        stack = [(j, 0) for j in preds[i]]
        seen: Dict[int, int] = {}
        while stack:
            j, ws = stack.pop()
            if ws >= WAIT_STATES or seen.get(j, WAIT_STATES) <= ws:
                continue
            seen[j] = ws
            lnj, t, _ = ins[j]
            hit = _valu_scalar_writes(t) & need
            if hit:
                found.append((lnj, t, ln, s, ws))
                continue
            ws2 = ws + _wait_states(t)
            for k in preds[j]:
                stack.append((k, ws2))
    return found


_MATRIX = ("v_mfma_", "v_smfmac_")
OPERAND_STATES = 2          # between a vector write of an operand and the matrix instruction that reads it
RESULT_STATES = 20          # between a matrix instruction (up to 16 passes) and anything else that touches its result
STORE_STATES = 2            # between a store of more than 8 bytes and a vector write of its data
_WIDE_STORE = re.compile(r"(global|flat|buffer|scratch)_store_dwordx[34]\b")


def _vector_regs(text: str) -> set:
    """Vector and accumulation registers named in an operand list, as ("v" or "a", number)."""
    out = set()
    for m in re.finditer(r"\b([va])\[(\d+):(\d+)\]|\b([va])(\d+)\b", text):
        if m.group(1):
            out |= {(m.group(1), r) for r in range(int(m.group(2)), int(m.group(3)) + 1)}
        else:
            out.add((m.group(4), int(m.group(5))))
    return out


def _valu_vector_writes(text: str) -> set:
    op = text.split()[0]
    if not op.startswith("v_") or op.startswith(_MATRIX):
        return set()
    ops = _operands(text)
    return _vector_regs(",".join(ops[:2] if op.startswith("v_swap") else ops[:1]))


def asm_matrix_hazards(isa_text: str) -> List[Tuple[int, str, int, str, int]]:
    """The compiler keeps no distance from matrix instructions and wide stores inside asm statements.  Findings, as in `hazards`:
      * a vector-ALU write of an operand or accumulator of such a matrix instruction less than OPERAND_STATES before it;
      * anything that reads or writes the result of one less than RESULT_STATES after it, but for the same instruction adding to the
        same registers again;
      * a vector-ALU write of the data of such a store of 12 or 16 bytes less than STORE_STATES behind it."""
    ins, preds = _flow(isa_text)
    succs: List[List[int]] = [[] for _ in ins]
    for i, ps in enumerate(preds):
        for p in ps:
            succs[p].append(i)
    found = []

    def near(i, states, way):
        """(j, wait states between) for what lies less than `states` from i over some path."""
        stack, seen = [(j, 0) for j in way[i]], {}
        while stack:
            j, ws = stack.pop()
            if ws >= states or seen.get(j, states) <= ws:
                continue
            seen[j] = ws
            stack += [(k, ws + _wait_states(ins[j][1])) for k in way[j]]
        return sorted(seen.items())

    for i, (ln, s, asm) in enumerate(ins):
        if not asm:
            continue
        if s.startswith(_MATRIX):
            ops = _operands(s)
            result, touched = _vector_regs(ops[0]), _vector_regs(",".join(ops))
            for j, ws in near(i, OPERAND_STATES, preds):
                if _valu_vector_writes(ins[j][1]) & touched:
                    found.append((ins[j][0], ins[j][1], ln, s, ws))
            for j, ws in near(i, RESULT_STATES, succs):
                t = _operands(ins[j][1])
                again = ins[j][1].split()[0] == s.split()[0] and t[0] == ops[0] and not result & _vector_regs(",".join(t[1:3]))
                if not again and result & _vector_regs(",".join(t)):
                    found.append((ln, s, ins[j][0], ins[j][1], ws))
        elif _WIDE_STORE.match(s):
            data = _vector_regs(_operands(s)[0 if s.startswith("buffer") else 1])
            for j, ws in near(i, STORE_STATES, succs):
                if _valu_vector_writes(ins[j][1]) & data:
                    found.append((ln, s, ins[j][0], ins[j][1], ws))
    return found


def _vregs(text: str) -> set:
    out = set()
    for m in re.finditer(r"\bv\[(\d+):(\d+)\]|\bv(\d+)\b", text):
        if m.group(1):
            out |= set(range(int(m.group(1)), int(m.group(2)) + 1))
        else:
            out.add(int(m.group(3)))
    return out


def spilled_asm_kernels(isa_text: str) -> List[Tuple[str, List[int]]]:
    """(kernel, registers) for every kernel that spills a vector register whose last writer, going back from the
    spill in program order, is a vector-memory load inside an asm statement (no wait in between)."""
    lines = isa_text.splitlines()
    kernel_at: List[str] = []
    in_asm_at: List[bool] = []
    cur, in_asm = None, False
    for raw in lines:
        s = raw.strip()
        m = re.match(r"^([A-Za-z_][\w$]*):", raw)
        if m and not raw.startswith("."):
            cur = m.group(1)
        if s.startswith(";;#ASMSTART"):
            in_asm = True
        elif s.startswith(";;#ASMEND"):
            in_asm = False
        kernel_at.append(cur)
        in_asm_at.append(in_asm)
    found: Dict[str, set] = {}
    for i, raw in enumerate(lines):
        s = raw.strip()
        if not s.startswith("scratch_store") or "Spill" not in s:
            continue
        ops = _operands(s.split(";")[0])
        regs = _vregs(ops[1] if len(ops) > 1 else "")
        for j in range(i - 1, max(i - 2000, -1), -1):
            if kernel_at[j] != kernel_at[i] or not regs:
                break
            t = lines[j].split(";")[0].strip() if not lines[j].strip().startswith(";;#") else ""
            if not t or t.endswith(":") or t.startswith("."):
                continue
            op = t.split()[0]
            if op == "s_waitcnt" and "vmcnt" in t:
                break                                   # whatever was in flight has been waited for (or counted) here
            if op.startswith(("v_", "ds_read", "ds_load")) or (op.startswith(_VMEM) and "load" in op and "lds" not in op):
                dst = _vregs(_operands(t)[0]) if _operands(t) else set()
                hit = dst & regs
                if hit:
                    if in_asm_at[j] and op.startswith(_VMEM):
                        found.setdefault(kernel_at[i], set()).update(hit)
                    regs = regs - hit
    return [(k, sorted(v)) for k, v in found.items()]


_COPY = ("v_mov_b32", "v_mov_b64", "v_accvgpr_write", "v_accvgpr_read", "v_accvgpr_mov")


def copied_asm_kernels(isa_text: str) -> List[Tuple[str, List[int]]]:
    """(kernel, registers) for every kernel that moves a vector register which, in program order, an asm load wrote and no
    vector-memory wait has followed."""
    found: Dict[str, set] = {}
    cur, in_asm, flying = None, False, set()
    for raw in isa_text.splitlines():
        s = raw.strip()
        if raw and not raw[0].isspace() and not raw.startswith((".", ";")):
            cur, flying = raw.split(":")[0], set()
            continue
        if s.startswith(";;#ASM"):
            in_asm = s.startswith(";;#ASMSTART")
            continue
        t = s.split(";")[0].strip()
        if not t or t.startswith("."):
            continue
        op = t.split()[0]
        if op == "s_waitcnt":
            if "vmcnt" in t:
                flying = set()                              # whatever was in flight has been waited for (or counted) here
        elif op.startswith(_VMEM):
            if "load" in op and "lds" not in op:
                dst = _vregs(_operands(t)[0])
                flying = flying | dst if in_asm else flying - dst
        elif op.startswith(("v_", "ds_read", "ds_load")):
            ops = _operands(t)
            if op.startswith(_COPY):
                hit = _vregs(",".join(ops[1:])) & flying
                if hit:
                    found.setdefault(cur, set()).update(hit)
            flying = flying - _vregs(ops[0] if ops else "")
    return [(k, sorted(v)) for k, v in found.items()]


def compile_to_isa(source: str, out_path: str, hipcc: str, flags: List[str]) -> str:
    cmd = [hipcc, *flags, "-S", "--offload-device-only", "-o", out_path, source]
    subprocess.run(cmd, check=True, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    with open(out_path) as f:
        return f.read()


def check_source(source: str, build_dir: str, hipcc: str, flags: List[str]) -> List[tuple]:
    """Findings of the checks for one device source (empty: clean)."""
    out = os.path.join(build_dir, os.path.basename(source) + ".s")
    text = compile_to_isa(source, out, hipcc, flags)
    return hazards(text) + asm_matrix_hazards(text) + [(0, f"spills v{regs}", 0, f"kernel {name}: destinations of its asm loads", -1)
                            for name, regs in spilled_asm_kernels(text)] + \
        [(0, f"copies v{regs}", 0, f"kernel {name}: destinations of its asm loads, ahead of the wait", -1)
         for name, regs in copied_asm_kernels(text)]
