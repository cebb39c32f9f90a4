"""Checks on the assembly that the build makes of this library's own kernels: what the sources rely on and the compiler does not promise.

Matrix instructions inside inline assembly.
The compiler sees inline assembly as opaque: it neither inserts the wait states that a matrix instruction is due in front of its
result or behind its operands, nor knows that a copy or a spill of such a register in between goes wrong.  The attention core
writes the matrix instructions of its scores that way (the only ones whose result is in the v half of the register file), so
the build reads what the compiler made of it and fails if
  - the kernel spills registers,
  - anything but the next matrix instruction of the same chain touches a result within WAIT wait states, or
  - a vector instruction writes an operand within OPERAND_WAIT wait states of the matrix instruction that reads it.

Buffer stores of more than two registers at an offset in a scalar register.  They read their data late: where a vector instruction overwrites it
within STORE_WAIT wait states, that may be what is stored.  The compiler leaves the wait states for constant offsets only; the sources put
them behind the store (store_vector), which holds as long as the compiler does not copy the data out of its registers in between.

Spilled vector registers, in the kernels that are laid out to fill the register file.
"""
import re

WAIT = 12          # 11 are due behind a 32x32x16 product (eight passes) before another unit reads or writes its result
OPERAND_WAIT = 2   # between a vector instruction's result and a matrix instruction that reads it
STORE_WAIT = 2     # between a buffer store with a scalar offset and a vector instruction that overwrites its data

_REG = re.compile(r"\bv(?:(\d+)\b|\[(\d+):(\d+)\])")


def _regs(text):
    out = set()
    for one, lo, hi in _REG.findall(text):
        out |= {int(one)} if one else set(range(int(lo), int(hi) + 1))
    return out


def _file_regs(text):
    """Registers of both halves of the file: (half, number)."""
    out = set()
    for half, one, lo, hi in re.findall(r"\b([va])(?:(\d+)\b|\[(\d+):(\d+)\])", text):
        out |= {(half, int(one))} if one else {(half, r) for r in range(int(lo), int(hi) + 1)}
    return out


class _Code:
    """Instructions of one kernel in text order, out-of-line parts of inline assembly left out (they open with a wait of their own)."""

    def __init__(self, lines):
        self.ops, self.labels, out_of_line = [], {}, False
        for line in lines:
            line = line.split(";")[0].split("//")[0].strip()
            if line.startswith(".subsection"):
                out_of_line = line.split()[1] != "0"
            if not line or out_of_line:
                continue
            if line.endswith(":"):
                self.labels[line[:-1]] = len(self.ops)
            elif not line.startswith("."):
                self.ops.append(line)

    def states(self, i):
        m = re.match(r"s_nop (\d+)", self.ops[i])
        return int(m.group(1)) + 1 if m else 1

    def after(self, i):
        """Indices that may follow instruction i."""
        op = self.ops[i].split()
        nxt = [i + 1] if i + 1 < len(self.ops) and op[0] not in ("s_branch", "s_endpgm") else []
        if op[0].startswith(("s_branch", "s_cbranch")) and op[1] in self.labels:
            nxt.append(self.labels[op[1]])
        return nxt

    def within(self, i, states):
        """Indices of the instructions less than `states` wait states behind instruction i, on any path; visit(j) true ends the path."""
        best, todo = {}, [(j, 0) for j in self.after(i)]
        while todo:
            j, waited = todo.pop()
            if j >= len(self.ops) or waited >= states or best.get(j, states) <= waited:
                continue
            best[j] = waited
            stop = yield j
            if not stop:
                todo += [(k, waited + self.states(j)) for k in self.after(j)]


def _is_score(op):
    return op.startswith("v_mfma") and re.match(r"v_mfma\S+\s+v", op) is not None


def check_code(lines):
    """Faults of one kernel's instructions, as texts."""
    code, faults = _Code(lines), []
    for i, op in enumerate(code.ops):
        if _is_score(op):
            result = _regs(op.split(",")[0])
            walk = code.within(i, WAIT)
            stop = None
            while True:
                try:
                    j = walk.send(stop)
                except StopIteration:
                    break
                other = code.ops[j]
                stop = _is_score(other) and _regs(other.split(",")[0]) == result   # the chain goes on: its own wait counts
                operands = ",".join(other.split(",")[1:3]) if stop else other
                if _regs(operands) & result:
                    faults.append("result touched early: `%s` behind `%s`" % (other, op))
        elif op.startswith("v_") and not op.startswith("v_mfma"):
            written = _regs(op.split(",")[0]) | (_regs(",".join(op.split(",")[:2])) if "swap" in op else set())
            walk = code.within(i, OPERAND_WAIT)
            for j in walk:
                if _is_score(code.ops[j]) and _regs(",".join(code.ops[j].split(",")[1:])) & written:
                    faults.append("operand written late: `%s` in front of `%s`" % (op, code.ops[j]))
    return faults


_LATE_STORE = re.compile(r"buffer_store_dwordx[34]\s+([^,]+),[^,]+,\s*s\[\d+:\d+\],\s*(?:s\d+|m0|vcc_lo|vcc_hi|ttmp\d+)\b")


def check_stores(lines):
    """Buffer stores whose data is overwritten too early, as texts."""
    code, faults = _Code(lines), []
    for i, op in enumerate(code.ops):
        m = _LATE_STORE.match(op)
        if not m:
            continue
        data = _file_regs(m.group(1))
        for j in code.within(i, STORE_WAIT):
            other = code.ops[j]
            written = ",".join(other.split(",")[:2 if "swap" in other else 1])
            if other.startswith("v_") and _file_regs(written) & data:
                faults.append("data overwritten early: `%s` behind `%s`" % (other, op))
    return faults


def functions(text):
    """(name, lines) of the functions of a device assembly file."""
    name, body = None, []
    for line in text.splitlines():
        m = re.match(r"(_Z\w+):", line)
        if m:
            name, body = m.group(1), []
        elif line.startswith(".Lfunc_end") and name:
            yield name, body
            name = None
        elif name:
            body.append(line)


def _spills(text, kernel, keys=("vgpr_spill_count", "private_segment_fixed_size")):
    faults = []
    for entry in re.split(r"\n  - \.", text.split(".amdgpu_metadata")[-1]):
        name = re.search(r"\.name:\s+(\S+)", entry)
        if name and kernel in name.group(1):
            for key in keys:
                m = re.search(r"\.?%s:\s+(\d+)" % key, entry)
                if m is None or int(m.group(1)) != 0:
                    faults.append("%s: %s is %s" % (name.group(1), key, m and m.group(1)))
    return faults


def check_source(text, scores=None, spills=None):
    """Faults of a device assembly file: its stores, the matrix instructions in inline assembly of kernel `scores`, the spills of kernel `spills`."""
    faults = ["%s: %s" % (name, f) for name, lines in functions(text) for f in check_stores(lines)]
    if scores:
        faults += check(text, scores)
    return faults + (_spills(text, spills) if spills else [])


def check(text, kernel):
    """Faults of all instances of `kernel` in a device assembly file; at least one has to be there, with scores in it."""
    faults, lines, found = [], text.splitlines(), 0
    for start, line in enumerate(lines):
        m = re.match(r"(\w*%s\w*):" % kernel, line)
        if not m:
            continue
        end = next(i for i in range(start, len(lines)) if lines[i].startswith(".Lfunc_end"))
        body = lines[start + 1:end]
        found += 1
        if not any(_is_score(l.strip()) for l in body):
            faults.append("%s: no matrix instruction with its result in the v half" % m.group(1))
        faults += ["%s: %s" % (m.group(1), f) for f in check_code(body)]
    if not found:
        faults.append("no instance of %s" % kernel)
    return faults + _spills(text, kernel, ("vgpr_spill_count", "sgpr_spill_count", "private_segment_fixed_size"))
