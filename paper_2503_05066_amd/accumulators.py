"""What the build checks of the kernels that name their accumulation registers in asm statements (csrc/ffn.hip).

The compiler neither knows that these registers hold values nor sees the instructions that use them.  A copy or spill of its
own in one of them, or a matrix instruction closer to a write of its operands than the hardware allows, would give wrong
products without an error, and whether it makes one depends on its version and flags.  So the assembly that it wrote for the
very object that is linked is read, and the build ends where it does not keep to the rules.
"""
import re

OPERAND_STATES = 2   # between a vector instruction's write and a matrix instruction that takes the register
RESULT_STATES = 19   # between a matrix instruction and another use of its result (16-pass instructions; ours have 8)

_REGISTERS = re.compile(r"^([av])(?:\[(\w+):(\w+)\]|\[(\w+)\]|(\d+))$")
_LABEL = re.compile(r"^([\w.$]+):")
_FAR = re.compile(r"\(([\w.$]+)-\.Lpost_getpc\d+\)&")


class AccumulatorError(RuntimeError):
    pass


def _registers(operand):
    m = _REGISTERS.match(operand.strip())
    if not m:
        return frozenset()
    low = int(m[2] or m[4] or m[5], 0)
    return frozenset((m[1], r) for r in range(low, (int(m[3], 0) if m[3] else low) + 1))


def _parse(assembly):
    """[(name, operand registers, text)], the index of each label, and the places where the text of a function begins."""
    code, labels, starts, inside = [], {}, set(), False
    for line in assembly.splitlines():
        line = line.strip()
        if "#ASMSTART" in line or "#ASMEND" in line:
            inside = "#ASMSTART" in line
            continue
        label = _LABEL.match(line)
        if label:
            labels[label[1]] = len(code)
            if not label[1].startswith("."):
                starts.add(len(code))
            continue
        text = line.split(";")[0].strip()
        if not re.match(r"^[a-z]+_\w+(\s|$)", text):
            continue
        name, _, rest = text.partition(" ")
        operands = [_registers(o) for o in re.split(r",\s*|\s+", rest.strip())]
        if not inside and any(kind == "a" for o in operands for kind, _ in o):
            raise AccumulatorError("the compiler uses an accumulation register: " + text)
        code.append((name, operands, text))
    return code, labels, starts


def _predecessors(code, labels, starts):
    before = [[] for _ in range(len(code) + 1)]
    far = None
    for i, (name, _, text) in enumerate(code):
        m = _FAR.search(text)
        if m:
            far = m[1]  # the address that the next s_setpc jumps to
        if name == "s_setpc_b64":
            if far is None:
                raise AccumulatorError("a jump to an unknown place: " + text)
            before[labels[far]].append(i)
            far = None
        elif name == "s_branch" or name.startswith("s_cbranch"):
            before[labels[text.split()[-1]]].append(i)
        if name not in ("s_setpc_b64", "s_branch", "s_endpgm") and i + 1 not in starts:
            before[i + 1].append(i)
    return before


def _within(code, before, at, states):
    """Instructions from which at most `states` - 1 wait states lie before instruction `at`, on any path."""
    seen, found, todo = {}, set(), [(j, 0) for j in before[at]]
    while todo:
        j, passed = todo.pop()
        if passed >= states or seen.get(j, states) <= passed:
            continue
        seen[j] = passed
        found.add(j)
        name, _, text = code[j]
        passed += int(text.split()[1], 0) + 1 if name == "s_nop" else 1
        todo.extend((i, passed) for i in before[j])
    return found


def check(assembly: str) -> int:
    """Raises AccumulatorError where the assembly of a source with named accumulators breaks a rule: a use of an accumulation
    register outside the asm statements; a vector instruction that writes an operand of a matrix instruction fewer than
    OPERAND_STATES ahead of it; another use of a matrix instruction's result fewer than RESULT_STATES behind it.  All paths
    are followed, also around loops.  Returns the number of matrix instructions."""
    code, labels, starts = _parse(assembly)
    before = _predecessors(code, labels, starts)
    matrix = 0
    for at, (name, operands, text) in enumerate(code):
        if name.startswith("v_mfma"):
            matrix += 1
            if not all(operands[:4]):
                raise AccumulatorError("operands not understood: " + text)
            used = frozenset().union(*operands)
            for j in _within(code, before, at, OPERAND_STATES):
                other, written, its_text = code[j]
                if other.startswith("v_") and not other.startswith("v_mfma"):
                    if (written[0] | (written[1] if "swap" in other else frozenset())) & used:
                        raise AccumulatorError("%s: too close ahead of %s" % (its_text, text))
        elif name.startswith("v_accvgpr"):
            used = frozenset().union(*operands)
            for j in _within(code, before, at, RESULT_STATES):
                if code[j][0].startswith("v_mfma") and code[j][1][0] & used:
                    raise AccumulatorError("%s: too close behind %s" % (text, code[j][2]))
    return matrix
