"""Wait states that the hardware does not keep by itself, looked for in the compiler's gfx950 assembly (text only, no GPU).

The compiler keeps them between its own instructions; it does not look inside inline assembly, where the decode kernels
have their HBM -> LDS loads, the stores of their partials and the arguments that they keep in the lanes of a register.  Looked for, along every path through a function:
  - a memory instruction reading a scalar register less than 5 wait states after a vector instruction wrote it;
  - an LDS load less than 1 wait state after a scalar instruction wrote M0;
  - a vector instruction writing the data registers of a store of more than 8 bytes less than 2 wait states after it;
  - a vector instruction reading a scalar register less than 2 wait states after a vector instruction wrote it, or taking the lane
    of a v_readlane or v_writelane from it less than 4 after;
  - a v_readlane or v_readfirstlane of a vector register less than 1 wait state after a vector instruction wrote it.
An instruction is one wait state, s_nop N is N + 1."""
import re

SGPR_WAIT, M0_WAIT, DATA_WAIT, SGPR_TO_VECTOR_WAIT, SGPR_TO_LANE_WAIT, VGPR_TO_READLANE_WAIT = 5, 1, 2, 2, 4, 1
_LABEL = re.compile(r"^([\w.$]+):")
_CARRY = re.compile(r"v_(add|sub|subrev|addc|subb|subbrev)_co|v_div_scale|v_mad_[ui]64")


def _regs(text, kind):
    for one, lo, hi in re.findall(rf"(?<![\w.]){kind}(?:(\d+)\b|\[(\d+):(\d+)\])", text):
        yield from ([int(one)] if one else range(int(lo), int(hi) + 1))
    if kind == "s" and re.search(r"\bvcc\b", text):
        yield "vcc"


def functions(asm):
    """(name, lines of code) of every function of an assembly listing."""
    name, code = None, []
    for line in asm.splitlines():
        text = line.split(";")[0].strip()
        label = _LABEL.match(text)
        if label and not label[1].startswith("."):
            name, code = label[1], []
        elif line.startswith(".Lfunc_end"):
            if name:
                yield name, code
            name = None
        elif name and text and (label or not text.startswith(".")):
            code.append(text)


def _step(text, wait, found):
    """One instruction: what it breaks goes to `found`, and the wait states that are owed after it are returned."""
    op, _, rest = text.partition(" ")
    args = [x.strip() for x in re.split(r",(?![^\[]*\])", rest)]
    memory = re.match(r"(global|buffer|flat|scratch)_", op)
    if memory:
        found.update((text, f"s{r}") for r in _regs(rest, "s") if ("s", r) in wait)
        if "lds" in text and "m0" in wait:
            found.add((text, "m0"))
    if op.startswith("v_"):
        found.update((text, f"v{r}") for r in _regs(args[0], "v") if ("v", r) in wait)
        for i, src in enumerate(args[2 if _CARRY.match(op) else 1:], 1):      # SGPR_WAIT less what is left of it have passed
            least = SGPR_TO_LANE_WAIT if i == 2 and re.match(r"v_(read|write)lane_", op) else SGPR_TO_VECTOR_WAIT
            found.update((text, f"s{r}") for r in _regs(src, "s") if SGPR_WAIT - wait.get(("s", r), 0) < least)
        if op.startswith(("v_readlane", "v_readfirstlane")):
            found.update((text, f"v{r}") for r in _regs(args[1], "v") if ("written v", r) in wait)
    passed = int(rest, 0) + 1 if op == "s_nop" else 1
    wait = {k: n - passed for k, n in wait.items() if n > passed}
    if op.startswith("v_"):
        for dst in args[:2] if _CARRY.match(op) else args[:1]:
            wait.update({("s", r): SGPR_WAIT for r in _regs(dst, "s")})
        wait.update({("written v", r): VGPR_TO_READLANE_WAIT for r in _regs(args[0], "v")})
    elif op.startswith("s_") and not op.startswith(("s_cmp", "s_bitcmp", "s_cbranch", "s_nop", "s_waitcnt")):
        for r in _regs(args[0], "s"):
            wait.pop(("s", r), None)
        if args[0] == "m0":
            wait["m0"] = M0_WAIT
    if memory and re.search(r"store\w*x[34]", op):
        wait.update({("v", r): DATA_WAIT for r in _regs(args[0] if op.startswith("buffer") else args[1], "v")})
    return wait


def hazards(code):
    """The set of (instruction, register) that break a wait state on some path through a function's lines."""
    labels = {_LABEL.match(t)[1]: i for i, t in enumerate(code) if _LABEL.match(t)}
    owed, found, todo = {0: {}}, set(), [0]

    def reach(i, wait):
        old = owed.setdefault(i, None)
        if old is None or any(n > old.get(k, 0) for k, n in wait.items()):
            owed[i] = {k: max(n, wait.get(k, 0)) for k, n in {**wait, **(old or {})}.items()}
            todo.append(i)

    while todo:
        i = todo.pop()
        if i >= len(code):
            continue
        if _LABEL.match(code[i]):
            reach(i + 1, owed[i])
            continue
        wait = _step(code[i], owed[i], found)
        op, _, target = code[i].partition(" ")
        if op.startswith(("s_branch", "s_cbranch")) and target.strip() in labels:
            reach(labels[target.strip()], wait)
        if op not in ("s_branch", "s_endpgm", "s_setpc_b64"):
            reach(i + 1, wait)
    return found
