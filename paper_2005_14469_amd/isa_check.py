"""Static check of the generated GCN code of a kernel that issues loads from asm statements.

The SpDM kernel starts its B loads (and the loads of its schedule stream) with `global_load_*`
inside asm statements and waits for them with its own `s_waitcnt vmcnt(n)`; the compiler does not
know that those destination registers are still in flight.  That is only correct if no
instruction - the compiler's or the kernel's own asm - touches such a register before a wait has
covered its load.  This module proves it on the assembly text:

  * the kernel is cut into basic blocks and a control-flow graph is built from the branch
    instructions (compiler branches and the labels inside asm statements alike);
  * vector-memory operations complete in order, so the abstract state at a point is the queue of
    operations that may still be outstanding, oldest first, each with the registers it will
    write (stores carry none).  A load or store appends an entry, `s_waitcnt vmcnt(n)` keeps the
    youngest n entries, and where paths join the queues are aligned at their young end and
    merged entry by entry (what is outstanding at distance i from the youngest on any path);
  * a forward data-flow pass runs this to a fixed point, then every instruction that names a
    register of an entry still in the queue - other than a new load into it - is reported.
"""
from __future__ import annotations

import re

_LABEL = re.compile(r"^(\.LBB\d+_\d+|\d+):")
_BRANCH = re.compile(r"^\s*(s_cbranch_\w+|s_branch)\s+(\S+)")


def _regs(text: str) -> set[int]:
    out: set[int] = set()
    for m in re.finditer(r"\bv\[(\d+):(\d+)\]|\bv(\d+)\b", text):
        if m.group(1):
            out |= set(range(int(m.group(1)), int(m.group(2)) + 1))
        else:
            out.add(int(m.group(3)))
    return out


def kernel_body(asm_text: str, mangled_prefix: str) -> list[str]:
    lines = asm_text.split("\n")
    start = next(i for i, l in enumerate(lines) if l.startswith(mangled_prefix) and ":" in l)
    body = []
    for l in lines[start + 1:]:
        if l.startswith(".Lfunc_end"):
            break
        body.append(l)
    return body


def _graph(body: list[str]):
    """The basic blocks of a kernel: dict(labels, insts=[(index, text, in an asm statement)], succ=[indices])."""
    # instruction stream with asm flag; blocks start at labels and after branches
    insts = []          # (text, in_asm)
    in_asm = False
    for l in body:
        if "#ASMSTART" in l:
            in_asm = True
            continue
        if "#ASMEND" in l:
            in_asm = False
            continue
        t = l.split(";")[0].strip() if not l.strip().startswith(";") else ""
        if not t or t.startswith("."):
            m = _LABEL.match(l.strip())
            if not m:
                continue
            t = l.strip().split(";")[0].strip()
        insts.append((t, in_asm))
    # basic blocks
    blocks = []         # dict(label, insts=[(idx, text, in_asm)], succ=[...])
    cur = dict(labels=[], insts=[])
    for i, (t, a) in enumerate(insts):
        m = _LABEL.match(t)
        if m:
            if cur["insts"] or cur["labels"]:
                blocks.append(cur)
                cur = dict(labels=[], insts=[])
            cur["labels"].append(m.group(1))
            continue
        cur["insts"].append((i, t, a))
        if _BRANCH.match(t) or t.startswith("s_endpgm"):
            blocks.append(cur)
            cur = dict(labels=[], insts=[])
    if cur["insts"] or cur["labels"]:
        blocks.append(cur)
    # a block that is only labels merges into the next one
    merged = []
    pend = []
    for b in blocks:
        if not b["insts"]:
            pend += b["labels"]
            continue
        b["labels"] = pend + b["labels"]
        pend = []
        merged.append(b)
    blocks = merged

    # Numeric local labels (asm) may repeat: "1f"/"1b" resolve to the nearest one forward/backward.
    def resolve(bi: int, target: str):
        if target.startswith(".LBB"):
            for j, b in enumerate(blocks):
                if target in b["labels"]:
                    return j
            raise ValueError(f"label {target} not found")
        m = re.match(r"(\d+)([fb])$", target)
        if not m:
            raise ValueError(f"branch target {target}")
        rng = range(bi + 1, len(blocks)) if m.group(2) == "f" else range(bi, -1, -1)
        for j in rng:
            if m.group(1) in blocks[j]["labels"]:
                return j
        raise ValueError(f"local label {target} not found")

    for bi, b in enumerate(blocks):
        succ = []
        last = b["insts"][-1][1]
        m = _BRANCH.match(last)
        if m:
            succ.append(resolve(bi, m.group(2)))
            if m.group(1) != "s_branch" and bi + 1 < len(blocks):
                succ.append(bi + 1)
        elif not last.startswith("s_endpgm") and bi + 1 < len(blocks):
            succ.append(bi + 1)
        b["succ"] = succ

    return blocks


_VMEM = ("global_load", "global_store", "global_atomic", "buffer_load", "buffer_store", "flat_load", "flat_store",
         "scratch_load", "scratch_store")


def check(asm_text: str, mangled_prefix: str):
    """Returns (load destination registers, [(line number, instruction)] of offending instructions)."""
    blocks = _graph(kernel_body(asm_text, mangled_prefix))
    insts = [(t, a) for b in blocks for _, t, a in b["insts"]]
    load_regs: set[int] = set()
    for t, a in insts:
        if a and t.startswith("global_load"):
            load_regs |= _regs(t.split()[1].rstrip(","))
    CAP = 64

    def transfer(b, queue, report=None):
        queue = list(queue)
        for i, t, a in b["insts"]:
            op = t.split()[0]
            if op == "s_waitcnt":
                m = re.search(r"vmcnt\((\d+)\)", t)
                if m:
                    n = int(m.group(1))
                    queue = queue[len(queue) - n:] if n < len(queue) else queue
                    if n == 0:
                        queue = []
                continue
            used = _regs(t)
            if op.startswith(_VMEM):
                is_load = "_load" in op
                dst = _regs(t.split()[1].rstrip(",")) if is_load else set()
                if report is not None:
                    pending = set().union(*queue) if queue else set()
                    if (used - dst) & pending:                    # address/data operands must have arrived
                        report.append((i, t))
                queue.append(frozenset(dst))
                if len(queue) > CAP:
                    queue = [frozenset(queue[0] | queue[1])] + queue[2:]
                continue
            if report is not None and queue:
                pending = set().union(*queue)
                if used & pending:
                    report.append((i, t))
        return tuple(queue)

    def merge(q1, q2):
        if q1 is None:
            return q2
        n = max(len(q1), len(q2))
        p1 = (frozenset(),) * (n - len(q1)) + tuple(q1)
        p2 = (frozenset(),) * (n - len(q2)) + tuple(q2)
        return tuple(a | b for a, b in zip(p1, p2))

    entry = [None] * len(blocks)
    entry[0] = ()
    work = [0]
    while work:
        bi = work.pop()
        out = transfer(blocks[bi], entry[bi])
        for sj in blocks[bi]["succ"]:
            new = merge(entry[sj], out)
            if new != entry[sj]:
                entry[sj] = new
                work.append(sj)
    bad = []
    for bi, b in enumerate(blocks):
        if entry[bi] is not None:
            transfer(b, entry[bi], bad)
    return sorted(load_regs), bad


def check_arrivals(asm_text: str, mangled_prefix: str, plain_stores: tuple = ()):
    """The arrivals (`global_atomic_add_x2`) of a kernel whose workgroups hand words to the last of them without release and acquire.

    What one stores with agent scope (sc1) is past the caches of its XCD once the store is done, and a load with agent scope goes past
    those of the reader's.  Returns (number of arrivals, list of problems).  Proved on the control-flow graph, over all paths:
      * every arrival has nothing outstanding in front of it: a wait for vmcnt(0) behind the last vector-memory operation;
      * no vector-memory operation and no barrier follows an arrival without such a wait in between;
      * a store from which an arrival can be reached is one with agent scope, or of an opcode in `plain_stores` (what only later launches read);
      * a load that can be reached from an arrival is one with agent scope.
    """
    blocks = _graph(kernel_body(asm_text, mangled_prefix))
    arrival = "global_atomic_add_x2"
    reaches = [any(t.startswith(arrival) for _, t, _ in b["insts"]) for b in blocks]         # an arrival lies in the block or behind it
    changed = True
    while changed:
        changed = False
        for i, b in enumerate(blocks):
            if not reaches[i] and any(reaches[j] for j in b["succ"]):
                reaches[i] = changed = True
    problems, arrivals = [], set()

    def walk(bi, state, report):
        out, pending, behind = state                   # outstanding operations, an arrival not waited for, an arrival before
        insts = blocks[bi]["insts"]
        last = max((n for n, (_, t, _) in enumerate(insts) if t.startswith(arrival)), default=-1)
        later = any(reaches[j] for j in blocks[bi]["succ"])
        for n, (i, t, _) in enumerate(insts):
            op = t.split()[0]
            if op == "s_waitcnt":
                if re.search(r"vmcnt\(0\)", t):
                    out = pending = False
                continue
            if op == "s_barrier" and pending and report:
                problems.append(f"{i}: a barrier behind an arrival that was not waited for")
            if not op.startswith(_VMEM):
                continue
            if report:
                if pending:
                    problems.append(f"{i}: '{t}' behind an arrival that was not waited for")
                if op == arrival and out:
                    problems.append(f"{i}: an arrival with operations outstanding")
                if "_store" in op and (later or n < last) and " sc1" not in t and op not in plain_stores:
                    problems.append(f"{i}: '{t}' in front of an arrival without agent scope")
                if "_load" in op and behind and " sc1" not in t:
                    problems.append(f"{i}: '{t}' behind an arrival without agent scope")
            if op == arrival:
                arrivals.add(i)
                pending = behind = True
            out = True
        return out, pending, behind

    entry = [None] * len(blocks)
    entry[0] = (False, False, False)
    work = [0]
    while work:
        bi = work.pop()
        after = walk(bi, entry[bi], False)
        for j in blocks[bi]["succ"]:
            new = after if entry[j] is None else tuple(a or b for a, b in zip(entry[j], after))
            if new != entry[j]:
                entry[j] = new
                work.append(j)
    for bi in range(len(blocks)):
        if entry[bi] is not None:
            walk(bi, entry[bi], True)
    return len(arrivals), problems


def check_lds_loads(asm_text: str, mangled_prefix: str, in_flight: int = 0, asm_only: bool = False):
    """Loads that write LDS directly (`global_load_lds_*`, `buffer_load_* ... lds`) in a kernel that also uses the VGPR index mode.

    Such a load takes the LDS address of lane 0 from M0, and `s_set_gpr_idx_on/idx` overwrite M0.
    Returns (number of such loads, list of problems).  Proved on the text, block by block:
      * walking back from every such load, an instruction that writes M0 as a plain destination
        (`s_mov_b32 m0`, `s_add_i32 m0`, ...) comes before any label, branch or index-mode instruction
        (other loads to LDS in between are passed over: they leave M0 as it is);
      * walking back from every `s_barrier`, an `s_waitcnt` that names vmcnt(n), n <= in_flight, comes before
        any such load (what a wave has sent to LDS has arrived before the other waves are let past the
        barrier, except the youngest in_flight loads, which a kernel may keep on their way on purpose).
    asm_only: look at the asm statements only, for a kernel all of whose loads to LDS are in one of them that ends with
    nothing in flight.
    """
    lines, inside = [], False
    for l in kernel_body(asm_text, mangled_prefix):
        if "#ASMSTART" in l or "#ASMEND" in l:
            inside = "#ASMSTART" in l
        elif inside or not asm_only:
            lines.append(l)
    body = [l.split(";")[0].strip() for l in lines]
    body = [l for l in body if l]
    def to_lds(t):
        return t.startswith("global_load_lds") or (t.startswith("buffer_load") and t.endswith(" lds"))

    problems = []
    loads = 0
    for i, line in enumerate(body):
        if to_lds(line):
            loads += 1
            j = i - 1
            while j >= 0:
                t = body[j]
                if re.match(r"^s_\w+\s+m0\b", t):
                    break
                if _LABEL.match(t) or _BRANCH.match(t) or t.startswith("s_set_gpr_idx"):
                    problems.append(f"line {i}: '{line}' has no M0 write of its own (stopped at '{t}')")
                    break
                j -= 1
            else:
                problems.append(f"line {i}: '{line}' has no M0 write before it")
        elif line.startswith("s_barrier"):
            j = i - 1
            while j >= 0:
                t = body[j]
                waited = re.search(r"vmcnt\((\d+)\)", t) if t.startswith("s_waitcnt") else None
                if waited and int(waited.group(1)) <= in_flight:
                    break
                if to_lds(t):
                    problems.append(f"line {i}: barrier with a load to LDS ('{t}') not awaited")
                    break
                if _LABEL.match(t):            # the walk stays in the block: a barrier that opens a block is judged unsafe
                    if any(to_lds(b) for b in body):
                        problems.append(f"line {i}: barrier at the start of a block, no wait seen")
                    break
                j -= 1
    return loads, problems


def asm_scalar_writes(asm_text: str, mangled_prefix: str):
    """(scalar registers written, scalar registers only read) by the asm statements of a kernel: the first set has to be what
    their clobber lists name, or the compiler may keep something of its own there."""
    def regs(text):
        out = set()
        for m in re.finditer(r"\bs\[(\d+):(\d+)\]|\bs(\d+)\b", text):
            out |= set(range(int(m.group(1)), int(m.group(2)) + 1)) if m.group(1) else {int(m.group(3))}
        return out

    written, read, in_asm = set(), set(), False
    for l in kernel_body(asm_text, mangled_prefix):
        if "#ASMSTART" in l or "#ASMEND" in l:
            in_asm = "#ASMSTART" in l
            continue
        t = l.split(";")[0].strip()
        if not in_asm or not t or t.startswith("."):
            continue
        op, _, rest = t.partition(" ")
        ops = rest.split(",")
        writes = op.startswith("s_") and not re.match(r"s_(cbranch|branch|barrier|waitcnt|nop|cmp|bitcmp|set_gpr_idx)", op) or op.startswith("v_read")
        if writes:
            written |= regs(ops[0])
            ops = ops[1:]
        for x in ops:
            read |= regs(x)
    return written, read - written
