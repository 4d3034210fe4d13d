"""Checks on the built library's gfx950 code (its own disassembly) that the compiler makes for code it understands and
cannot make across inline assembly:

  * matrix instructions: a vector register written by the vector ALU is read by a matrix instruction two wait states
    later at the earliest; a result is touched by anything else 12 wait states after the instruction at the earliest
    (v_mfma_f32_16x16x128_f8f6f4; 8 for v_mfma_f32_16x16x32_bf16).  These are the distances the compiler keeps for the
    builtins.  A matrix instruction that follows another one is taken to wait until the unit is free (8 / 4 wait states).
  * stores of more than 64 bits: the vector ALU writes a register of their data two wait states later at the earliest (buffer
    stores with a scalar register as offset need none).
  * loads into registers: no instruction touches the destination before an s_waitcnt vmcnt that covers the load.

Both run over the control-flow graph of every kernel, worst case over all paths."""
import functools
import os
import re
import shutil
import subprocess
import tempfile

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
_REG = re.compile(r"\b([va])(?:(\d+)|\[(\d+):(\d+)\])(?![\w\[])")
_LINE = re.compile(r"^\t(\S+)\s*(.*?)\s*// ([0-9A-F]{12}):")
_SYM = re.compile(r"^[0-9a-f]+ <(.+)>:$")
_VM = ("global_", "buffer_", "flat_", "scratch_")


@functools.lru_cache(maxsize=1)
def disassemble(library: str) -> dict:
    """kernel name -> [(address, mnemonic, operands)]"""
    kernels: dict = {}
    with tempfile.TemporaryDirectory() as tmp:
        lib = shutil.copy(library, os.path.join(tmp, "lib.so"))
        subprocess.run([OBJDUMP, "--offloading", lib], check=True, capture_output=True, cwd=tmp)
        for obj in sorted(f for f in os.listdir(tmp) if f.endswith("gfx950")):
            text = subprocess.run([OBJDUMP, "-d", os.path.join(tmp, obj)], check=True, capture_output=True, text=True).stdout
            code = None
            for line in text.splitlines():
                if m := _LINE.match(line):
                    code.append((int(m[3], 16), m[1], m[2]))
                elif m := _SYM.match(line):
                    code = kernels.setdefault(m[1], [])
    return kernels


def _regs(text: str) -> list:
    out = []
    for f, one, lo, hi in _REG.findall(text):
        base = 0 if f == "v" else 512          # two register files
        out += [base + int(one)] if one else range(base + int(lo), base + int(hi) + 1)
    return out


class _Ins:
    __slots__ = ("kind", "defs", "uses", "n", "addr", "text", "data")


def _decode(addr: int, op: str, args: str) -> _Ins:
    i = _Ins()
    i.addr, i.text, i.kind, i.defs, i.uses, i.n, i.data = addr, f"{op} {args}", "other", (), (), 1, ()
    if op == "s_nop":
        i.kind, i.n = "nop", int(args, 0) + 1
    elif op == "s_waitcnt":
        m = re.search(r"vmcnt\((\d+)\)", args)
        i.kind, i.n = "wait", int(m[1]) if m else 63
    elif op.startswith("v_mfma"):
        dst, rest = args.split(",", 1)
        i.kind, i.defs, i.uses, i.n = "mfma", _regs(dst), _regs(rest), 4 if "bf16" in op else 8
    elif op.startswith(_VM):
        if "load" in op and not re.search(r"\blds\b", args):
            dst, rest = args.split(",", 1)
            i.kind, i.defs, i.uses = "load", _regs(dst), _regs(rest)
        elif "atomic" in op or "store" in op or "load" in op:
            i.kind, i.uses = "vmem", _regs(args)
            if re.search(r"_store_(dwordx[34]|format_xyzw?)$", op):
                part = args.split(",")
                buffer = op.startswith("buffer_")
                if not (buffer and re.match(r"\s*(s\d+|m0)\b", part[3] if len(part) > 3 else part[2])):
                    i.data = _regs(part[0 if buffer else 1])
    elif op.startswith("ds_"):
        regs = args.split(",", 1)
        if "read" in op or "rtn" in op or "permute" in op:
            i.kind, i.defs, i.uses = "lds", _regs(regs[0]), _regs(regs[1]) if len(regs) > 1 else ()
        else:
            i.kind, i.uses = "lds", _regs(args)
    elif op.startswith("v_"):
        regs = args.split(",")
        nd = 2 if "swap" in op else 1
        i.kind, i.defs, i.uses = "valu", _regs(",".join(regs[:nd])), _regs(",".join(regs[nd:] if nd == 1 else regs))
    return i


def _targets(code: list) -> dict:
    """index -> successors, at block ends"""
    at = {a: k for k, (a, _, _) in enumerate(code)}
    succ = {}
    for k, (a, op, args) in enumerate(code):
        if op.startswith("s_cbranch") or op == "s_branch":
            d = int(args.split()[0])
            t = at[a + 4 + 4 * (d - 65536 if d >= 32768 else d)]
            succ[k] = [t] if op == "s_branch" else [t, k + 1]
        elif op == "s_endpgm":
            succ[k] = []
        assert not op.startswith(("s_setpc", "s_swappc")), "indirect control flow"
    return succ


def check_kernel(code: list) -> list:
    """Violations as texts."""
    ins = [_decode(*c) for c in code]
    succ = _targets(code)
    leaders = {0} | {t for s in succ.values() for t in s} | {k + 1 for k in succ if k + 1 < len(code)}
    starts = sorted(leaders)
    end_of = {s: (starts[n + 1] if n + 1 < len(starts) else len(code)) for n, s in enumerate(starts)}
    bad: dict = {}

    def flow(s, state):
        # written: register -> wait states a reading matrix instruction still needs; result: register -> wait states until it
        # may be touched; stored: register -> wait states until the vector ALU may write it; unit: until the matrix unit is
        # free; flight: register -> vector-memory operations issued since its load
        written, result, stored, unit, flight = dict(state[0]), dict(state[1]), dict(state[2]), state[3], dict(state[4])
        for k in range(s, end_of[s]):
            x = ins[k]
            cost = x.n if x.kind == "nop" else 1
            if x.kind == "mfma" and unit > 0:
                written = {r: w - unit for r, w in written.items() if w > unit}
                result = {r: w - unit for r, w in result.items() if w > unit}
                stored = {r: w - unit for r, w in stored.items() if w > unit}
            if stored and x.kind == "valu":
                for r in x.defs:
                    if r in stored:
                        bad[x.addr] = f"{x.addr:#x} {x.text}: writes the data of a store {stored[r]} wait states too early"
            if flight and (x.defs or x.uses):
                for r in x.uses if x.kind == "load" else (*x.defs, *x.uses):     # (loads return in order)
                    if r in flight:
                        bad[x.addr] = f"{x.addr:#x} {x.text}: touches a load in flight"
            if x.kind == "mfma":
                for r in x.uses:
                    if r in written:
                        bad[x.addr] = f"{x.addr:#x} {x.text}: operand written by the vector ALU {written[r]} wait states too late"
                own = set(x.defs)
                for r in x.uses:
                    if r in result and r not in own:
                        bad[x.addr] = f"{x.addr:#x} {x.text}: reads a result {result[r]} wait states too early"
            elif result:
                for r in (*x.defs, *x.uses):
                    if r in result:
                        bad[x.addr] = f"{x.addr:#x} {x.text}: touches a result {result[r]} wait states too early"
            if written:
                written = {r: w - cost for r, w in written.items() if w > cost}
            if result:
                result = {r: w - cost for r, w in result.items() if w > cost}
            if stored:
                stored = {r: w - cost for r, w in stored.items() if w > cost}
            for r in x.data:
                stored[r] = 2
            unit = max(unit - cost, 0) if x.kind != "mfma" else x.n - 1
            if x.kind == "valu":
                for r in x.defs:
                    written[r] = 2
            elif x.kind == "mfma":
                for r in x.defs:
                    written.pop(r, None)
                    result[r] = x.n + 4
            elif x.kind in ("load", "vmem"):
                flight = {r: y + 1 for r, y in flight.items()}
                for r in x.defs:
                    flight[r] = 0
            elif x.kind == "wait" and flight:
                flight = {r: y for r, y in flight.items() if y < x.n}
        return written, result, stored, unit, flight

    def merge(a, b):
        if a is None:
            return b
        out = []
        for n in (0, 1, 2):
            m = dict(a[n])
            for r, w in b[n].items():
                m[r] = max(m.get(r, 0), w)
            out.append(m)
        f = dict(a[4])
        for r, y in b[4].items():
            f[r] = min(f.get(r, 99), y)
        return *out, min(a[3], b[3]), f

    state = {0: ({}, {}, {}, 0, {})}
    work = [0]
    while work:
        s = work.pop()
        out = flow(s, state[s])
        last = end_of[s] - 1
        for t in succ.get(last, [last + 1] if last + 1 < len(code) else []):
            m = merge(state.get(t), out)
            if m != state.get(t):
                state[t] = m
                if t not in work:
                    work.append(t)
    return list(bad.values())
