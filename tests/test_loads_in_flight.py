"""No register that a vector load fills is touched while the load is on its way.

The kernels issue operand reads in inline assembly and wait for them by count (mfma_tiles.h); the compiler takes their results as
there at once, so it may copy, spill or reuse such a register before it is filled, above all where control flow meets.  Nothing in the
source rules that out, so this looks at the code as it was compiled: no instruction of any kernel names a register of a load between
its request and the wait that covers it.

Reads of LDS: on any path, with the fewest younger reads that any path has.  Loads from memory, whose counts depend on which transfers
the branches before them made: what is on its way on every path to a point, with the most younger operations."""
import os
import re
import struct
import subprocess

import pytest

from paper_2602_12675_amd import api

OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")
LINE = re.compile(r"^\t(\S+)\s*(.*?)\s*// ([0-9A-F]+):")
REG = re.compile(r"\b([va])(?:(\d+)|\[(\d+):(\d+)\])(?![\w\[])")
COUNT = re.compile(r"(vmcnt|lgkmcnt)\((\d+)\)")
LDS, VM = 0, 1                            # counters; vector operations of either retire in the order of issue
FULL = 64                                 # more operations than a counter holds: the oldest have retired


def registers(text):
    out = set()
    for bank, one, lo, hi in REG.findall(text):
        lo, hi = (int(one), int(one)) if one else (int(lo), int(hi))
        out.update((bank, n) for n in range(lo, hi + 1))
    return out


def decode(op, args):
    """(counter of a vector memory operation or None, registers it fills, other registers it names, {counter: count waited for})"""
    counter = LDS if op.startswith("ds_") else VM if re.match(r"(global|buffer|scratch|flat)_(load|store|atomic)", op) else None
    fills = (counter == LDS and re.match(r"ds_(read|load|bpermute|permute|swizzle|\w+_rtn)", op)
             or counter == VM and "_load_" in op and "_load_lds_" not in op
             or counter == VM and "_atomic_" in op and re.search(r"\bsc0\b", args))
    first = args.split(",")[0] if fills else ""
    waits = {LDS if c == "lgkmcnt" else VM: int(n) for c, n in COUNT.findall(args)} if op == "s_waitcnt" else {}
    return counter, registers(first), registers(args[len(first):]), waits


def merge(x, y):
    out = {}
    for r in x.keys() | y.keys():
        a, b = x.get(r), y.get(r)
        if a and b:
            out[r] = (a[0], (min if a[0] == LDS else max)(a[1], b[1]))
        elif (a or b)[0] == LDS:
            out[r] = a or b
    return out


def violations(code):
    """code: (address, mnemonic, operands) of one kernel, in order.  [(address, what it touches)]"""
    index = {a: n for n, (a, _, _) in enumerate(code)}
    parsed = [decode(op, args) for _, op, args in code]
    starts, edges = {0}, {}
    for n, (a, op, args) in enumerate(code):
        assert not op.startswith(("s_setpc", "s_swappc", "s_call")), op          # no calls: every path is in this listing
        if op == "s_branch" or op.startswith("s_cbranch"):
            to = int(args.split()[0])
            to = index[a + 4 + 4 * (to - 65536 if to >= 32768 else to)]
            edges[n] = [to] if op == "s_branch" else [to, n + 1]
            starts.update([to, n + 1])
        elif op == "s_endpgm":
            edges[n] = []
            starts.add(n + 1)
    starts = sorted(s for s in starts if s < len(code))
    end = dict(zip(starts, starts[1:] + [len(code)]))
    at, work, bad = {0: {}}, [0], set()                    # before a block: register -> (counter, younger operations of that counter)
    while work:
        block = work.pop()
        state = dict(at[block])
        for n in range(block, end[block]):
            counter, fills, named, waits = parsed[n]
            for c, left in waits.items():
                state = {r: (k, age) for r, (k, age) in state.items() if k != c or age < left}
            for r in named & state.keys() | {r for r in fills & state.keys() if state[r][0] != counter}:   # (the same counter: filled in turn)
                bad.add((code[n][0], "%s touches %s%d" % (code[n][1], *r)))
            if counter is not None:
                state = {r: (k, age + (k == counter)) for r, (k, age) in state.items() if age < FULL}
                state.update((r, (counter, 0)) for r in fills)
        for to in edges.get(end[block] - 1, [end[block]]):
            if to < len(code):
                now = state if to not in at else merge(at[to], state)
                if to not in at or now != at[to]:
                    at[to] = now
                    work.append(to)
    return sorted(bad)


def kernels(path, folder):
    """(name, code) of every kernel in the device images of a library"""
    with open(path, "rb") as f:
        blob = f.read()
    at = blob.find(b"\x7fELF", 1)
    while at >= 0:
        if struct.unpack_from("<H", blob, at + 18)[0] == 224:                    # EM_AMDGPU
            shoff, = struct.unpack_from("<Q", blob, at + 40)
            size, count = struct.unpack_from("<HH", blob, at + 58)
            image = os.path.join(folder, "image")
            with open(image, "wb") as f:
                f.write(blob[at : at + shoff + size * count])
            text = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", image], capture_output=True, text=True, check=True).stdout
            name, code = None, []
            for line in text.splitlines():
                if line.endswith(">:"):
                    if code:
                        yield name, code
                    name, code = line.split("<")[1][:-2], []
                elif m := LINE.match(line):
                    code.append((int(m.group(3), 16), m.group(1), m.group(2)))
            if code:
                yield name, code
        at = blob.find(b"\x7fELF", at + 1)


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_no_load_in_flight_is_touched(tmp_path):
    reads, bad = 0, {}
    for name, code in kernels(api.LIB_PATH, str(tmp_path)):
        reads += sum(op.startswith("ds_read") for _, op, _ in code)
        if v := violations(code):
            bad[name] = ["%x %s" % x for x in v[:4]]
    assert reads > 1000 and not bad, bad


# what the check has to notice, and what it must let pass: (mnemonic, operands) at addresses 0, 4, 8, ...
READ, ADD, END = ("ds_read_b128", "v[0:3], v9"), ("v_add_f32_e32", "v8, v2, v8"), ("s_endpgm", "")
OTHER, TWO, NONE = ("ds_read_b64", "v[4:5], v9"), ("s_waitcnt", "lgkmcnt(1)"), ("s_waitcnt", "vmcnt(0) lgkmcnt(0)")
LOAD, DMA, LANDED = ("global_load_dword", "v2, v9, s[0:1]"), ("global_load_lds_dwordx4", "v9, s[0:1]"), ("s_waitcnt", "vmcnt(1)")


@pytest.mark.parametrize("code,ok", [
    ([READ, ADD, END], False),                                                  # no wait at all
    ([READ, NONE, ADD, END], True),
    ([READ, OTHER, TWO, ADD, END], True),                                       # counted: the older one of two
    ([OTHER, READ, TWO, ADD, END], False),                                      # ... is the other one
    ([READ, ("s_cbranch_scc1", "1"), ("v_mov_b32_e32", "v7, v3"), NONE, ADD, END], False),      # copied on one side of a branch
    ([READ, ("s_cbranch_scc1", "1"), OTHER, TWO, ADD, END], False),             # counted on one side only
    ([READ, ("s_cbranch_scc1", "1"), ("v_mov_b32_e32", "v7, v6"), NONE, ADD, END], True),
    ([READ, ("v_mov_b32_e32", "v1, 0"), NONE, END], False),                     # reused as if it were free
    ([READ, ("scratch_store_dwordx4", "off, v[0:3], off"), NONE, END], False),  # spilled
    ([READ, ("ds_write_b32", "v9, v0"), NONE, END], False),
    ([READ, READ, NONE, ADD, END], True),                                       # filled in turn
    ([LOAD, DMA, LANDED, ADD, END], True),
    ([DMA, LOAD, LANDED, ADD, END], False),
    ([LOAD, ("s_cbranch_scc1", "2"), DMA, LANDED, ADD, END], True),             # (memory: only what is on its way on every path)
    ([LOAD, ("s_cbranch_scc1", "1"), ("v_accvgpr_write_b32", "a0, v2"), NONE, ADD, END], False),
    ([ADD, READ, ("s_cbranch_scc1", "65533"), NONE, END], False),               # in flight into the next turn of a loop
])
def test_the_check_itself(code, ok):
    assert (not violations([(4 * n, *x) for n, x in enumerate(code)])) == ok
