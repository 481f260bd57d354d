"""Orderings that the kernels depend on and that no result shows reliably, checked on the machine code of the built
library along every path of every kernel (no GPU needed)."""
import functools
import os
import re
import shutil
import subprocess
from concurrent.futures import ProcessPoolExecutor

import pytest

from paper_2605_19049_amd import kvb

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
READELF = "/opt/rocm/llvm/bin/llvm-readelf"
TARGET = re.compile(r"<[^>+]*\+0x([0-9a-f]+)>")
REG = re.compile(r"\b([va])(?:(\d+)\b|\[(\d+):(\d+)\])")


def code_objects(tmp):
    """The gfx950 code objects of libkvb.so, disassembled: one list of lines each."""
    lib = os.path.join(tmp, "libkvb.so")
    shutil.copyfile(kvb.LIB_PATH, lib)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, stdout=subprocess.DEVNULL, cwd=tmp)
    return sorted(os.path.join(tmp, f) for f in os.listdir(tmp) if f.endswith("gfx950"))


def kernels(path):
    """(name, [instruction text], [address]) of every kernel of a code object."""
    text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", path], check=True, stdout=subprocess.PIPE, text=True).stdout
    name, ins, adr, base = None, [], [], 0
    for line in text.splitlines():
        if line.endswith(">:"):
            if name:
                yield name, ins, adr
            name, ins, adr, base = line.split("<")[1][:-2], [], [], int(line.split()[0], 16)
        elif line.startswith("\t") and "//" in line:   # (not the mark of skipped padding)
            body, _, tail = line.partition("//")
            body = body.strip()
            t = TARGET.search(tail)
            if t and body.startswith(("s_branch", "s_cbranch")):
                body = "%s -> %d" % (body.split()[0], base + int(t.group(1), 16))
            ins.append(body)
            adr.append(int(tail.split(":")[0], 16))
    if name:
        yield name, ins, adr


def blocks(ins, adr):
    """Basic blocks as (first, last + 1, successors by block number); block 0 is the entry."""
    at = {a: i for i, a in enumerate(adr)}
    starts, target = {0}, {}
    for i, x in enumerate(ins):
        if "->" in x:
            target[i] = at[int(x.split()[-1])]
            starts.update((target[i], i + 1))
        elif x.startswith("s_endpgm"):
            starts.add(i + 1)
        assert not x.startswith(("s_setpc", "s_swappc")), x
    starts = sorted(s for s in starts if s < len(ins))
    number = {s: n for n, s in enumerate(starts)}
    res = []
    for n, s in enumerate(starts):
        end = starts[n + 1] if n + 1 < len(starts) else len(ins)
        last, succ = ins[end - 1], []
        if "->" in last:
            succ.append(number[target[end - 1]])
        if not last.startswith(("s_branch", "s_endpgm")) and end < len(ins):
            succ.append(number[end])
        res.append((s, end, succ))
    return res


def unordered_tickets(ins, adr):
    """Additions to the fill word that some path reaches without a workgroup barrier."""
    bl = blocks(ins, adr)
    bad, seen, todo = [], {0}, [0]
    while todo:
        first, end, succ = bl[todo.pop()]
        for i in range(first, end):
            if ins[i].startswith("s_barrier"):
                break
            if ins[i].startswith("global_atomic_add"):
                bad.append(ins[i])
        else:
            for s in succ:
                if s not in seen:
                    seen.add(s)
                    todo.append(s)
    return bad


@functools.lru_cache(None)
def regs(operands):
    """Bit mask of the vector registers in an operand text (accumulation registers above the others)."""
    m = 0
    for kind, one, lo, hi in REG.findall(operands):
        lo, hi = (int(one), int(one)) if one else (int(lo), int(hi))
        m |= ((1 << (hi - lo + 1)) - 1) << (lo + (256 if kind == "a" else 0))
    return m


def mfma_wait(op):
    """Wait states between a matrix instruction and a read of its result: its passes of 4 cycles and 2 (fp32), or 4
    (16-bit types)."""
    return {"v_mfma_f32_16x16x4_f32": 8 + 2, "v_mfma_f32_16x16x32_bf16": 4 + 4, "v_mfma_f32_16x16x32_f16": 4 + 4,
            "v_mfma_f32_32x32x16_bf16": 8 + 4}[op]


@functools.lru_cache(None)
def effect(x):
    """(issue slots, mask of what is read before the slot ends, mask of matrix results, their wait)."""
    op, _, rest = x.partition(" ")
    if op == "s_nop":
        return int(rest.split()[0], 0) + 1, 0, 0, 0
    ops = rest.split(", ")
    if op.startswith("v_mfma"):   # (the accumulator input is forwarded)
        return 1, regs(ops[1]) | regs(ops[2]), regs(ops[0]), mfma_wait(op)
    if op.startswith(("v_fmac", "v_permlane", "v_swap")):   # (the destination is read as well)
        return 1, regs(rest), 0, 0
    if op.startswith("v_") or any(x in op for x in ("_load_", "_read", "permute", "swizzle")):
        return 1, regs(", ".join(ops[1:])), 0, 0
    if op.startswith(("ds_", "global_", "buffer_", "scratch_", "flat_")):
        return 1, regs(rest), 0, 0
    return 1, 0, 0, 0


def early_reads(ins, adr):
    """Instructions that some path lets read a matrix result before the wait states it needs."""
    bl = blocks(ins, adr)
    state, bad = {0: frozenset()}, set()
    todo = [0]
    while todo:
        n = todo.pop()
        first, end, succ = bl[n]
        pending = dict(state[n])   # result mask -> wait states still needed
        for i in range(first, end):
            slots, read, made, wait = effect(ins[i])
            if pending:
                if read and any(read & m for m in pending):
                    bad.add((i, ins[i]))
                pending = {m: w - slots for m, w in pending.items() if w > slots}
            if made:
                pending[made] = wait
        out = frozenset(pending.items())
        for s in succ:
            old = dict(state.get(s, ()))
            new = dict(old)
            for m, w in out:
                new[m] = max(w, new.get(m, 0))
            if s not in state or new != old:
                state[s] = frozenset(new.items())
                todo.append(s)
    return sorted(bad)


@functools.lru_cache(None)
def store_data(x):
    """Mask of the data registers of a store of more than 8 bytes, or 0."""
    op, _, rest = x.partition(" ")
    if not re.match(r"(global|flat|scratch|buffer)_store_\w*x[34]$", op):
        return 0
    ops = rest.split(", ")
    return regs(ops[0] if op.startswith("buffer") else ops[1])


@functools.lru_cache(None)
def written(x):
    """Mask of the vector registers that a vector instruction writes (a load's come from elsewhere)."""
    op, _, rest = x.partition(" ")
    if not op.startswith("v_"):
        return 0
    ops = rest.split(", ")
    return regs(", ".join(ops[:2]) if "swap" in op else ops[0])


STORE_WAIT = 2   # wait states for which the data registers of a store of more than 8 bytes stay as they are


def early_overwrites(ins, adr):
    """Vector instructions that some path lets overwrite the data of a store of more than 8 bytes before it has been read."""
    bl = blocks(ins, adr)
    state, bad, todo = {0: frozenset()}, set(), [0]
    while todo:
        n = todo.pop()
        first, end, succ = bl[n]
        pending = dict(state[n])   # data mask -> wait states still needed
        for i in range(first, end):
            if any(written(ins[i]) & m for m in pending):
                bad.add((i, ins[i]))
            slots = int(ins[i].split()[1], 0) + 1 if ins[i].startswith("s_nop") else 1
            pending = {m: w - slots for m, w in pending.items() if w > slots}
            if store_data(ins[i]):
                pending[store_data(ins[i])] = STORE_WAIT
        for s in succ:
            new = dict(state.get(s, ()))
            for m, w in pending.items():
                new[m] = max(w, new.get(m, 0))
            if s not in state or new != dict(state[s]):
                state[s] = frozenset(new.items())
                todo.append(s)
    return sorted(bad)


def spills(path):
    """Vector registers that each kernel spills, from the code object's metadata."""
    notes = subprocess.run([READELF, "--notes", path], check=True, stdout=subprocess.PIPE, text=True).stdout
    names, counts = [re.findall(r"^ {4}\.%s: +(\S+)$" % key, notes, re.M) for key in ("name", "vgpr_spill_count")]
    assert len(names) == len(counts) and names
    return dict(zip(names, map(int, counts)))


def waits_at_the_exit(ins, adr, window):
    """Waits for every load and atomic ahead of the compare of the fill with `window` + 1: (compares, those behind a wait)."""
    found, bad = 0, []
    for first, end, _ in blocks(ins, adr):
        compare = [i for i in range(first, end) if re.match(r"s_cmpk?_l[te]_[iu]32 s\d+, 0x%x$" % (window + 1), ins[i])]
        if compare and ins[end - 1].startswith("s_cbranch_scc"):
            found += 1
            bad += [ins[i] for i in range(first, compare[-1]) if re.match(r"s_waitcnt .*vmcnt\(0\)", ins[i])]
    return found, bad


def scan(path):
    res, spilled = [], spills(path)
    for name, ins, adr in kernels(path):
        res.append((name, len(ins), any(x.startswith("global_atomic_add") for x in ins), unordered_tickets(ins, adr),
                    early_reads(ins, adr), spilled[name],
                    waits_at_the_exit(ins, adr, 64) if "kvb_buffer_step_kernelILi128E" in name else None,
                    early_overwrites(ins, adr), sum(1 for x in ins if store_data(x))))
    return res


@pytest.fixture(scope="module")
def scanned(tmp_path_factory):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    files = code_objects(str(tmp_path_factory.mktemp("isa")))
    with ProcessPoolExecutor(4) as pool:
        return [r for one in pool.map(scan, files) for r in one]


def test_tickets_follow_a_barrier(scanned):
    """Each wave reads fill[slot] for itself, and the last addition of the request's workgroups makes the new count of it: a
    workgroup may only add when every wave of it has read.  The barrier stands behind the branch on the value read."""
    with_ticket = [r for r in scanned if r[2]]
    assert len(with_ticket) > 100, len(with_ticket)
    bad = [(r[0], r[3]) for r in with_ticket if r[3]]
    assert not bad, "%d kernels, e.g. %s" % (len(bad), bad[0])


def test_matrix_results_are_waited_for(scanned):
    """No path reads the result of a matrix instruction before the wait states it needs."""
    bad = [(r[0], r[4][:3]) for r in scanned if r[4]]
    assert not bad, "%d kernels, e.g. %s" % (len(bad), bad[:2])


def test_store_data_stays(scanned):
    """No path overwrites the data of a store of more than 8 bytes before the wait states it needs, stores written by hand
    (behind which the compiler places none) among them."""
    assert sum(r[8] for r in scanned) > 1000
    bad = [(r[0], r[7][:3]) for r in scanned if r[7]]
    assert not bad, "%d kernels, e.g. %s" % (len(bad), bad[:2])


@pytest.mark.parametrize("ins, found", [
    (["global_store_dwordx4 v[18:19], v[14:17], off sc1", "s_nop 0", "v_lshl_add_u64 v[14:15], v[0:1], 0, v[2:3]"], 1),
    (["global_store_dwordx4 v[18:19], v[14:17], off sc1", "s_nop 1", "v_lshl_add_u64 v[14:15], v[0:1], 0, v[2:3]"], 0),
    (["global_store_dwordx3 v18, v[14:16], s[0:1]", "v_mov_b32_e32 v16, 0"], 1),
    (["global_store_dwordx2 v[18:19], v[14:15], off sc1", "v_mov_b32_e32 v14, 0"], 0),
    (["global_store_dwordx4 v[18:19], v[14:17], off", "v_mov_b32_e32 v18, 0", "v_mov_b32_e32 v1, v14"], 0),   # addresses, reads
    (["buffer_store_dwordx4 v[4:7], v1, s[0:3], 0 offen", "s_nop 0", "v_swap_b32 v9, v7"], 1),
    (["global_store_dwordx4 v[18:19], v[14:17], off", "s_branch -> 12", "s_nop 0", "v_mov_b32_e32 v17, 0"], 1)])   # over a jump
def test_store_data_check(ins, found):
    adr = [4 * i for i in range(len(ins))]
    assert len(early_overwrites(ins + ["s_endpgm"], adr + [4 * len(ins)])) == found


# (pattern of the mangled name, registers): kernels held at three workgroups a CU that spill after all
SPILLS = [("kvb_step_kernelILi128EffLi64ELb1", 8),            # kvb_decode_flush, fp32, 64-record window
          (r"kvb_direct_mfma_kernelIN\S+EfLb1ELb0", 1)]       # kvb_direct above 64 tokens, contiguous fp32 records


def test_spills(scanned):
    """A value of a load in flight that is spilled makes the wave wait there for every load it has issued."""
    over = {}
    for r in scanned:
        allowed = max([n for pattern, n in SPILLS if re.search(pattern, r[0])], default=0)
        if r[5] > allowed:
            over[r[0]] = (r[5], allowed)
    assert not over, over


def test_short_windows_wait_for_no_atomic(scanned):
    """kvb_decode without a state: a context of up to 64 records leaves the loop over 64 records at a time without a wait for
    what the wave has in flight, the addition to the fill among it."""
    checked = [r for r in scanned if r[6] and re.search(r"Li128ENS_\S+Li1ELb[01]E", r[0])]   # 16-bit inputs, one head
    assert len(checked) == 8, [r[0] for r in checked]
    assert all(r[6][0] for r in checked), [r[0] for r in checked if not r[6][0]]
    bad = [(r[0], r[6][1]) for r in checked if r[6][1]]
    assert not bad, bad
