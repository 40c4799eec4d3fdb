"""The matrix kernels read their LDS fragments with inline asm, whose destination registers the compiler takes as
written at once.  A register that such a read has not filled yet must not be touched: a late return would replace what
was put there.  Followed here over every path of the machine code of the built library's expert-FFN kernels."""
import re
import shutil
import subprocess

import pytest

from paper_2407_00599_amd import api

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
REG = re.compile(r"\b([va])(?:(\d+)\b|\[(\d+):(\d+)\])")
LATER_MAX = 16      # more LDS operations than lgkmcnt can leave outstanding


def registers(text):
    out = []
    for kind, one, lo, hi in REG.findall(text):
        out += [kind + str(i) for i in (range(int(one), int(one) + 1) if one else range(int(lo), int(hi) + 1))]
    return out


def parse(listing):
    """{function: [(address, mnemonic, operands, branch target or None)]}"""
    funcs, cur = {}, None
    for line in listing.splitlines():
        m = re.match(r"^([0-9a-f]+) <(.+)>:$", line)
        if m:
            base, name = int(m.group(1), 16), m.group(2)
            cur = funcs.setdefault(name, [])
            continue
        m = re.match(r"^\s+(\S+)\s*(.*?)\s*// ([0-9A-F]+): [0-9A-F ]+(?:<.*?(\+0x[0-9a-f]+)?>)?$", line)
        if m and cur is not None:
            op, args, addr, off = m.groups()
            target = base + int(off or "0", 16) if op.startswith(("s_cbranch", "s_branch")) else None
            cur.append((int(addr, 16), op, args, target))
    return funcs


def step(state, op, args):
    """Registers with a read in flight -> how many LDS operations were issued after it (the smallest count over the
    paths; LDS operations of a wave return in order).  Returns the registers that the instruction must not touch."""
    if op == "s_waitcnt":
        m = re.search(r"lgkmcnt\((\d+)\)", args)
        if m:
            n = int(m.group(1))
            for r in [r for r, later in state.items() if later >= n]:
                del state[r]
        return []
    regs = registers(args)
    bad = [r for r in regs if r in state]
    if op.startswith("ds_"):
        for r in state:
            state[r] = min(state[r] + 1, LATER_MAX)
        if re.match(r"ds_(read|bpermute|permute|swizzle)", op):
            for r in registers(args.split(",")[0]):
                state[r] = 0
    return bad


def hazards(code):
    """Instructions that touch a register whose LDS read may still be in flight."""
    at = {c[0]: i for i, c in enumerate(code)}
    leaders = {0}
    for i, (_, op, _, target) in enumerate(code):
        if target is not None:
            leaders |= {at[target], i + 1}
    entry, work, found = {0: {}}, [0], set()
    while work:
        i = work.pop()
        state = dict(entry[i])
        while True:
            addr, op, args, target = code[i]
            for r in step(state, op, args):
                found.add((addr, op, args, r))
            nxt = [] if op in ("s_endpgm", "s_branch", "s_setpc_b64") else [i + 1]
            if target is not None:
                nxt.append(at[target])
            if nxt == [i + 1] and i + 1 not in leaders:
                i += 1
                continue
            break
        for n in nxt:
            old = entry.get(n)
            new = dict(state) if old is None else dict(old)
            for r, later in state.items():
                new[r] = min(new.get(r, LATER_MAX), later)
            if old != new:
                entry[n] = new
                work.append(n)
    return sorted(found)


def test_checker():
    code = lambda *rows: [(4 * i, op, args, t) for i, (op, args, t) in enumerate(rows)]
    read, add, end = ("ds_read_b128", "v[4:7], v1", None), ("v_add_f32_e32", "v5, v2, v3", None), ("s_endpgm", "", None)
    wait = lambda n: ("s_waitcnt", f"vmcnt(0) lgkmcnt({n})", None)
    assert [h[3] for h in hazards(code(read, add, wait(0), end))] == ["v5"]
    assert not hazards(code(read, wait(0), add, end))
    assert hazards(code(read, wait(1), add, end))
    assert not hazards(code(read, ("ds_write_b32", "v1, v2", None), wait(1), add, end))
    # around a loop: the read at its end meets the write at its beginning
    assert hazards(code(add, read, ("s_cbranch_scc1", "", 0), wait(0), end))
    # one path waits, the other does not
    assert hazards(code(read, ("s_cbranch_scc1", "", 12), wait(0), add, end))


@pytest.mark.skipif(shutil.which(OBJDUMP) is None, reason="needs the ROCm disassembler")
def test_no_register_is_touched_before_its_lds_read(tmp_path):
    api.lib()
    shutil.copy(api.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp_path, check=True, capture_output=True)
    kernels, found = 0, []
    for obj in sorted(tmp_path.glob("lib.so.*gfx950")):
        out = subprocess.run([OBJDUMP, "-d", obj.name], cwd=tmp_path, check=True, capture_output=True, text=True).stdout
        for name, code in parse(out).items():
            if "ffn_gemm_dma" in name or "ffn_bwd_trio" in name:
                kernels += 1
                found += [(name, hex(a), op, args, r) for a, op, args, r in hazards(code)]
    assert kernels >= 20, kernels
    assert not found, (len(found), found[:20])
