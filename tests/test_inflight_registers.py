"""The kernels' hand-written LDS reads are asm statements that return before
their data has arrived; a counted wait follows later.  The compiler takes the
destination registers as written at once, so nothing but the shape of the code
keeps it from copying or reusing one in between.  This test reads the assembly
of the library built here and follows every path through every kernel: no
instruction may touch the destination of an LDS read before a wait that covers
it (LDS operations complete in order, lgkmcnt(n) leaves the n youngest).  No
GPU needed."""
import os
import re
import subprocess

import pytest

from paper_2410_05985_amd import layup as LU

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def _regs(text):
    out = set()
    for lo, hi, one in re.findall(r"\bv\[(\d+):(\d+)\]|\bv(\d+)\b", text):
        out.update([int(one)] if one else range(int(lo), int(hi) + 1))
    return frozenset(out)


def _functions(lines):
    """{name: [(address, opcode, operands, branch target)]} of a disassembly."""
    funcs, cur, start = {}, None, 0
    for line in lines:
        m = re.match(r"^([0-9a-f]+) <(\S+)>:", line)
        if m:
            start, cur = int(m.group(1), 16), funcs.setdefault(m.group(2), [])
            continue
        m = re.match(r"^\s+(\S+)\s*(.*?)\s*// ([0-9A-F]+): [0-9A-F ]+(?:<\S+?(?:\+0x([0-9a-f]+))?>)?\s*$", line)
        if m and cur is not None:
            target = start + int(m.group(4) or "0", 16) if "branch" in m.group(1) else None
            cur.append((int(m.group(3), 16), m.group(1), m.group(2), target))
    return funcs


def touched_in_flight(ins):
    """Addresses of the instructions that touch an LDS read's destination too
    early.  State: for every register a read in flight may still write, the
    least number of younger LDS operations over all paths (a wait for
    lgkmcnt(n) covers it if that is at least n; n is at most 15)."""
    at = {addr: i for i, (addr, _, _, _) in enumerate(ins)}
    targets = {t for _, _, _, t in ins if t is not None}
    bad, known, work = set(), {}, [(0, {})]
    while work:
        i, state = work.pop()
        flying = dict(state)
        while i < len(ins):
            addr, op, rest, target = ins[i]
            if addr in targets:  # a block that several paths reach: go on only with news
                old = known.get(addr)
                if old is not None and all(old.get(r, 99) <= k for r, k in flying.items()):
                    break
                for r, k in (old or {}).items():
                    flying[r] = min(k, flying.get(r, 99))
                known[addr] = dict(flying)
            if op.startswith("ds_"):
                dst, _, src = rest.partition(",") if op.startswith(("ds_read", "ds_bpermute")) else ("", "", rest)
                dest = _regs(dst)
                if any(r in flying for r in _regs(src) | dest):
                    bad.add(addr)
                flying = {r: min(k + 1, 15) for r, k in flying.items()}
                flying.update((r, 0) for r in dest)
            elif op == "s_waitcnt":
                m = re.search(r"lgkmcnt\((\d+)\)", rest)
                if m:
                    flying = {r: k for r, k in flying.items() if k < int(m.group(1))}
            elif flying and any(r in flying for r in _regs(rest)):
                bad.add(addr)
            if op == "s_endpgm":
                break
            if target is not None:
                if op.startswith("s_branch"):
                    i = at[target]
                    continue
                work.append((at[target], dict(flying)))
            i += 1
    return bad


LISTING = """0000000000000100 <kernel>:
\tds_read_b128 v[4:7], v0          // 000000000100: 00000000 00000000
\tds_read_b128 v[8:11], v0         // 000000000108: 00000000 00000000
\ts_waitcnt lgkmcnt({n})           // 000000000110: 00000000
\ts_cbranch_scc1 1                 // 000000000114: 00000000 <kernel+0x1c>
\tv_mov_b32_e32 v1, v{early}       // 000000000118: 00000000
\tv_add_f32_e32 v1, v4, v1         // 00000000011C: 00000000
\ts_endpgm                         // 000000000120: 00000000
"""


@pytest.mark.parametrize("n,early,bad", [(1, 7, set()), (0, 11, set()), (1, 9, {0x118}), (2, 1, {0x11c}),
                                         (2, 5, {0x118, 0x11c})])
def test_a_read_before_its_wait_is_found(n, early, bad):
    ins = _functions(LISTING.format(n=n, early=early).splitlines())["kernel"]
    assert len(ins) == 7
    assert touched_in_flight(ins) == bad


def test_no_kernel_touches_an_lds_read_in_flight(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump of this toolchain")
    if not os.path.exists(LU.LIB_PATH):
        from paper_2410_05985_amd import build
        build.build()
    lib = tmp_path / "lib.so"
    lib.write_bytes(open(LU.LIB_PATH, "rb").read())
    subprocess.run([OBJDUMP, "--offloading", str(lib)], check=True, capture_output=True, cwd=tmp_path)
    objects = sorted(p for p in tmp_path.iterdir() if p.name.endswith("gfx950"))
    assert objects, "no gfx950 code in the library"
    kernels, bad = 0, {}
    for obj in objects:
        text = subprocess.run([OBJDUMP, "-d", str(obj)], check=True, capture_output=True, text=True).stdout
        for name, ins in _functions(text.splitlines()).items():
            if any(op.startswith("ds_read") for _, op, _, _ in ins):
                kernels += 1
                hits = touched_in_flight(ins)
                if hits:
                    bad[name] = sorted(hits)[:3]
    assert kernels > 50, kernels
    assert not bad, bad
