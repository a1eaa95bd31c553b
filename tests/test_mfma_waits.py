"""The attention kernels issue their score products from inline assembly (results in ordinary registers),
so the compiler does not see how long those results take and inserts no waits for them: the code leaves enough
matrix instructions or wait states between.  This reads the built library and checks that distance for every
matrix instruction of every kernel, along every path."""
import os
import re
import shutil
import subprocess

import pytest

SO = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2411_16102_amd", "libblendstep.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
# passes of four clocks, and wait states until something else than the accumulation of a following matrix instruction
# may touch the result (a wait state is the issue of one instruction; the next matrix instruction issues a
# matrix instruction's passes later)
PASSES = {"v_mfma_f32_16x16x32_bf16": 4, "v_mfma_f32_32x32x16_bf16": 8}
WAITS = {4: 8, 8: 12}
LINE = re.compile(r"^\t(\S+)\s*(.*?)\s*// ([0-9A-F]+): [0-9A-F ]+(?:<([^>+]+)(?:\+0x([0-9a-f]+))?>)?")
REG = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)")


def regs(text):
    out = set()
    for kind, lo, hi, one in REG.findall(text):
        out.update((kind, r) for r in (range(int(lo), int(hi) + 1) if lo else (int(one),)))
    return frozenset(out)


def violations(listing):
    """(kernel, address, text) of instructions that touch a matrix result too early."""
    kernels, name = {}, None
    for line in listing.splitlines():
        m = re.match(r"^([0-9a-f]+) <(.+)>:$", line)
        if m:
            name = m.group(2)
            kernels[name] = (int(m.group(1), 16), [])
        m = LINE.match(line)
        if m and name:
            op, args, addr, sym, off = m.groups()
            kernels[name][1].append((int(addr, 16), op, args, int(off or "0", 16) if sym == name else None))
    bad = set()
    for name, (base, code) in kernels.items():
        if not any(op in PASSES for _, op, _, _ in code):
            continue
        at = {addr: i for i, (addr, _, _, _) in enumerate(code)}
        parsed = []
        for addr, op, args, off in code:
            parts = [regs(a) for a in args.split(", ")] if op in PASSES else None
            parsed.append((op, regs(args), parts, at.get(base + off) if off is not None and "branch" in op else None))
        # state on entry of an instruction: result register -> (wait states still to pass, its result's registers)
        entry = {0: {}}
        work = [0]
        while work:
            i = work.pop()
            state = dict(entry[i])
            while i < len(parsed):
                op, used, parts, target = parsed[i]
                if parts:   # a matrix instruction: accumulating onto the same registers is in order
                    dst, a, b, c = parts
                    # it issues once the one before it has passed
                    state = {r: (w - p + 1, whole, p) for r, (w, whole, p) in state.items() if w - p + 1 > 0}
                    for r in a | b | (c - dst) | (dst - c):
                        if r in state and state[r][1] != dst:
                            bad.add((name, code[i][0], op + " " + code[i][2]))
                    waits = 1
                else:
                    for r in used:
                        if r in state:
                            bad.add((name, code[i][0], op + " " + code[i][2]))
                    waits = 1 + (int(code[i][2], 0) if op == "s_nop" else 0)
                state = {r: (w - waits, whole, p) for r, (w, whole, p) in state.items() if w > waits}
                if parts:
                    for r in dst:
                        state[r] = (WAITS[PASSES[op]], dst, PASSES[op])
                nxt = [t for t in (target, None if op in ("s_branch", "s_endpgm") else i + 1) if t is not None and t < len(parsed)]
                follow = None
                for t in nxt:
                    have = entry.get(t)
                    if target is None and t not in entry and t == i + 1:   # straight on
                        follow = t
                        continue
                    merged = dict(have or {})
                    for r, v in state.items():
                        if r not in merged or merged[r][0] < v[0]:
                            merged[r] = v
                    if have is None or merged != have:
                        entry[t] = merged
                        work.append(t)
                if follow is None:
                    break
                i = follow
    return bad


@pytest.fixture(scope="module")
def listings(tmp_path_factory):
    if not (os.path.exists(SO) and os.path.exists(OBJDUMP)):
        pytest.skip("needs the built library and llvm-objdump")
    where = tmp_path_factory.mktemp("objects")
    shutil.copy(SO, str(where / "l.so"))
    subprocess.run([OBJDUMP, "--offloading", "l.so"], cwd=str(where), check=True, stdout=subprocess.DEVNULL)
    out = []
    for f in sorted(os.listdir(str(where))):
        if "gfx950" in f:
            out.append(subprocess.run([OBJDUMP, "-d", f], cwd=str(where), check=True, stdout=subprocess.PIPE, text=True).stdout)
    assert sum(t.count("v_mfma_f32") for t in out) > 1000
    return out


def test_no_matrix_result_is_touched_early(listings):
    found = sorted(v for t in listings for v in violations(t))
    assert not found, "%d: %s" % (len(found), found[:5])


def test_the_check_sees_a_read_that_moved_up():
    code = ("0000000000001000 <kernel>:\n"
            "\tv_mfma_f32_32x32x16_bf16 v[0:15], v[16:19], v[20:23], 0 // 000000001000: D3B50080 07332580\n"
            "%s"
            "\tv_max_f32_e32 v30, v0, v1 // 000000002000: 16000000\n"
            "\ts_endpgm // 000000002004: BF810000\n")
    mfma = "\tv_mfma_f32_32x32x16_bf16 a[%d:%d], v[16:19], v[20:23], a[%d:%d] // 00000000%04X: D3B50080 07332580\n"
    two = "".join(mfma % (r, r + 15, r, r + 15, 0x1008 + r) for r in (0, 16))
    assert violations(code % "") and violations(code % "\ts_nop 9 // 000000001008: BF800009\n")
    assert violations(code % two[:two.index("\n") + 1])
    assert not violations(code % two) and not violations(code % "\ts_nop 11 // 000000001008: BF80000B\n")
