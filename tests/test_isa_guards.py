"""Guards on the generated code of the decode and prefill kernels (no GPU needed).

The decode kernel issues its loads through hand-written instructions that the compiler does not
track (so that it places no wait for them inside the tile loop); the waits are explicit.  That is
only correct while the compiler never reads a destination register of such a load between the load
and the next wait - e.g. through a register-to-register copy that joins two definitions.  This test
compiles the file to assembly and checks exactly that, for every instantiation of the kernel
(and the same for the scalar loads of the table entries in the prologue of both decode kernels).
The prefill kernels' hand-written loads go to LDS and have no destination registers; what is checked
of them is the register that holds the LDS address.
"""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _registers(text):
    used = set()
    for m in re.finditer(r"v\[(\d+):(\d+)\]", text):
        used.update(range(int(m.group(1)), int(m.group(2)) + 1))
    for m in re.finditer(r"\bv(\d+)\b", text):
        used.add(int(m.group(1)))
    return used


HAND = "  ;hand"        # suffix of an instruction that comes from an inline-assembly block


def _instructions(lines):
    """Instruction and label lines of a function, comments dropped; instructions between the
    compiler's markers of an inline-assembly block carry the suffix HAND.  The kernel's landing
    marks (an assembly comment `; landed <register>` right behind an explicit wait) are kept as
    pseudo-instructions `landed <register>`."""
    out, hand = [], False
    for raw in lines:
        if "#ASMSTART" in raw:
            hand = True
        elif "#ASMEND" in raw:
            hand = False
        m = re.match(r"\s*; landed (\S+)", raw)
        if hand and m:
            out.append("landed " + m.group(1) + HAND)
            continue
        l = raw.split(";")[0].strip()
        if l:
            out.append(l + HAND if hand else l)
    return out


def reads_of_inflight_registers(body, by_marks=False):
    """(load line, offending line) pairs: instructions that touch (read or write) a destination
    register of a hand-written vector-memory load (one from an inline-assembly block, which the
    compiler neither sees nor waits for) before the place the source names as the point where the
    load has landed.

    The control-flow graph of the function is explored with a small abstract state:
      * the registers with such a load possibly outstanding - a hand-written load (or an atomic
        that returns a value) adds its destination; a landing mark (the kernel puts one right
        behind the explicit wait that covers the load) or a wait for all vector-memory operations
        removes it;
      * the 64-bit scalar flags the compiler's structurizer sets to -1 or 0 and branches on later
        (`s_mov_b64 s[a:b], -1` or `s_cselect_b64 s[a:b], -1, 0` ... `s_and_b64 vcc, exec, s[a:b]`
        ... `s_cbranch_vccz`), so that several branches on one flag are not taken in
        contradictory ways.
    States that differ are followed separately; every (instruction, state) pair is visited once.
    Whether the count of a partial wait is right is not checked here: that is the kernel's own
    bookkeeping, which the parity tests exercise.
    by_marks: landing marks alone count.  A destination that no mark names on some path is free to the compiler
    from the load on, whatever wait the source has there."""
    n = len(body)
    hand = [l.endswith(HAND) for l in body]
    body = [l[:-len(HAND)] if l.endswith(HAND) else l for l in body]
    labels = {l[:-1]: i for i, l in enumerate(body) if l.endswith(":")}
    found = set()

    def first_operand_sgprs(line, op):
        first = line[len(op):].split(",")[0]
        regs = set(int(x) for x in re.findall(r"\bs(\d+)\b", first))
        for m in re.finditer(r"s\[(\d+):(\d+)\]", first):
            regs.update(range(int(m.group(1)), int(m.group(2)) + 1))
        return regs

    def step(i, state):
        """-> list of (next index, next state); state = (outstanding, flags, vcc)"""
        out_regs, flags, vcc = state
        line = body[i]
        op = line.split()[0]
        nxt = [i + 1] if i + 1 < n else []
        if op.endswith(":") or op.startswith("."):
            return [(j, state) for j in nxt]
        if op == "s_endpgm":
            return []
        if op == "s_waitcnt":
            if "vmcnt(0)" in line and not by_marks:
                out_regs = frozenset()
            return [(j, (out_regs, flags, vcc)) for j in nxt]
        if op == "landed":
            regs = _registers(line[len(op):])
            out_regs = frozenset(x for x in out_regs if x[0] not in regs)
            return [(j, (out_regs, flags, vcc)) for j in nxt]
        m = re.match(r"s_branch (\S+)$", line)
        if m:
            return [(labels[m.group(1)], state)]
        m = re.match(r"s_cbranch_(\w+) (\S+)$", line)
        if m:
            kind, target = m.group(1), labels[m.group(2)]
            # The lane mask can only be empty right behind an instruction that narrows it (the
            # compiler then skips the masked region with `s_cbranch_execz`).  Anywhere else - behind
            # the `s_or_b64 exec, exec, saved` that closes a region, or in a block that does not
            # write the mask - it is the non-empty mask the wave arrived with, and the branches
            # the structurizer puts there are decided: execz never taken, execnz always.
            narrowed = False
            for k in range(i - 1, -1, -1):      # the last write of the mask in this basic block
                if body[k].endswith(":") or body[k].startswith(("s_branch", "s_cbranch")):
                    break
                if re.search(r"\bexec\b", body[k].split(",")[0]) or "saveexec" in body[k] or body[k].startswith("v_cmpx"):
                    narrowed = not re.match(r"s_or_b64 exec, exec, s\[\d+:\d+\]$", body[k])
                    break
            if kind == "execz" and not narrowed:
                return [(j, state) for j in nxt]
            if kind == "execnz" and not narrowed:
                return [(target, state)]
            if kind in ("vccz", "vccnz") and isinstance(vcc, int):
                taken = (vcc == 0) == (kind == "vccz")
                return [(target, state)] if taken else [(j, state) for j in nxt]
            if kind in ("vccz", "vccnz") and vcc is not None:
                # vcc mirrors a flag whose value (-1 or 0) is not known yet: each way out of the
                # branch learns it
                key, same = vcc
                def learned(vcc_value):
                    val = vcc_value if same else -1 - vcc_value
                    fl = frozenset(f for f in flags if f[0] != key) | {(key, val)}
                    return (out_regs, fl, vcc_value)
                vcc_if_taken = 0 if kind == "vccz" else -1
                return [(target, learned(vcc_if_taken))] + [(j, learned(-1 - vcc_if_taken)) for j in nxt]
            return [(j, state) for j in nxt] + [(target, state)]
        # ordinary instruction: hazards first
        is_hand_load = hand[i] and op.startswith(("global_load", "global_atomic")) and not op.startswith("global_load_lds")
        # (a hand-written load may be issued again to the registers of one that is still
        # outstanding - an early request repeated with other addresses: loads return in order, the
        # later one wins - so only its address operands count as touched)
        touched = _registers(",".join(line[len(op):].split(",")[1:]) if is_hand_load else line[len(op):])
        for reg, k in out_regs:
            if reg in touched:
                found.add((body[k], line))
        if is_hand_load:
            dst = set()
            m = re.match(r"global_load_\w+ (v\[\d+:\d+\]|v\d+),", line)
            if m:
                dst = _registers(m.group(1))
            m = re.match(r"global_atomic_\w+ (v\d+), v", line)       # an atomic that returns a value
            if m and " sc0" in line:
                dst = _registers(m.group(1))
            out_regs = frozenset(x for x in out_regs if x[0] not in dst) | frozenset((r, i) for r in dst)
        # flags and vcc
        m = re.match(r"s_mov_b64 s\[(\d+):(\d+)\], (-1|0)$", line)
        m1 = re.match(r"s_cselect_b64 s\[(\d+):(\d+)\], (-1, 0|0, -1)$", line)
        m2 = re.match(r"s_(and|andn2)_b64 vcc, exec, s\[(\d+):(\d+)\]$", line)
        if m:
            key = (int(m.group(1)), int(m.group(2)))
            flags = frozenset(f for f in flags if f[0] != key) | {(key, int(m.group(3)))}
        elif m1:      # -1 or 0, not known which: "U"
            key = (int(m1.group(1)), int(m1.group(2)))
            flags = frozenset(f for f in flags if f[0] != key) | {(key, "U")}
        elif m2:
            key = (int(m2.group(2)), int(m2.group(3)))
            val = dict(flags).get(key)
            if val is None:
                vcc = None
            elif val == "U":
                vcc = (key, m2.group(1) == "and")
            else:
                vcc = val if m2.group(1) == "and" else -1 - val
        else:
            if "vcc" in line:
                vcc = None
            if flags:
                killed = first_operand_sgprs(line, op)
                if killed:
                    flags = frozenset(f for f in flags if not (set(range(f[0][0], f[0][1] + 1)) & killed))
        return [(j, (out_regs, flags, vcc)) for j in nxt]

    start = (0, (frozenset(), frozenset(), None))
    seen, work = {start}, [start]
    while work:
        i, state = work.pop()
        for nxt in step(i, state):
            if nxt not in seen:
                seen.add(nxt)
                work.append(nxt)
        assert len(seen) < 2000000, "state explosion"
    return sorted(found)


def reads_of_inflight_scalars(body):
    """The same for the hand-written scalar table loads (s_load_dword[x2] ..., 0x0 from a pointer other
    than the kernel-argument segment s[0:1]): instructions that touch their destinations before the next
    s_waitcnt lgkmcnt(0), and loads into the registers of an earlier one without a wait of the source's own in
    between (scalar loads return in any order, so that the earlier one may be the last to arrive; a wait that
    the compiler placed for something else may be gone with its next version)."""
    found, pending, unwaited = [], set(), set()
    hand = [l.endswith(HAND) for l in body]
    body = [l[:-len(HAND)] if l.endswith(HAND) else l for l in body]
    for line, by_hand in zip(body, hand):
        op = line.split()[0]
        if "lgkmcnt(0)" in line:
            pending = set()
            if by_hand:
                unwaited = set()
            continue
        m = re.match(r"s_load_dword(x2)? (?:s(\d+)|s\[(\d+):(\d+)\]), s\[(\d+):\d+\], 0x0$", line)
        if pending and not op.endswith(":") and not op.startswith("."):
            touched = line[len(op):] if not (m and by_hand) else line.split(",")[1]
            used = set(int(x) for x in re.findall(r"\bs(\d+)\b", touched))
            for x in re.finditer(r"s\[(\d+):(\d+)\]", touched):
                used.update(range(int(x.group(1)), int(x.group(2)) + 1))
            if used & pending:
                found.append(line)
        if m and m.group(5) != "0":
            first = int(m.group(2) or m.group(3))
            regs = set(range(first, int(m.group(4) or first) + 1))
            if by_hand and regs & unwaited:
                found.append(line)
            pending |= regs
            if by_hand:
                unwaited |= regs
    return found


def argument_lines_asked_for_late(body):
    """64-byte lines of the kernel arguments (s[0:1]) whose first load stands behind the first scalar wait: each is a miss of its own in
    the chain in front of the first tile.  What stands in front of the aligned entry of a kernel with preloaded arguments is for firmware without preloading."""
    entry = body.index(".p2align\t8") + 1 if ".p2align\t8" in body else 0
    asked, late, waited = set(), [], False
    for line in body[entry:]:
        m = re.match(r"s_load_dword(?:x(\d+))? \S+ s\[0:1\], 0x([0-9a-f]+)$", line)
        if m:
            at, size = int(m.group(2), 16), 4 * int(m.group(1) or 1)
            lines = set(range(at // 64, (at + size - 1) // 64 + 1))
            late += [(n, line) for n in sorted(lines - asked) if waited]
            asked |= lines
        elif line.startswith("s_waitcnt") and "lgkmcnt" in line:
            waited = True
        elif re.match(r"s_\w+ (s[01]|s\[\d+:\d+\]),", line) and not line.startswith(("s_cmp", "s_bitcmp")):
            first = [int(x) for x in re.findall(r"\d+", line.split(",")[0].split()[1])]
            if first[0] <= 1:                  # the address is gone
                break
    return late


def test_checker_flags_an_argument_line_behind_the_wait():
    load = lambda at, n="": "s_load_dword%s s[8:9], s[0:1], 0x%x" % (n, at)
    assert not argument_lines_asked_for_late([load(0), load(0x40), "s_waitcnt lgkmcnt(0)", load(0x20, "x8"), load(0x7c)])
    assert argument_lines_asked_for_late([load(0), load(0x40), "s_waitcnt lgkmcnt(0)", load(0x60, "x16")]) == [(2, load(0x60, "x16"))]
    assert argument_lines_asked_for_late([load(0x80), "s_waitcnt lgkmcnt(0)", ".p2align\t8", load(0), "s_waitcnt lgkmcnt(0)", load(0x80)])
    assert not argument_lines_asked_for_late([load(0), "s_waitcnt lgkmcnt(0)", "s_add_u32 s0, s0, s2", load(0x80)])


def test_checker_flags_a_copy_of_an_inflight_register():
    bad_s = ["s_load_dword s7, s[4:5], 0x0", "s_add_i32 s9, s7, 1", "s_waitcnt lgkmcnt(0)"]
    good_s = ["s_load_dword s7, s[4:5], 0x0", "s_add_i32 s9, s8, 1", "s_waitcnt lgkmcnt(0)",
              "s_add_i32 s9, s7, 1"]
    assert reads_of_inflight_scalars(bad_s) and not reads_of_inflight_scalars(good_s)
    assert reads_of_inflight_scalars([bad_s[0], "s_add_i32 s7, s8, 1", bad_s[2]])         # (written while it is out)
    twice, wait = "s_load_dword s7, s[4:5], 0x0" + HAND, "s_waitcnt lgkmcnt(0)"
    for between in ([], [wait], ["s_load_dword s9, s[4:5], 0x0" + HAND]):                 # (the compiler's wait is its own business)
        assert reads_of_inflight_scalars([twice] + between + [twice])
    assert not reads_of_inflight_scalars([twice, wait + HAND, twice, "s_add_i32 s9, s8, 1"])
    H = lambda lines: [l + HAND if l.startswith(("global_", "landed")) else l for l in lines]
    check = lambda lines: reads_of_inflight_registers(H(lines))
    bad = ["global_load_dwordx4 v[8:11], v[2:3], off", "v_mov_b32_e32 v20, v9", "s_waitcnt vmcnt(0)"]
    good = ["global_load_dwordx4 v[8:11], v[2:3], off", "v_mov_b32_e32 v21, v20", "s_waitcnt vmcnt(0)",
            "ds_write_b128 v1, v[8:11]"]
    assert check(bad) and not check(good)
    # a wait for everything does not keep a register that no mark names behind it
    unnamed = ["global_load_dwordx4 v[8:11], v[2:3], off", "s_waitcnt vmcnt(0)", "v_mov_b32_e32 v9, v20"]
    assert not check(unnamed) and reads_of_inflight_registers(H(unnamed), by_marks=True)
    assert not reads_of_inflight_registers(H(unnamed[:2] + ["landed v[8:11]", unnamed[2]]), by_marks=True)
    assert not reads_of_inflight_registers(bad)          # a load the compiler knows about is its business
    # a partial wait covers what the landing marks behind it name, nothing else
    partial = ["global_load_dwordx4 v[8:11], v[2:3], off", "global_load_lds_dwordx4 v[4:5], off",
               "global_load_dwordx4 v[12:15], v[2:3], off", "s_waitcnt vmcnt(1)", "landed v[8:11]",
               "v_mov_b32_e32 v20, v9"]
    assert not check(partial)
    assert check(partial + ["v_mov_b32_e32 v21, v13"])
    assert check(partial[:4] + ["v_mov_b32_e32 v20, v9"])
    # overwriting a register whose load is outstanding is flagged as well
    assert check(["global_load_dwordx4 v[8:11], v[2:3], off", "v_mov_b32_e32 v9, v20"])
    # an atomic that returns a value is a load
    assert check(["global_atomic_add v7, v[4:5], v2, off sc0", "v_readfirstlane_b32 s0, v7"])
    assert not check(["global_atomic_add v7, v[4:5], v2, off sc0", "s_waitcnt vmcnt(0)", "landed v7",
                      "v_readfirstlane_b32 s0, v7"])
    # across the back-edge of a loop: loaded at the bottom of a pass, read at the top of the next
    loop = [".LBB0_1:", "v_add_f32_e32 v30, v30, v8", "s_waitcnt vmcnt(0)",
            "global_load_dwordx4 v[8:11], v[2:3], off", "s_cbranch_scc1 .LBB0_1", "s_waitcnt vmcnt(0)"]
    assert check(loop)
    assert not check([loop[0], loop[2], loop[1]] + loop[3:])
    # the two arms of a branch do not see each other's loads, the code behind the join sees both
    arms = ["s_cbranch_scc1 .LBB0_2", "global_load_dwordx4 v[8:11], v[2:3], off", "s_branch .LBB0_3",
            ".LBB0_2:", "v_mov_b32_e32 v8, 0", ".LBB0_3:", "s_waitcnt vmcnt(0)", "v_mov_b32_e32 v20, v8"]
    assert not check(arms)
    assert check(arms[:6] + ["v_mov_b32_e32 v20, v8"])
    # the marks survive the reading of the compiler's output
    got = _instructions(["\t;;#ASMSTART", "\ts_waitcnt vmcnt(4)", "\t;;#ASMEND", "\t;;#ASMSTART",
                         "\t; landed v[62:65]", "\t;;#ASMEND", "\tv_mov_b32_e32 v1, v62 ; comment"])
    assert got == ["s_waitcnt vmcnt(4)" + HAND, "landed v[62:65]" + HAND, "v_mov_b32_e32 v1, v62"]


SET_M0 = r"s_mov_b32 m0, (s\d+|vcc_lo|vcc_hi)$"


def check_m0(body):
    """M0 (the LDS address of a DMA load) is set by the hand-written sequence itself, right in front of
    every such load, and nothing else in the kernel touches it.  -> number of such loads"""
    n = 0
    for i, l in enumerate(body):
        if l.startswith("global_load_lds"):
            assert re.match(SET_M0, body[i - 2]) and body[i - 1].startswith("s_nop"), body[i - 2:i + 1]
            n += 1
        elif re.search(r"\bm0\b", l):
            assert re.match(SET_M0, l) and body[i + 2].startswith("global_load_lds"), body[i:i + 3]
    return n


def _assembly(name, tmp_path):
    import __graft_entry__ as G
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("no hipcc")
    src = os.path.join(ROOT, "paper_2510_13797_amd", "csrc", name)
    out = str(tmp_path / (name + ".s"))
    flags = [f for f in G.HIPCC_FLAGS if f not in ("-shared", "-Wall")] + G.FILE_FLAGS.get(name, [])
    subprocess.check_call([hipcc] + flags + ["-w", "-I", os.path.join(ROOT, "include"), "-S",
                                             "--cuda-device-only", src, "-o", out])
    return open(out).read().split("\n")


def test_m0_check_flags_other_uses():
    load = ["s_mov_b32 m0, s4", "s_nop 0", "global_load_lds_dwordx4 v1, s[2:3]"]
    assert check_m0(load + load) == 2 and check_m0(["s_mov_b32 m0, vcc_lo"] + load[1:]) == 1
    for bad in (load[1:], load[:1] + load[2:], ["s_mov_b32 m0, 0"] + load[1:], ["s_mov_b32 m0, s4", "v_mov_b32_e32 v1, v2"] + load, ["s_add_i32 s3, m0, 1"] + load):
        with pytest.raises(AssertionError):
            check_m0(["s_nop 0", "s_nop 0"] + bad + ["s_nop 0", "s_nop 0"])


# Instantiations, and workgroups of four waves that share a compute unit at d = 128 and 64: what the rules of the launches reckon with
@pytest.mark.parametrize("name,kernels", [("bc_prefill.hip", {"prefill_kernel": (8, 3, 4)}),
                                          ("bc_prefill_bwd.hip", {"prefill_bwd_dq_kernel": (4, 2, 3), "prefill_bwd_dkv_kernel": (2, 3, 4),
                                                                  "prefill_bwd_joined_kernel": (2, 2, 3)})])
def test_prefill_kernels_set_m0_in_front_of_every_load_to_lds(name, kernels, tmp_path):
    text = _assembly(name, tmp_path)
    for kernel, (count, wide, narrow) in kernels.items():
        starts = [i for i, l in enumerate(text) if re.match(r"^_ZN2bc\d\d%s\w+:" % kernel, l)]
        assert len(starts) == count, (kernel, len(starts))
        for s in starts:
            e = next(i for i in range(s, len(text)) if text[i].startswith(".Lfunc_end"))
            marked = _instructions(text[s:e])
            body = [l[:-len(HAND)] if l.endswith(HAND) else l for l in marked]
            # a tile of K (Q) and of V (dO) at least, from each of the places that ask for one
            assert check_m0(body) >= 4, text[s][:80]
            # loops start where they are told to, not where the code in front of them happens to end
            if name == "bc_prefill.hip":
                loops = sum("Loop Header" in l for l in text[s:e])
                assert loops >= 8 and sum(l.strip() == ".p2align\t4" for l in text[s:e]) >= loops // 2, text[s][:80]
            # no hand-written load has a destination register, and nothing of the tile loop lives in scratch
            assert all("load_lds" in l for l in marked if l.endswith(HAND) and l.startswith("global_load")), text[s][:80]
            assert not any(l.startswith(("scratch_", "buffer_")) for l in body), text[s][:80]
            waves = next(int(x.group(1)) for x in (re.match(r"; Occupancy: (\d+)", l) for l in text[e:]) if x)
            assert waves >= (wide if "ILi128E" in text[s] else narrow), (text[s][:80], waves)


def _arguments(text):
    """Of every kernel: (offset, kind) of its arguments, from the metadata the compiler leaves behind the code."""
    found, args = {}, []
    for l in text[next(i for i, l in enumerate(text) if l.startswith("amdhsa.kernels:")):]:
        m = re.match(r"(    | {6}- | {8})\.(offset|value_kind|name): +(\S+)$", l)
        if l.startswith("    .args:"):
            args = []
        elif m and m.group(2) == "offset":
            args.append([int(m.group(3)), None])
        elif m and m.group(2) == "value_kind":
            args[-1][1] = m.group(3)
        elif m and m.group(1) == "    ":
            found[m.group(3)] = [tuple(a) for a in args if not a[1].startswith("hidden_")]
    return found


@pytest.mark.parametrize("name,count", [("bc_prefill.hip", 8), ("bc_prefill_bwd.hip", 11)])
def test_kernels_that_read_tables_of_their_arguments_have_one_argument(name, count, tmp_path):
    # they find the tables at a fixed place behind the start of the argument segment, where their parameters lie
    kernels = {k: a for k, a in _arguments(_assembly(name, tmp_path)).items() if "Params" in k}
    assert len(kernels) == count and all(a == [(0, "by_value")] for a in kernels.values()), kernels


def test_decode_kernel_never_reads_a_register_whose_load_is_in_flight(tmp_path):
    text = _assembly("bc_decode.hip", tmp_path)
    starts = [i for i, l in enumerate(text) if re.match(r"^_ZN2bc\d\ddecode_(lds|lds_cut|valu)_kernel\w+:", l)]
    assert len(starts) >= 16 + 5 + 20 + 20
    for s in starts:
        e = next(i for i in range(s, len(text)) if text[i].startswith(".Lfunc_end"))
        marked = _instructions(text[s:e])
        body = [l[:-len(HAND)] if l.endswith(HAND) else l for l in marked]
        if "decode_lds_" in text[s]:
            assert any(l.startswith("global_load_lds_dwordx4") for l in body)
            check_m0(body)
            # the landing marks are there, each behind one of the explicit waits
            marks = [i for i, l in enumerate(body) if l.startswith("landed ")]
            assert len(marks) >= 6, text[s][:80]
            for i in marks:
                back = [l for l in body[max(0, i - 40):i] if not l.startswith("landed ")]
                assert any(l.startswith("s_waitcnt vmcnt(") for l in back[-24:]), (text[s][:80], body[i])
            assert not reads_of_inflight_registers(marked, by_marks=True), (text[s][:80], reads_of_inflight_registers(marked, by_marks=True)[:3])
        if "decode_lds_cut" in text[s]:
            # waves without a tile make a round trip before they take their ticket, so as not to be in front of the others at the counter
            tickets = [i for i, l in enumerate(marked) if l.startswith("global_atomic_add v") and l.endswith(HAND)]
            assert any(re.match(r"global_load_dwordx4 \S+ \S+ off" + HAND, l) for i in tickets for l in marked[i - 30:i]), text[s][:80]
        if "decode_valu_kernel" in text[s]:
            # the plan takes two workgroups of four waves per compute unit, one of the widest groups of bf16 rows
            m = re.search(r"decode_valu_kernelI(f|NS_6bf16_tE)Li\d+ELi(\d)E", text[s])
            one = m.group(1) != "f" and int(m.group(2)) >= 4
            waves = next(int(x.group(1)) for x in (re.match(r"; Occupancy: (\d+)", l) for l in text[e:]) if x)
            assert (waves == 1) if one else (waves >= 2), (text[s][:80], waves)
        # the arguments' lines travel together
        assert not argument_lines_asked_for_late(body), (text[s][:80], argument_lines_asked_for_late(body)[:3])
        # the six table entries of the prologue (both kernels)
        assert sum(1 for l in body if re.match(r"s_load_dword(x2)? \S+ s\[(?!0:1)\d+:\d+\], 0x0$", l)) >= 6, text[s][:80]
        assert not reads_of_inflight_scalars(marked), (text[s][:80], reads_of_inflight_scalars(marked)[:3])


def test_fp32_decode_kernels_leave_the_ticket_alone_until_it_is_there(tmp_path):
    # the step's ticket is taken by hand and looked at behind the merge of the waves
    text = _assembly("bc_decode.hip", tmp_path)
    starts = [i for i, l in enumerate(text) if re.match(r"^_ZN2bc18decode_valu_kernelIf\w+Lb0EEE\w+:", l)]      # (on matrix instructions)
    assert len(starts) == 20
    for s in starts:
        e = next(i for i in range(s, len(text)) if text[i].startswith(".Lfunc_end"))
        marked = _instructions(text[s:e])
        assert any(l.startswith("global_atomic_add v") and l.endswith(HAND) for l in marked), text[s][:80]
        assert sum(1 for l in marked if l.startswith("landed ")) >= 1, text[s][:80]
        assert not reads_of_inflight_registers(marked), (text[s][:80], reads_of_inflight_registers(marked)[:3])
        assert not any(l.startswith(("scratch_", "buffer_")) for l in marked), text[s][:80]
