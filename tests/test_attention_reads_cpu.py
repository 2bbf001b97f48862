"""The transposing LDS reads that the attention kernels issue in one statement and wait for in another (csrc/attention_common.h): in the generated code
nothing may touch their destinations in between, on any path.  The compiler takes those registers as written at once, so only the code that it makes can
tell; compiled for gfx950 as the library is, no GPU needed."""
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

import __graft_entry__ as build

FILES = ("attention.hip", "attention_bwd.hip")


def registers(text):
    out = set()
    for kind, lo, up, one in re.findall(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)", text):
        out |= {(kind, r) for r in range(int(lo or one), int(up or one) + 1)}
    return out


def functions(asm):
    name, lines = None, []
    for line in asm.splitlines():
        start = re.match(r"(_Z\w+):", line)
        if start:
            name, lines = start.group(1), []
        elif line.startswith(".Lfunc_end") and name:
            yield name, lines
            name = None
        elif name:
            lines.append(line)


def unsafe(lines):
    """(hand-issued groups of reads, what touches a destination ahead of its wait, paths that end without one)"""
    label = {m.group(1): i for i, m in ((i, re.match(r"(\.LBB\w+):", l)) for i, l in enumerate(lines)) if m}
    groups, touched, open_ends, at = 0, [], 0, 0
    hand = False
    while at < len(lines):
        hand = "#ASMSTART" in lines[at] or (hand and "#ASMEND" not in lines[at])
        if not (hand and "ds_read_b64_tr_b16" in lines[at]):
            at += 1
            continue
        groups, dest = groups + 1, set()
        while "ds_read_b64_tr_b16" in lines[at]:
            dest |= registers(lines[at].split(",")[0])
            at += 1
        seen, todo = set(), [at]
        while todo:
            i = todo.pop()
            while i not in seen:
                seen.add(i)
                code = lines[i].split(";")[0].strip()
                if code.startswith("s_waitcnt") and "lgkmcnt(0)" in code:
                    break
                if code.startswith("s_endpgm"):
                    open_ends += 1
                    break
                if code and not code.startswith((".", "s_")) and registers(code) & dest:
                    touched.append(code)
                branch = re.match(r"s_(c?)branch\w*\s+(\.LBB\w+)", code)
                if branch:
                    todo.append(label[branch.group(2)])
                    if not branch.group(1):
                        break
                i += 1
    return groups, touched, open_ends


def assembly(file):
    cmd = [build.HIPCC, *build.FLAGS, *build.EXTRA_FLAGS.get(file, []), "-w", "--cuda-device-only", "-S", os.path.join(build.CSRC, file), "-o", "-"]
    return subprocess.run(cmd, capture_output=True, text=True, check=True).stdout


def test_nothing_touches_a_read_in_flight():
    with ThreadPoolExecutor(len(FILES)) as pool:
        code = list(pool.map(assembly, FILES))
    kernels = 0
    for file, asm in zip(FILES, code):
        for name, lines in functions(asm):
            groups, touched, open_ends = unsafe(lines)
            kernels += groups > 0
            assert not touched and not open_ends, (file, name, touched[:3], open_ends)
    assert kernels >= 20          # the pair, split, one-group, woven and wide kernels in their forms: the patterns above still find them


def test_the_check_finds_one():
    good = ["\t;;#ASMSTART", "\tds_read_b64_tr_b16 v[2:3], v9", "\t;;#ASMEND", ".LBB0_1:", "\tv_add_f32 v4, v5, v6", "\ts_cbranch_scc0 .LBB0_1",
            "\ts_waitcnt lgkmcnt(0)", "\tv_mov_b32 v4, v3", "\ts_endpgm"]
    assert unsafe(good) == (1, [], 0)
    assert unsafe(good[:6] + ["\tv_mov_b32 v1, v3"] + good[6:])[1] == ["v_mov_b32 v1, v3"]
    assert unsafe(good[:4] + ["\tv_mov_b32 v2, v7"] + good[4:])[1] == ["v_mov_b32 v2, v7"]
    assert unsafe(good[:6] + good[7:])[2] == 1
