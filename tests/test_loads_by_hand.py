"""Loads that the attention kernels issue by hand, and wait for by number: the compiler, which takes a result to be there at once, must leave
its register alone until the wait.  In the listings each such load, and the place behind the wait that takes what it brought, name the
register and the value: the registers are the same ones, and on every way from one to the other nobody writes to them, nor on ways past all such places."""
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

from paper_2502_06282_amd import build as b

_MARK = re.compile(r"; (asked|arrived) (v\d+|v\[\d+:\d+\]) as (\d+)")
_VECTOR = re.compile(r"(?<![\w.])v(?:(\d+)|\[(\d+):(\d+)\])")


def kernels(listing):
    found, lines = {}, None
    for line in listing.splitlines():
        if m := re.match(r"(_Z\w+):", line):
            lines = found.setdefault(m[1], [])
        elif line.startswith("\t.section"):
            lines = None
        elif lines is not None:
            lines.append(line)
    return found


def moved(lines):
    """Values that are asked for in other registers than they are taken from."""
    found = {}
    for line in lines:
        if m := _MARK.search(line):
            found.setdefault(int(m[3]), (set(), set()))[m[1] == "arrived"].add(m[2])
    return {value: registers for value, registers in found.items() if registers[0] != registers[1]}


def _registers(text):
    return {r for one, lo, hi in _VECTOR.findall(text) for r in range(int(one or lo), int(one or hi) + 1)}


def _written(code):
    name, _, operands = code.strip().partition(" ")
    if "store" in name or "_lds" in name or name.startswith("ds_write") or not operands:
        return set()
    return _registers(operands if "swap" in name else operands.split(",")[0])


def overwritten(lines):
    """Loads whose registers may be written to before they are taken, on any way through the branches."""
    label = {m[1]: i for i, line in enumerate(lines) if (m := re.match(r"(\.L\w+):", line))}
    code = [line.split(";")[0] for line in lines]
    written, found = [_written(c) for c in code], []

    def behind(i):
        t = code[i].split() or [""]
        if t[0] == "s_endpgm":
            return []
        return ([label[t[1]]] if "branch" in t[0] else []) + ([i + 1] if t[0] != "s_branch" else [])

    for i, line in enumerate(lines):
        m = _MARK.search(line)
        if not m or m[1] != "asked":
            continue
        own, seen, left = _registers(m[2]), set(), behind(i)
        while left:
            k = left.pop()
            if k in seen or k >= len(lines):
                continue
            seen.add(k)
            t = _MARK.search(lines[k])
            if t and t[1] == "arrived" and t.groups()[1:] == m.groups()[1:]:
                continue
            if own & written[k]:
                found.append((m[0], code[k].strip()))
                break
            left += behind(k)
    return found


def _listing(unit):
    source, flags = unit
    cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + b.FLAGS + flags + ["-x", "hip", "-S", "--cuda-device-only", os.path.join(b.CSRC, source), "-o", "-"]
    return subprocess.run(cmd, check=True, capture_output=True, text=True, timeout=300).stdout


def test_results_stay_where_they_were_asked_for():
    units = [("tva_bf16.hip", [f"-DJK_MERGE={m}"] + b.PRELOAD) for m in range(b.MERGES)] + [("tva_wide.hip", b.UNIT_FLAGS["tva_wide.hip"])]
    with ThreadPoolExecutor(min(8, int(os.environ.get("MAX_JOBS", "8")))) as pool:
        for unit, text in zip(units, pool.map(_listing, units)):
            found = kernels(text)
            assert len(found) == (4 if unit[0] == "tva_wide.hip" else 12)
            for name, lines in found.items():
                assert sum("; asked" in line for line in lines) >= 8, name  # (lengths, a row in four pieces or more, parents)
                assert not moved(lines) and not overwritten(lines), (unit, name, moved(lines), overwritten(lines))


def test_a_moved_result_and_one_that_is_written_over_are_found():
    fine = """\tglobal_load_dword v4, v[2:3], off ; asked v4 as 0
\ts_cbranch_scc1 .LBB0_2
\tds_write_b32 v4, v1
\ts_waitcnt vmcnt(0)
\tv_mov_b32 v1, v4 ; arrived v4 as 0
\ts_branch .LBB0_3
.LBB0_2:
\ts_waitcnt vmcnt(0)
\t; arrived v4 as 0
.LBB0_3:
\tv_mov_b32_e32 v4, 0
\ts_endpgm"""
    assert not moved(fine.splitlines()) and not overwritten(fine.splitlines())
    assert moved(fine.replace("arrived v4", "arrived v9").splitlines())
    assert overwritten(fine.replace("\t; arrived v4 as 0\n", "").splitlines())          # a way without a use: given away behind it
    assert overwritten(fine.replace("ds_write_b32 v4", "v_add_u32_e32 v4").splitlines())
    assert overwritten(fine.replace("ds_write_b32 v4, v1", "v_lshlrev_b64 v[4:5], 1, v[2:3]").splitlines())
