"""The one-launch decode steps advance a sequence's length when every attention workgroup has counted itself as a reader of the
old one.  Each of a workgroup's waves loads the length for itself, so a workgroup may count itself only behind a barrier: in the
compiled kernels no path leads from the entry to the count without one.  (A late wave that read the advanced length would be one
row ahead of its own workgroup; no run shows that reliably, the code does.)"""
import os
import re
import shutil
import subprocess

import pytest

import paper_2604_02570_amd as W

LLVM = "/opt/rocm/llvm/bin"
LIB = os.path.join(os.path.dirname(os.path.abspath(W.__file__)), "libwsvd.so")


def kernels(tmp_path, pattern):
    """{mangled name: [(address, instruction, branch target)]} of the library's kernels whose name matches."""
    lib = shutil.copy(LIB, tmp_path)
    subprocess.run([f"{LLVM}/llvm-objdump", "--offloading", lib], cwd=tmp_path, check=True, stdout=subprocess.DEVNULL)
    found = {}
    for name in sorted(os.listdir(tmp_path)):
        if not name.endswith("gfx950"):
            continue
        path = os.path.join(tmp_path, name)
        symbols = subprocess.run([f"{LLVM}/llvm-readelf", "--symbols", "--wide", path], check=True, capture_output=True, text=True).stdout
        names = {s for s in re.findall(r"FUNC .* (\S+)$", symbols, re.M) if re.search(pattern, s)}
        if not names:
            continue
        text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", f"--disassemble-symbols={','.join(sorted(names))}", path], check=True,
                              capture_output=True, text=True).stdout
        code, start = None, 0
        for line in text.splitlines():
            if head := re.match(r"([0-9a-f]+) <(\S+)>:", line):
                code, start = found.setdefault(head[2], []), int(head[1], 16)
            elif code is not None and (ins := re.match(r"\s+(\S.*?)\s*// ([0-9A-F]+):[^<]*(?:<[^>]*\+0x([0-9a-f]+)>)?", line)):
                code.append((int(ins[2], 16), ins[1], start + int(ins[3], 16) if ins[3] else None))
    return found


def unguarded(code, is_target):
    """Instructions that a path from the entry reaches without an s_barrier in front, of those that is_target picks."""
    at = {a: i for i, (a, _, _) in enumerate(code)}
    seen, todo, hit = set(), [0], []
    while todo:
        i = todo.pop()
        while i < len(code) and i not in seen:
            seen.add(i)
            _, ins, target = code[i]
            assert not ins.startswith(("s_setpc", "s_swappc", "s_call")), ins
            if is_target(ins):
                hit.append(ins)
            if ins.startswith(("s_barrier", "s_endpgm")):
                break
            if ins.startswith(("s_branch", "s_cbranch")):
                todo.append(at[target])
                if ins.startswith("s_branch"):
                    break
            i += 1
    return hit


def test_paths_are_followed():
    add = lambda ins: ins.startswith("global_atomic_add")
    code = [(0, "s_cbranch_scc0 2", 16), (4, "s_barrier", None), (8, "global_atomic_add v1, v2, s[0:1]", None), (12, "s_endpgm", None),
            (16, "v_nop", None), (20, "s_branch 8", 8)]
    assert unguarded(code, add)
    code[4] = (16, "s_barrier", None)
    assert not unguarded(code, add)


@pytest.mark.parametrize("pattern,least", [(r"k_step_f32", 48), (r"k_step_bf16", 18), (r"k_step_i8", 8)])
def test_a_workgroup_counts_itself_behind_a_barrier(tmp_path, pattern, least):
    found = kernels(tmp_path, pattern)
    assert len(found) >= least, sorted(found)
    for name, code in found.items():
        count = lambda ins: re.match(r"global_atomic_add\S* v\d+, v\d+, s", ins) is not None      # (the count is not read back)
        assert sum(count(ins) for _, ins, _ in code) == 1, name
        assert not unguarded(code, count), f"{name}: counted as a reader with no barrier behind the other waves' loads"
