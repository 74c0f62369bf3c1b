"""Workgroup barriers of the kernels: a wave's LDS writes are complete before it arrives.

The compiler has left out the wait that __syncthreads() implies where the barrier stands at the
top of a loop, so the sources spell it out (block_sync) and the built code is checked."""
import glob
import os
import re
import shutil
import struct
import subprocess

import pytest

import paper_2510_21956_amd as la

CSRC = os.path.join(os.path.dirname(la.library_path()), "csrc")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def test_every_barrier_goes_through_block_sync():
    found = []
    for path in glob.glob(os.path.join(CSRC, "*")):
        for n, line in enumerate(open(path), 1):
            if re.search(r"__syncthreads\s*\(\s*\)\s*;|__builtin_amdgcn_s_barrier\s*\(", line):
                found.append((os.path.basename(path), n, line.strip()))
    assert len(found) == 1 and found[0][0] == "la_common.h", found


def _code_objects(path):
    """The gfx950 code objects inside a shared library built by hipcc (offload bundles: magic,
    count, then offset, size and name of each entry)."""
    data = open(path, "rb").read()
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        pos = at + len(magic)
        count, = struct.unpack_from("<Q", data, pos)
        pos += 8
        if count < 16:
            for _ in range(count):
                off, size, n = struct.unpack_from("<QQQ", data, pos)
                name = data[pos + 24:pos + 24 + n]
                pos += 24 + n
                if b"gfx950" in name and size:
                    yield data[at + off:at + off + size]
        at = data.find(magic, at + 1)


def _barriers(listing):
    """(kernel, waits) for every s_barrier: waits is False if an LDS write can reach it along some
    path without an s_waitcnt lgkmcnt(0) in between."""
    for name, body in re.findall(r"^[0-9a-f]+ <(\S+)>:\n(.*?)(?=^[0-9a-f]+ <[^L]\S*>:|\Z)", listing,
                                 re.S | re.M):
        code, labels = [], {}
        for line in body.splitlines():
            line = line.split("//")[0].strip()
            m = re.match(r"(?:[0-9a-f]+ )?<(L\d+)>:$", line)
            if m:
                labels[m.group(1)] = len(code)
            elif line:
                code.append(line)
        preds = [[] for _ in range(len(code) + 1)]
        for i, line in enumerate(code):
            op = line.split()[0]
            if op.startswith(("s_branch", "s_cbranch")):
                target = re.search(r"<?(L\d+)>?$", line)
                assert target, line
                preds[labels[target.group(1)]].append(i)
            if op not in ("s_branch", "s_endpgm"):
                preds[i + 1].append(i)
        for i, line in enumerate(code):
            if line.split()[0] != "s_barrier":
                continue
            seen, todo, waits = set(), list(preds[i]), True
            while todo:
                k = todo.pop()
                if k in seen:
                    continue
                seen.add(k)
                op = code[k].split()[0]
                if (op == "s_waitcnt" and "lgkmcnt(0)" in code[k]) or op == "s_barrier":
                    continue
                if op.startswith("ds_write"):
                    waits = False
                    break
                todo += preds[k]
            yield name, waits


def test_built_barriers_wait_for_lds_writes(tmp_path):
    if not os.path.exists(la.library_path()):
        from paper_2510_21956_amd import build
        build.build_library()
    if shutil.which(OBJDUMP) is None:
        pytest.skip("no disassembler")
    total, bad = 0, []
    for n, obj in enumerate(_code_objects(la.library_path())):
        f = tmp_path / ("code%d.o" % n)
        f.write_bytes(obj)
        text = subprocess.run([OBJDUMP, "-d", "--symbolize-operands", "--no-show-raw-insn",
                               "--no-leading-addr", str(f)], check=True, capture_output=True,
                              text=True).stdout
        for name, waits in _barriers("\n".join(
                ("0 " + x) if re.match(r"<\S+>:$", x) else x for x in text.splitlines())):
            total += 1
            if not waits:
                bad.append(name)
    assert total > 500, total
    assert not bad, (len(bad), bad[:5])
