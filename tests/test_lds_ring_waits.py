"""CPU: waits of the attention kernels' LDS ring, read from the built library's own gfx950 code.

A wave's reads of the ring buffer that a step retires must have returned when the wave arrives at the
step's barrier: behind it any other wave copies the next tile but three into that buffer. The compiler may
move the matrix products (and the waits for their operands) past the barrier, so this is checked on what
it made: every path through a kernel is followed with the list of its LDS reads still in flight."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2606_01839_amd import conserve

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
LINE = re.compile(r"^\s+(\S+)\s*(.*?)\s*// ([0-9A-F]+):.*?(?:<[^+>]*(?:\+0x([0-9a-f]+))?>)?$")


def _kernels(tmp):
    """{kernel name: [(address, opcode, operands, branch target or None)]} of the library's device code."""
    lib = os.path.join(tmp, "lib.so")
    shutil.copy(conserve._LIB_PATH, lib)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, capture_output=True, cwd=tmp)
    out = {}
    for f in sorted(os.listdir(tmp)):
        if not f.endswith("gfx950"):
            continue
        text = subprocess.run([OBJDUMP, "-d", os.path.join(tmp, f)], check=True, capture_output=True, text=True).stdout
        body, start = None, 0
        for line in text.splitlines():
            head = re.match(r"^([0-9a-f]+) <(\S+)>:$", line)
            if head:
                body, start = out.setdefault(head[2], []), int(head[1], 16)
                continue
            m = LINE.match(line)
            if body is not None and m:
                target = start + int(m[4] or "0", 16) if "branch" in m[1] else None
                body.append((int(m[3], 16), m[1], m[2], target))
    return out


def _pending_at_barriers(body):
    """For every s_barrier the sets of LDS operations ("w" or (address register, offset), oldest first)
    that may be in flight there. LDS operations return in their order; a scalar load in flight only makes
    a wait stricter, so lgkmcnt(n) leaves at most the newest n."""
    at = {ins[0]: i for i, ins in enumerate(body)}
    seen = [set() for _ in body]
    work, found = [(0, ())], {}
    while work:
        i, pend = work.pop()
        while i < len(body) and pend not in seen[i]:
            seen[i].add(pend)
            _, op, args, target = body[i]
            if op.startswith("ds_"):
                r = re.match(r"v\[\d+:\d+\], (v\d+)(?: offset:(\d+))?", args)
                pend += ((r[1], int(r[2] or 0)) if op == "ds_read_b128" else "w",)
                pend = pend[-64:]
            elif op == "s_waitcnt":
                n = re.search(r"lgkmcnt\((\d+)\)", args)
                if n:
                    pend = pend[len(pend) - min(len(pend), int(n[1])):]
            elif op == "s_barrier":
                found.setdefault(i, set()).add(pend)
            elif op == "s_endpgm":
                break
            elif op == "s_branch":
                i = at[target]
                continue
            elif op.startswith("s_cbranch"):
                work.append((at[target], pend))
            i += 1
    return found


def _pending(body):
    return [p for sets in _pending_at_barriers(body).values() for p in sets if p]


def test_scan_follows_waits_and_branches():
    """The scan itself, on a loop whose branch skips the only wait."""
    body = [(0, "ds_read_b128", "v[0:3], v9 offset:16", None), (4, "s_cbranch_scc1", "2", 12),
            (8, "s_waitcnt", "vmcnt(2) lgkmcnt(0)", None), (12, "s_barrier", "", None),
            (16, "s_cbranch_scc0", "0", 0), (20, "s_endpgm", "", None)]
    found = _pending_at_barriers(body)
    assert () in found[3] and (("v9", 16),) in found[3]
    body[1] = (4, "s_nop", "0", None)
    assert _pending_at_barriers(body) == {3: {()}}


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="llvm-objdump not available")
def test_no_read_of_a_retired_buffer_crosses_a_barrier(tmp_path):
    kernels = _kernels(str(tmp_path))
    fwd = {n: re.search(r"attn_fwd_kernelILi(\d+)ELi\d+ELb([01])ELb[01]E", n) for n in kernels}
    mixed = {n: re.search(r"mixed_layer_kernelILi(\d+)ELi", n) for n in kernels}
    checked = 0
    for name, body in kernels.items():
        m = fwd[name] or mixed[name]
        if not m:
            continue
        checked += 1
        d, ahead = int(m[1]), mixed[name] is not None or m[2] == "1"
        assert any(op == "ds_read_b128" for _, op, _, _ in body)
        for pend in _pending(body):
            # reading ahead: the K reads of the next tile, whose buffer is rewritten two barriers on. Each
            # of D / 16 address registers reads the tile's two halves, at offsets 32 D bytes * 2 apart;
            # V^T reads go through one register.
            assert ahead, f"{name}: {pend} in flight at a barrier"
            assert "w" not in pend, f"{name}: {pend}"
            regs = {r for r, _ in pend}
            offs = sorted({o for _, o in pend})
            assert len(pend) <= d // 8 and len(offs) <= 2 and len(regs) >= len(pend) / 2, f"{name}: {pend}"
            assert len(offs) < 2 or offs[1] - offs[0] == 64 * d, f"{name}: {pend}"
    assert checked == 40, checked   # 4 groups x (attn_fwd: 2 forms at d 128, 4 at d 64; mixed_layer: 2 at each)
