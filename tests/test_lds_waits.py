"""Waits of the kernels whose loads write LDS directly, checked in the built library's own code.

These kernels request a tile's left factors ahead with loads that write LDS, and before the barrier
that ends a (half) tile wait until no more vector-memory operations are outstanding than they issued
after the requests that must have landed.  The compiler may move the other loads that the count
assumes (it once moved the last one of a tile behind the wait), so the count is checked where it is
certain: over every path of the disassembled kernels.

Per program point: for the requests issued since the last barrier and for the older ones, the fewest
operations issued after the latest of them on any path (None: all have completed).  A wait for n
completes those with at least n operations behind them.  At a barrier the older requests must have
completed, and in k_far_wide64, whose two buffers are requested one half ahead, every request.
"""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1812_10722_amd", "liblspr.so")
OBJDUMP = shutil.which("llvm-objdump", path="/opt/rocm/llvm/bin:" + os.environ.get("PATH", ""))
KERNELS = re.compile(r"k_far_(half|narrow64|wide64|wide)I")

pytestmark = pytest.mark.skipif(not os.path.exists(LIB) or OBJDUMP is None,
                                reason="liblspr.so or llvm-objdump not there")


def kernels(listing):
    """name -> [(address, mnemonic, operands)] of the kernels in a disassembly."""
    out, cur = {}, None
    for line in listing.splitlines():
        m = re.match(r"[0-9a-f]+ <(\S+)>:$", line)
        if m:
            cur = out.setdefault(m.group(1), []) if KERNELS.search(m.group(1)) else None
            continue
        m = re.match(r"\s+(\S+)\s*(.*?)\s*//\s*([0-9A-Fa-f]+):(.*)", line)
        if cur is not None and m:
            target = re.search(r"<\S+?\+0x([0-9a-f]+)>", m.group(4))
            cur.append((int(m.group(3), 16), m.group(1), m.group(2),
                        int(target.group(1), 16) if target else None))
    return out


def late_requests(code, one_ahead):
    """Addresses of the barriers that some path reaches with a request outstanding that must have
    completed, and the numbers of requests and barriers seen."""
    base = code[0][0]
    index = {a - base: k for k, (a, *_) in enumerate(code)}
    least = lambda a, b: b if a is None else (a if b is None else min(a, b))
    state = [None] * len(code)  # (of this barrier's requests, of older ones) before instruction k
    state[0] = (None, None)
    todo, late, n_req, n_bar = [0], set(), set(), set()
    while todo:
        k = todo.pop()
        new, old = state[k]
        a, op, args, target = code[k]
        if op.startswith(("buffer_", "global_", "flat_", "scratch_")) and not op.startswith("buffer_wbl2") \
                and not op.startswith("buffer_inv"):
            new, old = (x if x is None else min(x + 1, 64) for x in (new, old))
            if re.search(r"\blds\b", args):
                new = 0
                n_req.add(a)
        elif op == "s_waitcnt":
            m = re.search(r"vmcnt\((\d+)\)", args)
            if m or re.fullmatch(r"0x[0-9a-f]+|\d+", args):
                raw = None if m else int(args, 0)
                n = int(m.group(1)) if m else (raw & 15) | (raw >> 14 & 3) << 4
                new, old = (x if x is None or x < n else None for x in (new, old))
        elif op == "s_barrier":
            n_bar.add(a)
            if old is not None or (one_ahead and new is not None):
                late.add(a)
            new, old = None, least(new, old)
        if op == "s_endpgm":
            continue
        after = []
        if op != "s_branch":
            after.append(k + 1)
        if op.startswith(("s_branch", "s_cbranch")):
            after.append(index[target if target is not None else 0])
        assert not op.startswith(("s_setpc", "s_swappc", "s_call")), op
        for q in after:
            was = state[q]
            now = (new, old) if was is None else (least(was[0], new), least(was[1], old))
            if now != was:
                state[q] = now
                todo.append(q)
    return late, len(n_req), len(n_bar)


def check(lib, tmp):
    shutil.copy(lib, os.path.join(tmp, "lib.so"))
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp, check=True, capture_output=True)
    found = {}
    for f in sorted(os.listdir(tmp)):
        if "gfx950" in f and KERNELS.search(open(os.path.join(tmp, f), "rb").read().decode("latin1")):
            text = subprocess.run([OBJDUMP, "-d", f], cwd=tmp, check=True, capture_output=True, text=True)
            for name, code in kernels(text.stdout).items():
                found[name] = late_requests(code, "k_far_wide64" in name)
    return found


def test_requests_into_lds_have_landed_at_every_barrier(tmp_path):
    found = check(LIB, str(tmp_path))
    for kind in ("half", "narrow64", "wide64", "wide"):
        assert any(f"k_far_{kind}I" in name for name in found), kind
    for name, (late, requests, barriers) in found.items():
        assert requests > 0 and barriers > 1, name
        assert not late, (name, [hex(a) for a in late])
