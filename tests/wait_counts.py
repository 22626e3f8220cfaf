"""Reads the waits of the big-tile GEMM kernels out of the library built here.

The kernels publish a token stage with ``s_waitcnt vmcnt(N)`` and a barrier: the newest N vector-memory
operations may still be in flight.  N counts the token moves of two stages and the weight loads issued
beside them, so it is right only while the built code holds every load that the source counts: a load
whose result nothing reads is removed by the compiler, and the wait then lets the guarded moves
themselves stay in flight.
"""
import heapq
import os
import re
import shutil
import subprocess

LLVM = "/opt/rocm/llvm/bin"
IN_FLIGHT_STAGES = 2  # token stages that may be in flight at a wait; the one before them is published

_VMEM = re.compile(r"^(buffer|global|flat|scratch)_(load|store|atomic)")
_BRANCH = re.compile(r"^s_(c?branch\S*)\s+(-?\d+)")
_VMCNT = re.compile(r"vmcnt\((\d+)\)")


def disassemble(lib, tmp, name):
    """{symbol: [(address, text)]} of the gfx950 kernels of `lib` whose symbol holds `name`."""
    copy = shutil.copy(lib, os.path.join(tmp, "lib.so"))
    subprocess.run([f"{LLVM}/llvm-objdump", "--offloading", copy], check=True, capture_output=True)
    out = {}
    for f in sorted(os.listdir(tmp)):
        if not f.endswith("gfx950"):
            continue
        text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", os.path.join(tmp, f)], check=True,
                              capture_output=True, text=True).stdout
        cur = None
        for line in text.splitlines():
            m = re.match(r"^[0-9a-f]+ <(\S+)>:", line)
            if m:
                cur = out.setdefault(m.group(1), []) if name in m.group(1) else None
            elif cur is not None and "//" in line:
                ins, addr = line.split("//", 1)
                cur.append((int(addr.split(":")[0], 16), ins.strip()))
    return out


def is_move(ins):
    """A move into LDS (buffer_load ... lds)."""
    return ins.startswith("buffer_load") and ins.endswith(" lds")


def _predecessors(code):
    at = {addr: i for i, (addr, _) in enumerate(code)}
    pred = [[] for _ in code]
    for i, (addr, ins) in enumerate(code):
        assert not ins.startswith(("s_swappc", "s_call")), ins
        m = _BRANCH.match(ins)
        if m:
            off = int(m.group(2))
            pred[at[addr + 4 + 4 * (off - 65536 if off >= 32768 else off)]].append(i)
        elif ins.startswith("s_setpc"):
            # A jump out of a branch's range: s_getpc_b64, s_add_u32 with the offset, s_addc_u32, s_setpc_b64.
            assert code[i - 3][1].startswith("s_getpc") and code[i - 2][1].startswith("s_add_u32"), (hex(addr), ins)
            off = int(code[i - 2][1].split(",")[-1], 0)
            pred[at[code[i - 2][0] + (off - (1 << 32) if off >= 1 << 31 else off)]].append(i)
        if not (m and m.group(1) == "branch") and not ins.startswith(("s_endpgm", "s_setpc")) and i + 1 < len(code):
            pred[i + 1].append(i)
    return pred


def _walk(code, pred, start, step, done):
    """The backward paths from `start`, as (least cost, state) where a path ends: where done() holds of its
    state, or step(ins, state) is None; else step gives (cost, state) of passing an instruction."""
    heap, seen, found = [(0, start, 0)], set(), []
    while heap:
        cost, i, state = heapq.heappop(heap)
        if (i, state) in seen:
            continue
        seen.add((i, state))
        for p in pred[i]:
            r = step(code[p][1], state)
            if r is None:
                found.append((cost, state))
            elif done(r[1]):
                found.append((cost + r[0], r[1]))
            else:
                heapq.heappush(heap, (cost + r[0], p, r[1]))
    return found


def counted_waits(code):
    """[(address, N, least)] of each counted wait ahead of a barrier: the count N it leaves in flight, and
    the fewest vector-memory operations that any path issues behind the last of the moves it guards."""
    pred = _predecessors(code)
    out = []
    for b, (addr, ins) in enumerate(code):
        if not ins.startswith("s_barrier"):
            continue
        # The barrier's own wait is the nearest one with a vmcnt, with no vector-memory operation between.
        w = b - 1
        while w >= 0 and not _VMCNT.search(code[w][1]) and not _VMEM.match(code[w][1]) \
                and not code[w][1].startswith(("s_barrier", "s_cbranch", "s_branch")):
            w -= 1
        m = _VMCNT.search(code[w][1])
        if not m or int(m.group(1)) == 0:
            continue
        # Moves since the barrier before: one stage in the K loop, three ahead of it.
        moves = {s for _, s in _walk(code, pred, w, lambda i, s: None if i.startswith("s_barrier") else
                                     (0, s + is_move(i)), lambda s: s > 24)}
        assert len(moves) == 1, (hex(addr), moves)
        stage = moves.pop()
        stage = {6: 2, 12: 4, 24: 8}.get(stage, stage)
        assert stage in (2, 4, 8), (hex(addr), stage)
        # Operations behind the first move that is not one of the newest stages'.
        ahead = IN_FLIGHT_STAGES * stage
        paths = _walk(code, pred, w, lambda i, s: (int(bool(_VMEM.match(i)) and not (s == ahead and is_move(i))),
                                                   s + is_move(i)), lambda s: s > ahead)
        out.append((addr, int(m.group(1)), min(c for c, _ in paths)))
    return out
