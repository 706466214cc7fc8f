"""The order of memory instructions that the persistent INT8 GEMM counts on, read from the assembly of its source:
the relaxed wait for a tile's operands lets the previous tile's stores stay outstanding, which is right only if exactly
so many stores follow the loads of the next tile's head and none of them can move ahead of a load."""
import os
import re
import subprocess

from paper_2508_03984_amd import build

STORE = re.compile(r"\s(global|flat|buffer)_store_")
LOAD = re.compile(r"\s(global|flat|buffer)_load_")
FENCE = "sched_barrier mask(0x00000000)"


def _functions(asm):
    out, cur = {}, None
    for line in asm.splitlines():
        m = re.match(r"(_ZN\S+):", line)
        if m:
            cur = out.setdefault(m.group(1), [])
        elif line.startswith(".Lfunc_end"):
            cur = None
        elif cur is not None:
            cur.append(line)
    return out


def test_stores_of_a_tile_follow_the_loads_of_the_next_head(tmp_path):
    asm = tmp_path / "gemm.s"
    flags = [f for f in build.FLAGS if f not in ("-fPIC", "-shared")]
    subprocess.check_call([build.HIPCC] + flags + ["-x", "hip", "--cuda-device-only", "-S",
                                                   os.path.join(build.CSRC, "oz2_int8_gemm.hip"), "-o", str(asm)])
    checked = 0
    for name, body in _functions(asm.read_text()).items():
        m = re.search(r"k_int8_gemm_persistentILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi2EE", name)   # kOutU8
        if not m:
            continue
        wm, wn, tm, tn, bk, stages = (int(g) for g in m.groups())
        loads_per_tile = (32 * tm * wm + 32 * tn * wn) * (bk // 16) // (64 * wm * wn)
        youngest, stores = (stages - 3) * loads_per_tile, tm * tn
        at = [i for i, line in enumerate(body) if STORE.search(line)]
        assert len(at) == stores, name                                # what the relaxed wait counts
        waits = {int(w) for line in body for w in re.findall(r"vmcnt\((\d+)\)", line)}
        assert waits == {0, youngest, youngest + stores}, (name, waits)
        # one basic block, no load among the stores, and a fence on either side with nothing in between
        inside = body[at[0]:at[-1] + 1]
        assert not any(LOAD.search(line) or line.startswith(".LBB") for line in inside), name
        before = next(i for i in range(at[0], -1, -1) if FENCE in body[i] or LOAD.search(body[i]) or STORE.search(body[i]) and i != at[0])
        assert FENCE in body[before], (name, body[before])
        after = next(i for i in range(at[-1] + 1, len(body))
                     if FENCE in body[i] or LOAD.search(body[i]) or body[i].startswith(".LBB"))
        assert FENCE in body[after], (name, body[after])
        checked += 1
    assert checked == 1
