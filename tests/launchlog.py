"""Runs calls of libbcsched on the stand-in runtime of hip_stub.cpp (no GPU, nothing dereferenced) and returns what
they enqueued.  The calls run in a process of their own, which loads the stand-in before the library.

    log = run(tmp_path, '''
    rc = L.bcs_expand(5, 40, 0, 5, T(1), T(2), T(3), T(4), None)
    show(rc)
    ''')

In the script: L is the library, T(i) a made-up device address (16 TiB apart), show(value) records a value; the result
is a list of ("show", value), ("launch", {...}), ("malloc", ...) and so on, in the order of the calls."""
import json
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(ROOT, "paper_2205_10072_amd", "libbcsched.so")

HEAD = r'''
import ctypes, json, sys, threading, time
S = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
L = ctypes.CDLL(sys.argv[2])
i32, i64, sz, P = ctypes.c_int32, ctypes.c_int64, ctypes.c_size_t, ctypes.c_void_p
class Entry(ctypes.Structure):
    _fields_ = [("kind", i32), ("stream", ctypes.c_uint64), ("pointer", ctypes.c_uint64), ("bytes", ctypes.c_uint64),
                ("grid", ctypes.c_uint32 * 3), ("block", ctypes.c_uint32 * 3), ("name", ctypes.c_char * 64),
                ("arg", ctypes.c_uint64 * 12)]
S.stub_count.restype = i64
S.stub_get.argtypes = [i64, ctypes.POINTER(Entry)]
S.stub_slow.argtypes = [ctypes.c_uint64, ctypes.c_int]
for name, sizes in (("k_expand_rows", "88888"), ("k_rows_to_bytes", "444488"), ("k_partner_tables", "4444888"),
                    ("k_batch", "8888888"), ("k_pack_plan_one", "44888"), ("k_allgather_tables_flat", "888888"),
                    ("k_sched", "84444488")):
    S.stub_signature(name.encode(), sizes.encode())
S.stub_signature(b"k_expand", b"8E")                     # E: a struct of four addresses
L.bcs_sched_rooted_ws.argtypes = [i32] * 4 + [P] * 3 + [sz, P]
L.bcs_sched_expand_ws.argtypes = [i32] * 3 + [P] * 5 + [sz, P]
L.bcs_sched_expand.argtypes = [i32] * 3 + [P] * 5
L.bcs_expand.argtypes = [i32] * 4 + [P] * 5
L.bcs_expand_ws.argtypes = [i32] * 4 + [P] * 5 + [sz, P]
L.bcs_sched_batch.argtypes = [i64] + [P] * 7
L.bcs_allgather_tables.argtypes = [i32] * 3 + [P] * 3
L.bcs_allgather_tables_ws.argtypes = [i32] * 3 + [P] * 3 + [sz, P]
L.bcs_allgather_partners.argtypes = L.bcs_census_partners.argtypes = [i32] * 3 + [P] * 3
L.bcs_pack_plan_rounds.argtypes = [i32, i32, i64] + [P] * 5
L.bcs_pack_round_planned.argtypes = [i32] + [P] * 4 + [i64, P]
L.bcs_pack_round.argtypes = [i32, i32] + [P] * 4 + [i64] + [P] * 2 + [sz, P]
L.bcs_valu_peak_launch.argtypes = [ctypes.c_uint32, ctypes.c_uint32, P, P]
for f in ("sched_workspace_bytes", "sched_expand_workspace_bytes", "expand_workspace_bytes", "allgather_workspace_bytes",
          "pack_workspace_bytes"):
    getattr(L, "bcs_" + f).restype = i64
def T(i): return i << 44
shown, KINDS = [], ("launch", "malloc", "free", "sync", "record", "wait")
def show(value): shown.append((S.stub_count(), value))
'''

TAIL = r'''
out, at = [], 0
for i in range(S.stub_count() + 1):
    while at < len(shown) and shown[at][0] <= i:
        out.append(("show", shown[at][1]))
        at += 1
    if i < S.stub_count():
        e = Entry()
        S.stub_get(i, e)
        out.append((KINDS[e.kind], {"name": e.name.decode(), "stream": e.stream, "pointer": e.pointer, "bytes": e.bytes,
                                    "grid": list(e.grid), "lanes": e.grid[0] * e.block[0], "arg": list(e.arg)}))
print("LOG " + json.dumps(out))
'''


def build_stub(tmp_path):
    stub = str(tmp_path / "libhipstub.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-Wall", "-o", stub,
                    os.path.join(HERE, "hip_stub.cpp")], check=True)
    return stub


def run(tmp_path, script):
    if not os.path.exists(LIB):
        import paper_2205_10072_amd.build as b
        b.build()
    res = subprocess.run([sys.executable, "-c", HEAD + script + TAIL, build_stub(tmp_path), LIB], capture_output=True,
                         text=True, timeout=120)
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-4000:]
    line = [x for x in res.stdout.splitlines() if x.startswith("LOG ")][-1]
    return [tuple(x) for x in json.loads(line[4:])]


def launches(log, name=None):
    return [e for kind, e in log if kind == "launch" and (name is None or e["name"] == name)]


def shown(log):
    return [v for kind, v in log if kind == "show"]
