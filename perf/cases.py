"""What is measured of this library: calls of its public entry points as a program makes them.

Every case is one kind of call with its sizes.  The graph size p, the number of blocks n and the buffer sizes are those
of the library's own configurations and of its benchmark; `draw` gives others over the same ranges.  Roots, ranges of
ranks, processes, triples and payloads come from the seed.  All results are whole numbers and are compared exactly.
"""
import math

import numpy as np
import torch

import paper_2205_10072_amd as bcs

STEP = 1000003          # prime: neighbouring seeds give different residues for every p in use


def listed():
    return [
        # a launcher asking for the schedules of a small communicator: latency of one call, 1000 rows of 10 entries
        {"name": "sched_small", "kind": "sched", "p": 1000, "want": "both", "ws": False},
        # all ranks of p = 2^20 + 1 (every level odd: the most irregular graph), 2 x 88 MB
        {"name": "sched_2e20", "kind": "sched", "p": 2**20 + 1, "want": "both", "ws": True},
        # the largest configuration: all ranks of p = 2^27 - 1, 2 x 14.5 GB
        {"name": "sched_2e27", "kind": "sched", "p": 2**27 - 1, "want": "both", "ws": True},
        # one GPU's share of that graph when the ranks are spread over eight GPUs: no rows of other ranks at hand
        {"name": "shard_2e27", "kind": "shard", "p": 2**27 - 1, "rows": 2**24},
        # block tables from schedule rows at the paper's own run (1152 processes, 1658 blocks), without scratch memory
        {"name": "expand_paper", "kind": "expand", "p": 1152, "n": 1658, "ws": False},
        # long rows: p = 65537, n = 4096, 2 x 1.08 GB, with scratch memory
        {"name": "expand_long", "kind": "expand", "p": 65537, "n": 4096, "ws": True},
        # schedules and block tables in one call: many ranks, 256 blocks, 2 x 1.16 GB of block tables
        {"name": "sched_expand_2e20", "kind": "sched_expand", "p": 2**20 + 1, "n": 256},
        # the same call with few blocks (short messages), where the schedules are a large part of the work
        {"name": "sched_expand_short", "kind": "sched_expand", "p": 200003, "n": 64},
        # a service answering unrelated (p, rank, root) requests: a million triples of mixed size
        {"name": "batch_2e20", "kind": "batch", "count": 2**20, "want": "both"},
        # index tables of one process of an irregular allgather, 2^20 + 1 processes, 256 blocks per buffer
        {"name": "allgather_tables", "kind": "allgather", "p": 2**20 + 1, "n": 256},
        # one round of packing and unpacking at the paper's own run: 241 KB a message, latency
        {"name": "pack_paper", "kind": "pack", "p": 1152, "m": 10**8, "n": 1658, "planned": False},
        # the same with large buffers and the plans of all rounds made ahead: 268 MB a message, bandwidth
        {"name": "pack_large", "kind": "pack", "p": 1152, "m": 2**31, "n": 32, "planned": True},
    ]


def _log(rng, lo, hi):
    """A whole number of [lo, hi], uniform over its logarithm."""
    return min(hi, max(lo, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng):
    kind = rng.choice(["sched", "sched", "shard", "expand", "sched_expand", "sched_expand", "batch", "allgather", "pack"])
    if kind == "sched":
        return {"kind": kind, "p": _log(rng, 16, 2**27 - 1), "want": rng.choice(["both", "both", "both", "recv", "send"]),
                "ws": rng.random() < 0.7}
    if kind == "shard":
        p = _log(rng, 10**4, 2**31 - 1)
        return {"kind": kind, "p": p, "rows": _log(rng, 64, min(p // 2, 2**24))}
    if kind in ("expand", "sched_expand"):
        p = _log(rng, 64, 2**22)
        most = max(2, min(8192, 2**28 // p - 32))       # at most about 2 x 1 GB of block tables
        c = {"kind": kind, "p": p, "n": _log(rng, 1, most)}
        if kind == "expand":
            c["ws"] = rng.random() < 0.5
        return c
    if kind == "batch":
        return {"kind": kind, "count": _log(rng, 64, 2**20), "want": rng.choice(["both", "both", "recv", "send"])}
    if kind == "allgather":
        p = _log(rng, 64, 2**20 + 1)
        return {"kind": kind, "p": p, "n": _log(rng, 1, max(2, min(8192, 2**28 // p - 32)))}
    p = _log(rng, 32, 5000)
    return {"kind": kind, "p": p, "m": _log(rng, 50 * p, 2**30), "n": _log(rng, 32, 2000), "planned": rng.random() < 0.5}


def _empty(*shape):
    return torch.empty(shape, dtype=torch.int32, device="cuda")


def _scratch(nbytes):
    return torch.empty(max(int(nbytes), 1), dtype=torch.uint8, device="cuda")


def _triples(count, rng):
    """p log-uniform in [2, 2^31 - 1] (bit length uniform in 2..31), rank and root uniform in [0, p)."""
    bits = rng.integers(2, 32, count)
    lo = np.left_shift(np.int64(1), bits - 1)
    p = lo + (rng.random(count) * lo).astype(np.int64)
    r = (rng.random(count) * p).astype(np.int64)
    root = (rng.random(count) * p).astype(np.int64)
    return [torch.from_numpy(a.astype(np.int32)).cuda() for a in (p, r, root)]


def _sizes(p, m):
    """Buffer sizes of the paper's irregular allgather: (r mod 3) * floor(m / p), the last process takes the rest."""
    sizes = (np.arange(p, dtype=np.int64) % 3) * (m // p)
    sizes[p - 1] = m - int(sizes[:p - 1].sum())
    displs = np.zeros(p + 1, dtype=np.int64)
    np.cumsum(sizes, out=displs[1:])
    return sizes, displs


def prepare(case, seed):
    s = dict(case)
    kind = s["kind"]
    if kind in ("sched", "shard"):
        p = s["p"]
        q = bcs.bcs_q(p)
        if kind == "sched":
            s["root"], s["r0"], s["r1"] = seed * STEP % p, 0, p
            want = s["want"]
        else:
            s["root"], s["r0"] = 0, seed * STEP % (p - s["rows"] + 1)
            s["r1"] = s["r0"] + s["rows"]
            want, s["ws"] = "both", True
        rows = s["r1"] - s["r0"]
        s["recv"] = _empty(rows, q) if want != "send" else None
        s["send"] = _empty(rows, q) if want != "recv" else None
        if s["ws"]:
            s["scratch"] = _scratch(bcs.bcs_sched_workspace_bytes(p, s["r0"], s["r1"], s["send"] is not None))
    elif kind in ("expand", "sched_expand"):
        p, n = s["p"], s["n"]
        q, R = bcs.bcs_q(p), bcs.bcs_rounds(p, n)
        s["root"] = seed * STEP % p
        s["recv"], s["send"] = _empty(p, q), _empty(p, q)
        s["recv_blocks"], s["send_blocks"] = _empty(p, R), _empty(p, R)
        if kind == "expand":
            bcs.bcs_sched_rooted(p, s["root"], 0, p, s["recv"], s["send"])
            if s["ws"]:
                s["scratch"] = _scratch(bcs.bcs_expand_workspace_bytes(p, n, 0, p))
        else:
            s["scratch"] = _scratch(bcs.bcs_sched_expand_workspace_bytes(p, n))
    elif kind == "batch":
        count, want = s["count"], s["want"]
        s["triples"] = _triples(count, np.random.default_rng(seed))
        s["recv"] = _empty(count, bcs.BATCH_STRIDE) if want != "send" else None
        s["send"] = _empty(count, bcs.BATCH_STRIDE) if want != "recv" else None
        s["q"] = _empty(count)
    elif kind == "allgather":
        p, n = s["p"], s["n"]
        R = bcs.bcs_rounds(p, n)
        s["r"] = seed * STEP % p
        s["pack"], s["unpack"] = _empty(R, p), _empty(R, p)
        s["scratch"] = _scratch(bcs.bcs_allgather_workspace_bytes(p))
    else:
        p, m, n = s["p"], s["m"], s["n"]
        sizes, displs = _sizes(p, m)
        R = bcs.bcs_rounds(p, n)
        r = seed * STEP % p
        pack, unpack = _empty(R, p), _empty(R, p)
        bcs.bcs_allgather_tables(p, n, r, pack, unpack)
        j = R // 2                                       # a steady-state round: (nearly) every root moves a block
        gen = torch.Generator(device="cuda").manual_seed(seed)
        s["displs"] = torch.from_numpy(displs).cuda()
        s["data"] = torch.randint(0, 1 << 30, (m,), dtype=torch.int32, device="cuda", generator=gen)
        most = int((-(-sizes // n)).sum())               # no round's message is longer
        s["message"] = torch.randint(0, 1 << 30, (most,), dtype=torch.int32, device="cuda", generator=gen)
        s["packed"] = torch.zeros(most, dtype=torch.int32, device="cuda")
        offsets = torch.empty((2, p + 1), dtype=torch.int64, device="cuda")
        src = torch.empty((2, p), dtype=torch.int64, device="cuda")
        s["idx"] = torch.stack((pack[j], unpack[j]))
        bcs.bcs_pack_plan_rounds(n, s["idx"], s["displs"], offsets, src)
        s["length"] = [int(v) for v in offsets[:, p].cpu()]
        s["offsets"] = [offsets[0], offsets[1]]
        s["src"] = [src[0], src[1]]
        s["idx"] = [s["idx"][0].clone(), s["idx"][1].clone()]
        s["received"] = s["message"][:s["length"][1]]
        s["scratch"] = _scratch(bcs.bcs_pack_workspace_bytes(p))
    return s


def run(s):
    kind = s["kind"]
    if kind in ("sched", "shard"):
        if s["ws"]:
            bcs.bcs_sched_rooted_ws(s["p"], s["root"], s["r0"], s["r1"], s["recv"], s["send"], s["scratch"])
        else:
            bcs.bcs_sched_rooted(s["p"], s["root"], s["r0"], s["r1"], s["recv"], s["send"])
        return s["recv"], s["send"]
    if kind == "expand":
        args = (s["p"], s["n"], 0, s["p"], s["recv"], s["send"], s["recv_blocks"], s["send_blocks"])
        if s["ws"]:
            bcs.bcs_expand_ws(*args, s["scratch"])
        else:
            bcs.bcs_expand(*args)
        return s["recv_blocks"], s["send_blocks"]
    if kind == "sched_expand":
        bcs.bcs_sched_expand_ws(s["p"], s["root"], s["n"], s["recv"], s["send"], s["recv_blocks"], s["send_blocks"],
                                s["scratch"])
        return s["recv"], s["send"], s["recv_blocks"], s["send_blocks"]
    if kind == "batch":
        bcs.bcs_sched_batch(*s["triples"], s["recv"], s["send"], s["q"])
        return s["recv"], s["send"], s["q"]
    if kind == "allgather":
        bcs.bcs_allgather_tables_ws(s["p"], s["n"], s["r"], s["pack"], s["unpack"], s["scratch"])
        return s["pack"], s["unpack"]
    # a round of the allgather: pack the message for one neighbour, unpack the one that came from the other
    if s["planned"]:
        bcs.bcs_pack_round_planned(s["offsets"][0], s["src"][0], s["data"], s["packed"])
        bcs.bcs_unpack_round_planned(s["offsets"][1], s["src"][1], s["data"], s["received"], s["length"][1])
    else:
        bcs.bcs_pack_round(s["n"], s["idx"][0], s["displs"], s["data"], s["packed"], s["offsets"][0], s["scratch"])
        bcs.bcs_unpack_round(s["n"], s["idx"][1], s["displs"], s["data"], s["received"], s["length"][1], s["offsets"][1],
                             s["scratch"])
    return s["packed"], s["data"], s["offsets"][0], s["offsets"][1]


def work(case):
    """Every output written once, every input read once; the schedules are whole-number work without a contraction."""
    kind = case["kind"]
    if kind == "sched":
        total = 4 * case["p"] * bcs.bcs_q(case["p"]) * (2 if case["want"] == "both" else 1)
    elif kind == "shard":
        total = 2 * 4 * case["rows"] * bcs.bcs_q(case["p"])
    elif kind in ("expand", "sched_expand"):
        total = 2 * 4 * case["p"] * (bcs.bcs_q(case["p"]) + bcs.bcs_rounds(case["p"], case["n"]))
    elif kind == "batch":
        tables = 2 if case["want"] == "both" else 1
        total = case["count"] * (3 * 4 + 4 + tables * 4 * bcs.BATCH_STRIDE)
    elif kind == "allgather":
        total = 2 * 4 * case["p"] * bcs.bcs_rounds(case["p"], case["n"])
    else:
        sizes, _ = _sizes(case["p"], case["m"])
        plan = (2 * 8 if case["planned"] else 4 + 2 * 8) * case["p"]
        total = 2 * (2 * 4 * int((sizes // case["n"]).sum()) + plan)
    return {"bytes": total, "flops": 0}


def tolerance(case):
    return "exact"
