"""CPU tests of the closed-form rows (csrc/bcs_rows.h), made as the kernels make them, against the oracle and against their
definition by windows (csrc/bcs_core.h): every rank of small p, and the ends of blocks of large p (where the exceptions of
the closed form lie)."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import oracle

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2205_10072_amd", "csrc")


@pytest.fixture(scope="module")
def rows(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("rows") / "librows.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wno-unknown-pragmas", "-I", CSRC, "-o", lib,
                    os.path.join(HERE, "bcs_rowscheck.cpp")], check=True)
    L = ctypes.CDLL(lib)
    i32p = ctypes.POINTER(ctypes.c_int32)
    L.rc_rows.argtypes = [ctypes.c_int32, i32p, ctypes.c_int64, ctypes.c_int, i32p, i32p]
    L.rc_windows.argtypes = [ctypes.c_int32, i32p, ctypes.c_int64, i32p, i32p]

    def call(p, ranks, wave_q):
        v = np.ascontiguousarray(ranks, dtype=np.int32)
        out = np.full((2, len(v), 32), 12345, dtype=np.int32)
        ptr = [a.ctypes.data_as(i32p) for a in (v, out[0], out[1])]
        if wave_q == "windows":
            assert L.rc_windows(p, ptr[0], len(v), ptr[1], ptr[2]) == 0
        else:
            assert L.rc_rows(p, ptr[0], len(v), wave_q, ptr[1], ptr[2]) == 0
        q = (p - 1).bit_length()
        assert (out[:, :, q:] == 12345).all()
        return out[0, :, :q], out[1, :, :q]
    return call


def test_rows_every_rank_of_small_p(rows):
    for p in list(range(2, 700)) + [1000, 1023, 1024, 1025, 2047, 2049, 2731, 4095, 4097, 5461, 6001]:
        recv, send = oracle.sched_range(p, 0, 0, p)
        q = (p - 1).bit_length()
        for wave_q in (0, min(31, q + 3)):
            got_r, got_s = rows(p, np.arange(p), wave_q)
            assert np.array_equal(got_r, recv), (p, wave_q)
            assert np.array_equal(got_s, send), (p, wave_q)


@pytest.mark.parametrize("q", [13, 17, 20, 21, 24, 27, 28, 30, 31])
def test_rows_at_the_ends_of_blocks(rows, q):
    """Runs of ranks around sums of large skips, around those minus one skip, and around both ends of the ring, for p
    with few, all, and random odd levels (17 and more of them at and above level 7 bring the rarest exception)."""
    rng = np.random.default_rng(q)
    lo, hi = (1 << (q - 1)) + 1, min(1 << q, 2**31 - 1)
    ps = [lo, lo + 4, hi, hi - 1, hi - 3, lo + (1 << (q - 3)), lo + (1 << (q // 2))] + [int(x) for x in rng.integers(lo, hi, 4)]
    ps += [lo - 1 + int(x) for x in rng.integers(1, 130, 3)]
    for p in ps:
        skips = oracle.skips(p)
        bases = [0, p - 70]
        for _ in range(14):
            y, s, cut = int(rng.integers(0, p)), 0, int(rng.integers(0, q))
            for k in range(q - 1, cut - 1, -1):
                if y >= skips[k]:
                    y -= skips[k]
                    s += skips[k]
            bases += [s - 36, s - skips[int(rng.integers(0, q))] - 36]
        for base in bases:
            r0 = base % p
            r0 = min(r0, p - 72)
            recv, send = oracle.sched_range(p, 0, r0, r0 + 72)
            for wave_q in (0, 31):
                got_r, got_s = rows(p, np.arange(r0, r0 + 72), wave_q)
                assert np.array_equal(got_r, recv), (p, r0, wave_q)
                assert np.array_equal(got_s, send), (p, r0, wave_q)


def _p_of(rng, q):
    """p of q bits: random, or with few, many or all levels odd above the lowest six bits."""
    kind = int(rng.integers(0, 4))
    if kind == 0:
        return int(rng.integers((1 << (q - 1)) + 1, min(1 << q, 2**31 - 1) + 1))
    odd = [0.05, 0.95, 1.0][kind - 1]
    bits = "".join("0" if rng.random() < odd else "1" for _ in range(q - 7))
    return min(2**31 - 1, (1 << (q - 1) | int(bits + format(int(rng.integers(0, 64)), "06b"), 2)) + 1)


@pytest.mark.parametrize("q", range(2, 32))
def test_rows_against_windows(rows, q):
    """The two constructions share the table of the low levels and nothing else.  Ranks at random, at the ends of the ring and
    within 150 of sums of skips, on both sides."""
    rng = np.random.default_rng(100 + q)
    for _ in range(25):
        p = _p_of(rng, q) if q > 7 else int(rng.integers((1 << (q - 1)) + 1, (1 << q) + 1))
        skips = [((p - 1) >> (q - k)) + 1 for k in range(q + 1)]
        centres = [0, p] + [sum(s for s in skips[:q] if rng.random() < 0.4) for _ in range(10)]
        ranks = [int(x) for x in rng.integers(0, p, 40)]
        for c in centres:
            ranks += [int((c + d) % p) for d in rng.integers(-150, 151, 30)]
        want = rows(p, ranks, "windows")
        for wave_q in (0, q, 31):
            got = rows(p, ranks, wave_q)
            assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1]), (p, wave_q)
