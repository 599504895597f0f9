"""Sweeps of the closed-form rows against their definition by windows (bcs_windows.hip), 3.0e11 ranks in all; three
minutes, run with BCS_RUN_SLOW=1.  Smaller counts of the same run always (test_gpu_parity.py, test_rows.py)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu, pytest.mark.slow]


@pytest.fixture(scope="module")
def bcs():
    import paper_2205_10072_amd as m
    m.lib()
    return m


def _odd_pattern(rng, q):
    """p of q bits whose levels above the lowest six bits are odd seldom, mostly, all, or at random."""
    odd = [0.05, 0.5, 0.95, 1.0][int(rng.integers(0, 4))]
    bits = "".join("0" if rng.random() < odd else "1" for _ in range(q - 7))
    return min(2**31 - 1, (1 << (q - 1) | int(bits + format(int(rng.integers(0, 64)), "06b"), 2)) + 1)


def _all_ranks(bcs, ps, seed):
    """Receive rows against windows, send rows against the look-up in them, every rank of every p, random roots."""
    import windows
    rng = np.random.default_rng(seed)
    flat = [torch.empty(max(ps) * bcs.bcs_q(max(ps)), dtype=torch.int32, device="cuda") for _ in range(2)]
    ranks = 0
    for i, p in enumerate(ps):
        q, root = bcs.bcs_q(p), int(rng.integers(0, p))
        recv, send = (t[:p * q] for t in flat)
        bcs.bcs_sched_rooted(p, root, 0, p, recv, send)
        windows.check(p, root, 0, p, recv, send)
        ranks += p
        if i % 500 == 499 or i + 1 == len(ps):
            assert windows.differences() == 0, "one of %r" % (ps[i - i % 500:i + 1],)
        if i % 10000 == 9999 or i + 1 == len(ps):
            print("p = %d, %d of %d, %.3e ranks" % (p, i + 1, len(ps), ranks), flush=True)


def test_every_rank_of_every_p_to_200000(bcs):
    _all_ranks(bcs, list(range(2, 200001)), 1)


@pytest.mark.parametrize("part", range(4))
def test_every_rank_of_larger_p_to_2_to_23(bcs, part):
    rng = np.random.default_rng(20 + part)
    ps = []
    while len(ps) < 35000:
        q = int(rng.integers(18, 24))
        ps.append(_odd_pattern(rng, q) if rng.random() < 0.6 else int(rng.integers(2**(q - 1) + 1, 2**q + 1)))
    _all_ranks(bcs, ps, part)


@pytest.mark.parametrize("part", range(4))
def test_slices_of_large_p(bcs, part):
    """Slices of 2^16 ranks of p of 23 to 31 bits at random, around sums of skips, those less one skip, and the ends of the
    ring; send rows by Alg. 5."""
    import windows
    rng = np.random.default_rng(40 + part)
    W = 1 << 16
    flat = [torch.empty(W * 31, dtype=torch.int32, device="cuda") for _ in range(2)]
    for i in range(10000):
        q = int(rng.integers(23, 32))
        p = _odd_pattern(rng, q) if rng.random() < 0.6 else int(rng.integers(2**(q - 1) + 1, min(2**q, 2**31 - 1) + 1))
        skips = bcs.bcs_skips(p)
        c = [int(rng.integers(0, p)), 0, p, sum(s for s in skips[:q] if rng.random() < 0.4)][int(rng.choice(4, p=[.2, .05, .05, .7]))]
        if rng.random() < 0.3:
            c -= skips[int(rng.integers(0, q))]
        root = int(rng.integers(0, p))
        r0 = min(max(0, (c + root) % p - W // 2), p - W)
        recv, send = (t[:W * q] for t in flat)
        bcs.bcs_sched_rooted(p, root, r0, r0 + W, recv, send)
        windows.check(p, root, r0, r0 + W, recv, send)
        if i % 500 == 499:
            assert windows.differences() == 0, (part, i)
        if i % 2500 == 2499:
            print("%d slices" % (i + 1), flush=True)
