"""GPU tests of tables that one launch of a kernel cannot cover (2^32 lanes), against the index arithmetic of Alg. 6 and the
oracle.  What is launched for such sizes is checked in full on the CPU (test_launches.py)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bcs():
    import paper_2205_10072_amd as m
    m.lib()
    return m


def _check(p, n, sched, blocks, oracle, seed):
    """`blocks` against the index arithmetic of Alg. 6 on `sched` with tensor operations, a range of rows at a time, and
    sampled rows against the oracle."""
    q, R = sched.shape[1], blocks.shape[1]
    x = (q - R % q) % q
    j = torch.arange(R, device="cuda")
    k = (x + j) % q
    shift = (j - k).to(torch.int32)
    step = max(1, (1 << 28) // R)
    for r0 in range(0, p, step):
        want = (sched[r0:r0 + step][:, k] + shift).clamp_(min=-1, max=n - 1)
        assert torch.equal(blocks[r0:r0 + step], want), r0
        del want
    rng = np.random.default_rng(seed)
    for r in [0, 1, p - 1] + [int(v) for v in rng.integers(0, p, 20)]:
        assert np.array_equal(blocks[r].cpu().numpy()[None], oracle.expand(p, n, sched[r:r + 1].cpu().numpy())), r


def test_block_tables_of_more_than_2_to_34_entries(bcs, oracle):
    """2 x 69 GB in one call with the schedules' workspace, then one of them again through bcs_expand_ws."""
    p, n, root = (1 << 20) + 1, 16500, 12345
    q, R = bcs.bcs_q(p), bcs.bcs_rounds(p, n)
    assert p * R > 1 << 34
    print("one call, 2 x %.1f GB" % (4e-9 * p * R), flush=True)
    recv, send = (torch.empty((p, q), dtype=torch.int32, device="cuda") for _ in range(2))
    rb, sb = (torch.full((p, R), 4242, dtype=torch.int32, device="cuda") for _ in range(2))
    ws = torch.empty(bcs.bcs_sched_workspace_bytes(p, 0, p), dtype=torch.uint8, device="cuda")
    bcs.bcs_sched_expand_ws(p, root, n, recv, send, rb, sb, ws)
    torch.cuda.synchronize()
    orecv, osend = oracle.sched_range(p, root=root, threads=16)
    assert np.array_equal(recv.cpu().numpy(), orecv) and np.array_equal(send.cpu().numpy(), osend)
    _check(p, n, recv, rb, oracle, 1)
    _check(p, n, send, sb, oracle, 2)
    print("bcs_expand_ws, one table", flush=True)
    sb.fill_(4242)
    ws = torch.empty(bcs.bcs_expand_workspace_bytes(p, n, 0, p), dtype=torch.uint8, device="cuda")
    bcs.bcs_expand_ws(p, n, 0, p, recv, None, sb, None, ws)
    torch.cuda.synchronize()
    assert torch.equal(rb, sb)
    del recv, send, rb, sb, ws
    torch.cuda.empty_cache()


def test_allgather_table_of_more_than_2_to_34_entries(bcs, oracle):
    """One 69 GB table, every round against the defining index arithmetic on the oracle's receive rows."""
    p, n, r = (1 << 20) + 1, 16500, 777777
    q, R = bcs.bcs_q(p), bcs.bcs_rounds(p, n)
    assert p * R > 1 << 34
    pack = torch.full((R, p), 4242, dtype=torch.int32, device="cuda")
    ws = torch.empty(bcs.bcs_allgather_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    bcs.bcs_allgather_tables_ws(p, n, r, pack, None, ws)
    torch.cuda.synchronize()
    recv = torch.from_numpy(oracle.sched_range(p, want_send=False, threads=16)[0]).cuda()
    skips, x = bcs.bcs_skips(p), (q - R % q) % q
    vr = (r - torch.arange(p, device="cuda")) % p
    cols = [recv[:, k].contiguous()[(vr + int(skips[k])) % p] for k in range(q)]
    same = torch.ones((), dtype=torch.bool, device="cuda")
    for j in range(R):
        k = (x + j) % q
        same &= (pack[j] == (cols[k] + (j - k)).clamp_(min=-1, max=n - 1)).all()
    assert bool(same)
    del pack, recv, cols, ws
    torch.cuda.empty_cache()


def test_partner_table_of_more_than_2_to_34_entries(bcs):
    """The to-processes of so many processes that a second launch writes the end of the table (69 GB): every entry against
    the distances of Alg. 7."""
    p, r0 = 2**30 + 1, 77
    q, rows = bcs.bcs_q(p), 2**34 // bcs.bcs_q(p) + 1001
    assert rows * q > 1 << 34 and r0 + rows < p
    to = torch.full((rows, q), -7, dtype=torch.int32, device="cuda")
    bcs.bcs_allgather_partners(p, r0, r0 + rows, to, None)
    torch.cuda.synchronize()
    dist = torch.tensor(bcs.bcs_skips(p)[:q], device="cuda", dtype=torch.int64)
    step = 1 << 22
    for a in range(0, rows, step):
        r = torch.arange(r0 + a, r0 + min(rows, a + step), device="cuda", dtype=torch.int64)
        assert torch.equal(to[a:a + step].long(), (r[:, None] - dist) % p), a
    del to
    torch.cuda.empty_cache()


def test_batch_of_more_than_2_to_32_triples(bcs):
    """The round counts of 2^32 + 77 triples (the last of them invalid) against the counts of their p."""
    count = (1 << 32) + 77
    p = torch.empty(count, dtype=torch.int32, device="cuda")
    zero = torch.zeros(count, dtype=torch.int32, device="cuda")
    step = 1 << 26
    for a in range(0, count, step):
        i = torch.arange(a, min(count, a + step), device="cuda", dtype=torch.int64)
        p[a:a + step] = (i * 2654435761 % ((2 << (i % 30)) - 1) + 1).to(torch.int32)
    p[-1] = 0
    q = torch.full((count,), -7, dtype=torch.int32, device="cuda")
    bcs.bcs_sched_batch(p, zero, zero, None, None, q)
    torch.cuda.synchronize()
    powers = torch.tensor([1 << k for k in range(32)], device="cuda", dtype=torch.int64)
    for a in range(0, count, step):
        want = torch.searchsorted(powers, p[a:a + step].long()).to(torch.int32)       # least k with 2^k >= p
        if a + step >= count:
            want[-1] = -1
        assert torch.equal(q[a:a + step], want), a
    del p, zero, q
    torch.cuda.empty_cache()
