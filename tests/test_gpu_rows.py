"""GPU tests of the schedule kernel's cut by pieces of the tables and of the chunks of the fused schedule-and-expand call."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bcs():
    import paper_2205_10072_amd as m
    m.lib()
    return m


@pytest.fixture(scope="module")
def oracle():
    import oracle as o
    return o


@pytest.mark.parametrize("p", [2, 5, 64, 65, 128, 129, 65536, 65537, 131073, 2**20 + 1, 2**27 - 1, 2**28 + 1, 2**31 - 1])
def test_rows_of_ranges_that_end_inside_a_piece(bcs, oracle, p):
    """A workgroup writes 1024 entries (64 rows below q = 17): ranges that end before, at and after a piece, over the
    wrap of the root, with either table alone, and into outputs that allow no 16-byte stores.  Nothing past the range
    is touched."""
    q = bcs.bcs_q(p)
    per = 1024 // q if q >= 17 else 64
    rng = np.random.default_rng(p % 1000)
    for count in {1, 2, per - 1, per, per + 1, 63, 64, 65, 2 * per + 1, 1024}:
        count = min(count, p)
        r0 = int(rng.integers(0, p - count + 1))
        root = (r0 + count // 2) % p
        want = oracle.sched_range(p, root, r0, r0 + count)
        for shift in (0, 1):
            bufs = [torch.full((count * q + 8,), 777, dtype=torch.int32, device="cuda") for _ in range(4)]
            outs = [b[shift:shift + count * q] for b in bufs]
            bcs.bcs_sched_rooted(p, root, r0, r0 + count, outs[0], outs[1])
            bcs.bcs_sched_rooted(p, root, r0, r0 + count, outs[2], None)
            bcs.bcs_sched_rooted(p, root, r0, r0 + count, None, outs[3])
            for i, b in enumerate(bufs):
                got = b.cpu().numpy()
                assert np.array_equal(got[shift:shift + count * q].reshape(count, q), want[i % 2]), (p, r0, count, shift, i)
                assert (got[:shift] == 777).all() and (got[shift + count * q:] == 777).all(), (p, r0, count, shift, i)


@pytest.mark.parametrize("p,n", [(5, 30), (10001, 40), (10001, 3), (300007, 400), (1500001, 20)])
def test_sched_expand_with_any_workspace(bcs, oracle, p, n):
    """Both tables at once, table by table (block tables above 128 MB), and in chunks of ranks: a workspace of the schedules'
    size alone holds no byte rows of both tables (up to 128 MB a table: bcs_expand; above: chunks), and the byte rows of
    1500001 ranks exceed 32 MB."""
    q, R, root = bcs.bcs_q(p), bcs.bcs_rounds(p, n), p // 3
    want = oracle.sched_range(p, root, 0, p)
    blocks = [oracle.expand(p, n, w) for w in want]
    for nbytes in {bcs.bcs_sched_workspace_bytes(p, 0, p), bcs.bcs_sched_expand_workspace_bytes(p, n)}:
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        outs = [torch.full((p, w), 777, dtype=torch.int32, device="cuda") for w in (q, q, R, R)]
        bcs.bcs_sched_expand_ws(p, root, n, *outs, ws)
        for got, exp in zip(outs, list(want) + blocks):
            assert np.array_equal(got.cpu().numpy(), exp), (p, n, nbytes)
