"""GPU test of a round packed and unpacked by one launch (few processes, short messages) around the sizes where the launch
changes: lanes' shares of the roots, the last root, capacities that end inside a piece, messages off 16 bytes."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [1, 2, 3, 255, 256, 257, 511, 513, 1152, 2047, 2048, 2049])
@pytest.mark.parametrize("mean,n", [(0, 3), (7, 3), (300, 5), (2000, 7)])
def test_round_in_one_launch(p, mean, n):
    import oracle
    import paper_2205_10072_amd as bcs
    rng = np.random.default_rng(p * 10 + n)
    sizes = rng.integers(0, 2 * mean + 1, p) * rng.integers(0, 2, p)            # half of the buffers are empty
    displs = np.zeros(p + 1, dtype=np.int64)
    np.cumsum(sizes, out=displs[1:])
    idx = rng.integers(-1, n + 2, p).astype(np.int32)                            # no block, blocks, and beyond the last
    data = rng.integers(0, 1 << 30, int(displs[p]) + 1).astype(np.int32)
    want, want_offsets = oracle.pack_round(n, idx, displs, data)
    length = len(want)
    d_idx, d_displs = torch.from_numpy(idx).cuda(), torch.from_numpy(displs).cuda()
    ws = torch.empty(bcs.bcs_pack_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    for shift in (0, 1):
        for capacity in {length + 5, length, max(length - 3, 0), 512 << 10, (512 << 10) + 1}:       # the last: two launches
            offsets = torch.full((p + 1,), -1, dtype=torch.int64, device="cuda")
            buf = torch.full((capacity + 8,), 777, dtype=torch.int32, device="cuda")
            bcs.bcs_pack_round(n, d_idx, d_displs, torch.from_numpy(data).cuda(), buf[shift:shift + capacity], offsets, ws)
            got, m = buf.cpu().numpy(), min(capacity, length)
            assert np.array_equal(got[shift:shift + m], want[:m]), (shift, capacity)
            assert (got[:shift] == 777).all() and (got[shift + m:] == 777).all(), (shift, capacity)
            assert np.array_equal(offsets.cpu().numpy(), want_offsets)
        message = rng.integers(0, 1 << 30, length + 8).astype(np.int32)
        exp = data.copy()
        oracle.unpack_round(n, idx, displs, exp, np.ascontiguousarray(message[shift:shift + length]))
        d_data = torch.from_numpy(data).cuda()
        bcs.bcs_unpack_round(n, d_idx, d_displs, d_data, torch.from_numpy(message).cuda()[shift:shift + length], length,
                             offsets, ws)
        assert np.array_equal(d_data.cpu().numpy(), exp), shift
