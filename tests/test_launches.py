"""CPU tests of what the calls enqueue: the real library on a stand-in runtime (launchlog.py), which refuses a launch of
2^32 lanes or more as the HIP runtime does."""
import pytest

from launchlog import launches, run, shown


def _covers(pieces, start, entries, size=4):
    """(address, entries) pieces follow one another from `start` and make up `entries`, each at a 16-byte address."""
    at = start
    for address, count in pieces:
        assert address == at and address % 16 == 0 and count > 0
        at += count * size
    assert at == start + entries * size


BIG = [((1 << 20) + 1, 17000), ((1 << 20) + 1, 16405), (9, 2**31 - 100), (33, 600000000), (70000, 300000)]


@pytest.mark.parametrize("need", ["L.bcs_sched_workspace_bytes(p, 0, p, 1)", "L.bcs_sched_expand_workspace_bytes(p, n)"])
@pytest.mark.parametrize("p,n", BIG)
def test_block_tables_of_more_than_2_to_34_entries_in_one_call(tmp_path, p, n, need):
    """bcs_sched_expand_ws, with the schedules' workspace alone and with its own: every launch stays below 2^32 lanes and
    the pieces of both block tables are complete."""
    log = run(tmp_path, """
p, n = %d, %d
show(L.bcs_sched_expand_ws(p, 1, n, T(1), T(2), T(3), T(4), T(5), %s, None))
""" % (p, n, need))
    assert shown(log) == [0]
    R = n - 1 + (p - 1).bit_length()
    for table in (3, 4):
        _covers([(e["arg"][3], e["arg"][0]) for e in launches(log, "k_expand_rows") if e["arg"][3] >> 44 == table],
                table << 44, p * R)


@pytest.mark.parametrize("p,n", BIG)
def test_block_tables_of_more_than_2_to_34_entries_from_schedule_rows(tmp_path, p, n):
    log = run(tmp_path, """
need = L.bcs_expand_workspace_bytes(%d, %d, 1, %d)
show(L.bcs_expand_ws(%d, %d, 1, %d, T(1), T(2), T(3), T(4), T(5), need, None))
""" % (p, n, p, p, n, p))
    R, q = n - 1 + (p - 1).bit_length(), (p - 1).bit_length()
    assert shown(log) == [0]
    for table in (3, 4):
        _covers([(e["arg"][3], e["arg"][0]) for e in launches(log, "k_expand_rows") if e["arg"][3] >> 44 == table],
                table << 44, (p - 1) * R)
    # each expansion reads what the conversion before it left: the same rows
    todo = launches(log)
    for made, used in zip(todo[0::2], todo[1::2]):
        assert (made["name"], used["name"]) == ("k_rows_to_bytes", "k_expand_rows")
        assert made["arg"][0] * R == used["arg"][0] and made["arg"][5] == used["arg"][1] == 5 << 44
        first = (used["arg"][3] - ((used["arg"][3] >> 44) << 44)) // (4 * R)
        assert made["arg"][4] == ((used["arg"][3] >> 44) - 2 << 44) + 4 * first * q


@pytest.mark.parametrize("p,n,one", [((1 << 20) + 1, 17000, False), ((1 << 20) + 1, 17000, True), (9, 2**31 - 100, False),
                                     ((1 << 20) + 1, 16300, False)])
def test_allgather_tables_of_more_than_2_to_34_entries(tmp_path, p, n, one):
    log = run(tmp_path, """
need = L.bcs_allgather_workspace_bytes(%d)
show(L.bcs_allgather_tables_ws(%d, %d, 3, T(1), %s, T(3), need, None))
""" % (p, p, n, "None" if one else "T(2)"))
    assert shown(log) == [0]
    last = launches(log)[-1]
    flat = p * (n - 1 + (p - 1).bit_length()) < 1 << 34            # else by slots and pieces of 4096 roots
    assert last["name"] == ("k_allgather_tables_flat" if flat else "k_allgather_tables")
    assert last["grid"][:2] == ([last["grid"][0], 2] if flat else [(p + 4095) // 4096, (p - 1).bit_length()])


@pytest.mark.parametrize("call", ["bcs_allgather_partners", "bcs_census_partners"])
@pytest.mark.parametrize("p,r0,r1", [(2**31 - 1, 0, 2**31 - 1), (2**30 + 1, 5, 2**30), (2**29 + 1, 0, 2**29 + 1)])
def test_partner_tables_of_any_length(tmp_path, call, p, r0, r1):
    log = run(tmp_path, "show(L.%s(%d, %d, %d, T(1), T(2), None))" % (call, p, r0, r1))
    assert shown(log) == [0]
    q, done = (p - 1).bit_length(), launches(log, "k_partner_tables")
    for table in (1, 2):
        _covers([(e["arg"][4 + table], e["arg"][4]) for e in done], table << 44, (r1 - r0) * q)
    row = r0
    for e in done:                                                   # the first process of each piece
        assert e["arg"][:4] == [p, q, int("census" in call), row] and e["arg"][4] % q == 0
        assert e["lanes"] * 4 >= e["arg"][4]
        row += e["arg"][4] // q
    assert row == r1


def test_plans_of_more_rounds_than_a_launch_has_workgroups(tmp_path):
    p, rounds = 3, (1 << 25) + 5
    log = run(tmp_path, "show(L.bcs_pack_plan_rounds(%d, %d, %d, T(1), T(2), T(3), T(4), None))" % (p, rounds, rounds))
    assert shown(log) == [0]
    at = 0
    for e in launches(log, "k_pack_plan_one"):
        assert e["arg"][2] == (1 << 44) + 4 * p * at and e["arg"][3] == 2 << 44
        assert e["arg"][4] == (3 << 44) + 8 * (p + 1) * at          # the plan's first member: where the offsets go
        at += e["grid"][0]
    assert at == rounds


def test_batches_of_more_than_2_to_32_triples(tmp_path):
    """Only the round counts asked for: 69 GB of triples and counts, which the card holds."""
    count = (1 << 32) + 77
    log = run(tmp_path, "show(L.bcs_sched_batch(%d, T(1), T(2), T(3), None, None, T(4), None))" % count)
    assert shown(log) == [0]
    at = 0
    for e in launches(log, "k_batch"):
        assert e["arg"][1:4] == [(t << 44) + 4 * at for t in (1, 2, 3)] and e["arg"][4:6] == [0, 0]
        assert e["arg"][6] == (4 << 44) + 4 * at and 0 < e["arg"][0] <= e["lanes"]
        at += e["arg"][0]
    assert at == count
    log = run(tmp_path, "show(L.bcs_sched_batch(%d, T(1), T(2), T(3), T(5), T(6), None, None))" % count)
    at = 0
    for e in launches(log, "k_batch"):
        assert e["arg"][4:7] == [(5 << 44) + 128 * at, (6 << 44) + 128 * at, 0]
        at += e["arg"][0]
    assert at == count


@pytest.mark.parametrize("p,n", [(33, 2**31 - 100), (5000000, 13800), (40, 2**31 - 100)])
def test_expansion_without_workspace_of_more_lanes_than_a_launch_has(tmp_path, p, n):
    """Sixteen entries a lane: a table of 275 GB and more."""
    log = run(tmp_path, "show(L.bcs_expand(%d, %d, 1, %d, T(1), T(2), T(3), T(4), None))" % (p, n, p))
    assert shown(log) == [0]
    R, q = n - 1 + (p - 1).bit_length(), (p - 1).bit_length()
    done = launches(log, "k_expand")                                 # arg: entries, rows of both tables, both block tables
    for table in (3, 4):
        mine = [e["arg"] for e in done if e["arg"][3] >> 44 == table]
        _covers([(a[3], a[0]) for a in mine], table << 44, (p - 1) * R)
        for a in mine:
            first = (a[3] - (table << 44)) // (4 * R)
            assert a[1] == ((table - 2) << 44) + 4 * q * first and a[2] == a[4] == 0


@pytest.mark.parametrize("call", ["bcs_pack_round_planned(3, T(1), T(2), T(3), T(4), 1 << 38, None)",
                                  "bcs_pack_round(3, 4, T(1), T(2), T(3), T(4), 1 << 38, T(5), T(6), 1 << 20, None)",
                                  "bcs_valu_peak_launch(1 << 24, 1, T(1), None)"])
def test_sizes_beyond_a_launch_and_the_card_are_refused_before_anything_is_enqueued(tmp_path, call):
    log = run(tmp_path, "show(L.%s)" % call)
    assert shown(log) == [-1] and not launches(log)


PLAIN = {"bcs_sched_expand": "L.bcs_sched_expand(%s, 0, 300, T(1), T(2), T(3), T(4), %s)",
         "bcs_allgather_tables": "L.bcs_allgather_tables(%s, 300, 0, T(1), T(2), %s)"}


@pytest.mark.parametrize("first", PLAIN)
@pytest.mark.parametrize("second", list(PLAIN) + ["bcs_release"])
def test_plain_calls_of_two_threads_do_not_come_between_one_another(tmp_path, first, second):
    """Plain calls share one allocation.  While one is enqueueing its kernels (each launch takes 50 ms here), another
    thread calls with more ranks, or releases: the allocation may be freed, and the other stream ordered behind the
    first, only when the first call's kernels are all enqueued."""
    other = PLAIN[second] % (8000000, "3 << 20") if second in PLAIN else "L.bcs_release()"
    log = run(tmp_path, """
L.bcs_sched_rooted_ws(5, 0, 0, 5, T(1), None, None, 0, None)           # fills the tables
S.stub_reset()
S.stub_slow(2 << 20, 50000)
rcs = [None, None]
def one(): rcs[0] = %s
def two(): rcs[1] = %s
a, b = threading.Thread(target=one), threading.Thread(target=two)
a.start()
while not S.stub_count(): time.sleep(0.001)                            # it has its memory
time.sleep(0.01)
b.start()
a.join()
b.join()
show(rcs)
""" % (PLAIN[first] % (1000003, "2 << 20"), other))
    assert shown(log) == [[0, 0]]
    last = max(i for i, (kind, e) in enumerate(log) if kind == "launch" and e["stream"] == 2 << 20)
    assert all(kind in ("launch", "malloc") and e["stream"] in (0, 2 << 20) for kind, e in log[:last])
    freed = [i for i, (kind, e) in enumerate(log) if kind == "free"]
    assert len(freed) == 1 and freed[0] > last


def test_a_plain_call_on_another_stream_is_ordered_behind_all_of_the_call_before(tmp_path):
    """The same with the same sizes: no allocation changes hands, the order between the streams is what counts."""
    log = run(tmp_path, """
L.bcs_sched_rooted_ws(5, 0, 0, 5, T(1), None, None, 0, None)
S.stub_reset()
S.stub_slow(2 << 20, 50000)
a = threading.Thread(target=lambda: L.bcs_sched_expand(1000003, 0, 300, T(1), T(2), T(3), T(4), 2 << 20))
b = threading.Thread(target=lambda: L.bcs_sched_expand(1000003, 0, 300, T(5), T(6), T(7), T(8), 3 << 20))
a.start()
while not S.stub_count(): time.sleep(0.001)
time.sleep(0.01)
b.start()
a.join()
b.join()
""")
    order = [(kind, e["stream"] >> 20) for kind, e in log if kind in ("launch", "record", "wait")]
    mine = order.count(("launch", 2))
    assert mine > 1 and order == [("launch", 2)] * mine + [("record", 2), ("wait", 3)] + [("launch", 3)] * mine


@pytest.mark.parametrize("p,n", [(1000, 16), (1000, 64), (10001, 40), (20000, 200), (200003, 14), (65537, 400)])
def test_one_call_with_the_schedules_workspace_alone_takes_two_launches_while_it_is_short(tmp_path, p, n):
    """Byte rows of both tables do not fit such a workspace; short calls are bound by their launches."""
    log = run(tmp_path, """
p, n = %d, %d
L.bcs_sched_rooted_ws(5, 0, 0, 5, T(1), None, None, 0, None)
S.stub_reset()
L.bcs_sched_expand_ws(p, 0, n, T(1), T(2), T(3), T(4), T(5), L.bcs_sched_workspace_bytes(p, 0, p, 1), None)
""" % (p, n))
    assert [e["name"] for e in launches(log)] == ["k_sched", "k_expand"]


@pytest.mark.parametrize("p,capacity,want", [(2048, 512 << 10, ["k_pack_round"]), (1, 1, ["k_pack_round"]),
                                             (2048, (512 << 10) + 1, ["k_pack_plan_one", "k_pack_copy"]),
                                             (2049, 1000, ["k_pack_plan_one", "k_pack_copy"]),
                                             (8192, 1000, ["k_pack_plan_one", "k_pack_copy"]), (2048, 0, ["k_pack_plan_one"]),
                                             (8193, 0, ["k_pack_plan_local", "k_pack_plan_totals", "k_pack_plan_finish"])])
def test_launches_of_a_packed_round(tmp_path, p, capacity, want):
    log = run(tmp_path, "show(L.bcs_pack_round(%d, 4, T(1), T(2), T(3), T(4), %d, T(5), T(6), 1 << 20, None))" % (p, capacity))
    assert shown(log) == [0] and [e["name"] for e in launches(log)] == want
