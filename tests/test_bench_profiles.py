"""CPU tests of what bench.py prints from counter profiles: figures are tied to the code they were taken on."""
import os

import pytest

import bench

PROFILES = os.path.join(os.path.dirname(os.path.abspath(bench.__file__)), "profiles")


def test_the_digest_is_of_the_code():
    code = bench.code_only('int a = 1; // one\n/* two\n   lines */ int b;\nchar s[] = "// no comment \\" /* nor this */";')
    assert code == 'int a = 1; int b; char s[] = "// no comment \\" /* nor this */";'
    assert bench.code_only("int  a;\n\n// x\nint b;") == bench.code_only("int a; int b;  // y")
    assert bench.code_only("int a;") != bench.code_only("int b;")


@pytest.mark.parametrize("key", bench.PROFILED, ids=" ".join)
def test_every_entry_names_the_profile_and_the_code_it_comes_from(key):
    ent = bench.PROFILED[key]
    with open(os.path.join(PROFILES, ent["source"]), encoding="utf-8") as f:
        text = f.read()
    assert "`%s`" % ent["csrc"] in text, "the profile was taken on other code than the entry says"
    for field in ("fetch_kib", "write_kib"):
        assert format(ent[field], ",").replace(",", " ") in text, (key, field)
    assert str(ent["valu_per_wave"]) in text and str(ent["salu_per_wave"]) in text, key


def test_an_entry_of_other_code_is_stale():
    key = ("C4", "k_expand_rows")
    digest = bench.PROFILED[key]["csrc"]
    assert bench.profiled(*key, digest)["stale"] is False
    rec = bench.profiled(*key, "0" * 16)
    assert rec["stale"] is True and rec["profiled_at_csrc"] == digest and rec["source"].startswith("profiles/c4_")
    assert bench.profiled("C9", "k_none", digest) is None
