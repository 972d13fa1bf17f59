"""The packed network tables, on the CPU."""
from test_host_logic import _build_and_run


def test_packed_tables_are_the_reactions(tmp_path):
    assert "net tables ok" in _build_and_run("nettables_test.cpp", tmp_path)
