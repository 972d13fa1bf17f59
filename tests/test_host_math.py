"""Device arithmetic that has to give the same bits as what it stands for, on the CPU."""
from test_host_logic import _build_and_run


def test_log_of_normal_numbers_is_the_series_bit_by_bit(tmp_path):
    assert "log_normal ok" in _build_and_run("log_normal_test.cpp", tmp_path)


def test_division_by_small_integers_is_the_rounded_quotient(tmp_path):
    assert "div_small ok" in _build_and_run("div_small_test.cpp", tmp_path)
