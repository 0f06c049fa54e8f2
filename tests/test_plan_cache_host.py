"""Plan-cache entries of many-plans (tuned among the rules' kernels, pass by
pass) and of single plans, on the host."""
import ctypes

import pytest

from paper_1501_07350_amd import _lib

DIMS = (60, 64, 90)
RULES = "order=cba;a=5x4x3/32/x;b=16x4/32/x;c=5x3x3x2/16"      # kernels of the radix-sequence rules
OTHER = "order=abc;a=5x4x3/32/x;b=16x4/32/x;c=5x3x3x2/16"
TABLE = "order=cba;a=10x6/32/x;b=16x4/32/x;c=10x9/16/10"       # with kernels of the default table only


@pytest.fixture()
def cache(tmp_path):
    path = str(tmp_path / "plans.txt")
    f = _lib.load().offt_test_plan_cache
    f.argtypes = [ctypes.c_char_p, ctypes.c_int, ctypes.POINTER(ctypes.c_int64), ctypes.c_int, ctypes.c_char_p, ctypes.c_char_p,
                  ctypes.c_size_t]
    f.restype = ctypes.c_int

    def call(many, store=None):
        buf = ctypes.create_string_buffer(512)
        rc = f(path.encode(), 1, (ctypes.c_int64 * 3)(*DIMS), int(many), store.encode() if store else None, buf, 512)
        return buf.value.decode() if rc > 0 else rc
    call.path = path
    return call


def test_a_many_plans_entry_is_not_a_single_plans(cache):
    assert cache(True, RULES) == RULES
    assert cache(False) == _lib.ERR_IO
    assert cache(False, TABLE) == TABLE
    assert cache(True) == RULES
    keys = [ln.split("\t")[0] for ln in open(cache.path)]
    assert len(set(keys)) == 2


def test_a_many_plan_takes_single_plan_entries_of_its_own_kernels(cache):
    """Files of earlier versions have one kind of entry."""
    assert cache(False, RULES) == RULES
    assert cache(True) == RULES
    # the latest one, unless its own kind is there
    assert cache(False, OTHER) == OTHER and cache(True) == OTHER
    assert cache(True, RULES) == RULES
    assert cache(False, OTHER) == OTHER and cache(True) == RULES


def test_table_kernels_are_a_miss_for_a_many_plan(cache):
    assert cache(False, TABLE) == TABLE
    assert cache(True) == _lib.ERR_IO
