"""nr_plan_launches rejects bad arguments (its answers are read by the GPU tests of the
schedule)."""
import ctypes


def test_arguments():
    from paper_2509_06924_amd import _native as n
    L, k = n.lib(), ctypes.c_int32()
    assert L.nr_plan_launches(None, 2, 0, None, ctypes.byref(k)) == n.NR_EINVAL
