"""Null arguments of the calls that need no device to be refused."""
import ctypes

from paper_2505_02438_amd import _lib


def test_backward_scratch_refuses_null():
    L = _lib.lib()
    n = ctypes.c_int64(-7)
    mat = _lib.Material(1.0, 1e-9, 0.3, 3.0, 0)
    assert L.soptx_backward_scratch_size(None, ctypes.byref(n)) == -1 and n.value == -7
    assert L.soptx_assemble_backward_scratch(None, ctypes.byref(mat), None, None, None, None, 0, None, 0, None) == -1


def test_oc_form_before_any_update():
    L = _lib.lib()
    f = ctypes.c_int32(-7)
    assert L.soptx_debug_oc_form(None) == -1
    assert L.soptx_debug_oc_form(ctypes.byref(f)) == 0 and f.value == -1


def test_pcg_variant_takes_its_values_only():
    L = _lib.lib()
    assert [L.soptx_debug_set_pcg_variant(v) for v in (0, 1, -2, -1)] == [0, -1, -1, 0]


def test_fail_optional_refuses_negative_counts():
    L = _lib.lib()
    assert [L.soptx_debug_fail_optional(a, b) for a, b in ((-1, 0), (0, -1), (0, 0))] == [-1, -1, 0]
