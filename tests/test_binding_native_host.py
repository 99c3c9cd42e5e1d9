"""The C half of the Python binding against the ctypes structures it stands for, without a GPU: the same bytes, the same refusals, and
unusual arguments handed on to ctypes."""
import ctypes
import importlib.machinery
import os

import pytest
import torch

from paper_2605_19269_amd import coda


def _tensors():
    t = torch.zeros(6, 16, dtype=torch.bfloat16)
    return [t, t[:, 8:], t[2:4], t[:0], t[:, :1], torch.zeros(4, 16, dtype=torch.uint8), torch.zeros(4, 16, dtype=torch.float8_e4m3fn), torch.zeros(3, 8)]


@pytest.mark.parametrize("i", range(8))
@pytest.mark.parametrize("trans", [False, True])
def test_operands(i, trans):
    t = _tensors()[i]
    assert coda._binding.mat(t, trans, coda._DTYPES if coda._torch else (coda._import_torch(), coda._DTYPES)[1]) == bytes(coda.mat(t, trans))


def test_sizes_of_a_product():
    coda._import_torch()
    A, B = torch.zeros(3, 5), torch.zeros(5, 7)
    for ta in (False, True):
        for tb in (False, True):
            a, b = (A.t().contiguous() if ta else A), (B.t().contiguous() if tb else B)
            assert coda._binding.gemm_mats(a, b, ta, tb, coda._DTYPES) == (3, 7, 5, bytes(coda.mat(a, ta)), bytes(coda.mat(b, tb)))


@pytest.mark.parametrize("bad", [torch.zeros(4), torch.zeros(2, 3, 4), torch.zeros(4, 8).t()])
def test_what_is_no_row_major_matrix_is_refused(bad):
    ok = torch.zeros(4, 4)
    for call in (lambda: coda.mat(bad), lambda: coda.coda_gemm(bad, ok, [], stream=0), lambda: coda.coda_gemm(ok, bad, [], stream=0),
                 lambda: coda.coda_row_sumsq(bad, torch.zeros(4), stream=0)):
        with pytest.raises(AssertionError):
            call()


def test_ops_hold_pointers_pitches_and_tensors():
    m, v = torch.zeros(4, 24)[:, :16], torch.zeros(16)
    o = coda.rmsnorm_bwd(m, v, v[1:], v[2:], c_out=m[1:], dgamma_out=v[3:], z_sum_over=11)
    assert (o.kind, o.flags, o.in_, o.ld_in, o.out, o.ld_out, o.out2) == (coda.CODA_EPI_RMSNORM_BWD, 0, m.data_ptr(), 24, m[1:].data_ptr(), 24, v[3:].data_ptr())
    assert (o.in2, o.in3, o.in4, o.out3, o.i0, o.i1) == (v.data_ptr(), v[1:].data_ptr(), v[2:].data_ptr(), None, 11, 0)
    assert o._keep[0] is m and isinstance(o, coda.coda_epi_op)
    o = coda.row_scale(v)
    assert (o.in_, o.ld_in, o.out, o.ld_out) == (v.data_ptr(), 0, None, 0)          # a pitch is a matrix's
    assert coda.rmsnorm_bwd(m, v, v, v, z_sum_over=None).i0 == 0
    for bad in (lambda: coda.row_scale(3), lambda: coda.rmsnorm_bwd(m, v, v, v, z_sum_over=1.5)):
        with pytest.raises((TypeError, AttributeError)):
            bad()


@pytest.mark.parametrize("n", [-1, 0, True, 2 ** 63 - 1, 2 ** 63, 2 ** 64 - 8, 2 ** 64 + 128, -2 ** 63, -2 ** 70 - 3])
def test_whole_numbers_of_any_size(n):
    m, v = torch.zeros(4, 16), torch.zeros(16)
    field = coda.coda_epi_op(0, 0, i0=n, i1=n)
    assert coda.rmsnorm_bwd(m, v, v, v, z_sum_over=n).i0 == field.i0
    o = coda.rope(m, m, v, n, n)
    assert (o.i0, o.i1) == (field.i0, field.i1)


def test_programs_are_the_structures_one_after_the_other():
    v = torch.zeros(16)
    ops = [coda.row_scale(v), coda.store(v.view(4, 4)), coda.coda_epi_op(9, 8, 7)]
    for n in range(4):
        arr, count = coda._prog(ops[:n])
        assert coda._binding.prog(ops[:n], coda.coda_epi_op) == bytes(arr) and count == n
    assert coda._binding.prog([ops[0], (1, 2)], coda.coda_epi_op) is None              # ctypes takes tuples for structures


def test_calls_take_every_form_of_argument():
    X, out = torch.zeros(0, 8, dtype=torch.bfloat16), torch.zeros(4)
    for stream in (0, None, ctypes.c_void_p(None), type("S", (), {"cuda_stream": 0})()):
        coda.coda_row_sumsq(X, out, stream=stream if stream is not None else 0)
        coda.coda_row_finalize(out, 0, 1, sum_out=out, d=4, eps=0, stream=stream if stream is not None else 0)   # an int eps
    m = coda.mat(X)
    assert coda._lib.coda_row_sumsq(None, ctypes.byref(m), out.data_ptr()) == coda.CODA_OK
    assert coda._lib.coda_row_sumsq(None, None, out.data_ptr()) == coda.CODA_ERR_NULL
    with pytest.raises((ctypes.ArgumentError, TypeError)):
        coda.coda_row_finalize(out, 1.0, 1, sum_out=out, stream=0)
    with pytest.raises(coda.CodaError):
        coda.coda_row_finalize(out, 4, 1, stream=0)                                      # no output


def test_the_extension_is_that_of_this_interpreter():
    from paper_2605_19269_amd import build
    suffix = importlib.machinery.EXTENSION_SUFFIXES[0]                                   # .cpython-<version>-<platform>.so
    assert "cpython" in suffix and coda._binding.__file__.endswith("_binding" + suffix)
    assert os.path.samefile(coda._binding.__file__, build.BINDING)
