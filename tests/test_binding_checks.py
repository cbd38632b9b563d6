"""Host-side argument checks of the binding (CPU only): tensors that do not
match a plan's storage type or shape, or coefficient arrays that are too
short, are refused before any pointer reaches the library."""
import pytest
import torch

from paper_2107_13500_amd import binding as B


def fields(nx=6, ny=5, nz=8, dtype=torch.float64):
    return [torch.zeros(nx + 2, ny + 2, nz, dtype=dtype) for _ in range(6)]


def coefs(nz=8, dtype=torch.float64):
    return [torch.zeros(nz, dtype=dtype) for _ in range(4)]


SHAPE = B.PwShape(6, 5, 8, 0, 0, 0)


def test_wrong_storage_dtype_is_refused():
    with pytest.raises(ValueError, match="dtype"):
        B.check_fields(B.F64, SHAPE, fields(dtype=torch.float32), coefs())
    f = fields()
    f[4] = f[4].float()
    with pytest.raises(ValueError, match="sv has dtype"):
        B.check_fields(B.F64, SHAPE, f, coefs())


def test_smaller_or_differently_strided_fields_are_refused():
    f = fields()
    f[3] = torch.zeros(7, 7, 8, dtype=torch.float64)   # one x plane short
    with pytest.raises(ValueError, match="su has shape"):
        B.check_fields(B.F64, SHAPE, f, coefs())
    f = fields()
    f[0] = torch.zeros(8, 7, 10, dtype=torch.float64)[:, :, :8]   # padded columns: sy = 10, not nz
    with pytest.raises(ValueError, match="u has shape"):
        B.check_fields(B.F64, SHAPE, f, coefs())


def test_short_or_non_double_coefficients_are_refused():
    with pytest.raises(ValueError, match="at least nz"):
        B.check_fields(B.F64, SHAPE, fields(), coefs(nz=7))
    with pytest.raises(ValueError, match="float64"):
        B.check_fields(B.F64, SHAPE, fields(), coefs(dtype=torch.float32))


def test_host_tensors_are_refused_for_device_calls():
    with pytest.raises(ValueError, match="CUDA tensor"):
        B.check_fields(B.F64, SHAPE, fields(), coefs())


class FakePlan:
    storage = B.F64
    shapes = [SHAPE]
    _layout = None


class OnDevice:
    """A host tensor that reports a GPU device, so that the comparisons of a
    device call can be checked without one."""

    def __init__(self, t, dev=0):
        self.t, self.dev, self.is_cuda = t, dev, dev >= 0
        self.dtype, self.shape = t.dtype, t.shape
        self.stride, self.numel, self.is_contiguous = t.stride, t.numel, t.is_contiguous

    def get_device(self):
        return self.dev


def test_the_quick_check_refuses_whatever_check_fields_refuses():
    """fields_fit accepts only what check_fields accepts: one wrong property in
    any of the ten tensors makes it fall back to the naming check."""
    good = [OnDevice(t) for t in fields()], [OnDevice(t) for t in coefs()]
    assert B.fields_fit(FakePlan(), *good)
    bad_fields = [torch.zeros(8, 7, 8, dtype=torch.float32), torch.zeros(7, 7, 8, dtype=torch.float64),
                  torch.zeros(8, 7, 10, dtype=torch.float64)[:, :, :8], torch.zeros(8, 7, 16, dtype=torch.float64)[:, :, ::2],
                  torch.zeros(8, 8, 7, dtype=torch.float64).transpose(1, 2), torch.zeros(8, 7, 8, 1, dtype=torch.float64)]
    for i in range(6):
        for t in bad_fields:
            f = list(good[0])
            f[i] = OnDevice(t)
            assert not B.fields_fit(FakePlan(), f, good[1]), (i, t.shape, t.stride())
        f = list(good[0])
        f[i] = OnDevice(fields()[0], dev=1)
        assert not B.fields_fit(FakePlan(), f, good[1])
    for i in range(4):
        for t in (torch.zeros(8, dtype=torch.float32), torch.zeros(7, dtype=torch.float64),
                  torch.zeros(16, dtype=torch.float64)[::2]):
            z = list(good[1])
            z[i] = OnDevice(t)
            assert not B.fields_fit(FakePlan(), good[0], z)
        z = list(good[1])
        z[i] = OnDevice(coefs()[0], dev=1)
        assert not B.fields_fit(FakePlan(), good[0], z)
    host = [OnDevice(t, dev=-1) for t in fields()], [OnDevice(t, dev=-1) for t in coefs()]
    assert not B.fields_fit(FakePlan(), *host)


def test_the_quick_check_leaves_host_arrays_and_layouts_without_strides_to_the_naming_check():
    """What is no tensor of plain strides gets check_fields' own error, not one
    from a query that it lacks."""
    import numpy as np
    good = [OnDevice(t) for t in fields()], [OnDevice(t) for t in coefs()]
    for odd in (np.zeros((8, 7, 8)), None, torch.zeros(8, 7, 8, dtype=torch.float64).to_sparse()):
        for i in range(6):
            f = list(good[0])
            f[i] = odd
            assert not B.fields_fit(FakePlan(), f, good[1])
        for i in range(4):
            z = list(good[1])
            z[i] = odd
            assert not B.fields_fit(FakePlan(), good[0], z)
    with pytest.raises(ValueError, match="dtype"):
        B.check_fields(B.F64, SHAPE, [np.zeros((8, 7, 8))] * 6, coefs())
