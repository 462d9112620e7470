"""The forms in which the binding takes its host arguments: coefficients as
fp32 arrays (the short way), fp64 or strided arrays, lists, tuples, and
iterators; shapes with Python or numpy numbers; empty and non-contiguous
tensors.  All through calls that need no GPU."""
import numpy as np
import pytest
import torch

import tracegen


@pytest.fixture(scope="module")
def llmv():
    from paper_2608_08382_amd import llmv as mod
    mod.load()
    return mod


def host(llmv, co, shape):
    off = np.array([0, 2, 5], np.int64)
    p = np.array([1, 1, 7, 1, 1], np.int32)
    c = np.array([9, 4, 0, 3, 2], np.int32)
    t = np.array([0, 1, 1, 0, 2], np.int32)
    return llmv.llmv_attribute_host(off, p, c, t, shape, co, 3)


def test_coefficient_forms(llmv):
    co = tracegen.base_coeffs(11)
    shape = tracegen.SHAPES["70b-like"]
    want = host(llmv, co, shape)
    wide = np.empty(40, np.float32)
    wide[::2] = co
    for form in (co.copy(), co.astype(np.float64), wide[::2], list(co), tuple(float(v) for v in co),
                 (float(v) for v in co), torch.from_numpy(co), co.astype(">f4")):
        got = host(llmv, form, shape)
        for k in want:
            assert np.array_equal(got[k], want[k]), (type(form), k)


def test_coefficient_counts(llmv):
    co = tracegen.base_coeffs(11)
    # fewer than 20 are filled up with zeros, more are refused
    short, full = co[:19].copy(), co.copy()
    full[19] = 0.0
    a, b = host(llmv, short, None), host(llmv, full, None)
    assert all(np.array_equal(a[k], b[k]) for k in a)
    with pytest.raises(Exception):
        host(llmv, np.zeros(21, np.float32), None)


def test_shape_forms(llmv):
    shape = tracegen.SHAPES["qwen2.5-14b"]
    want = llmv.llmv_shape_constants(shape)
    assert llmv.llmv_shape_constants({k: np.int64(v) for k, v in shape.items()}) == want
    assert llmv.llmv_shape_constants({k: float(v) for k, v in shape.items()}) == want
    assert llmv.llmv_shape_constants(llmv.make_shape(shape)) == want
    with pytest.raises(KeyError):
        llmv.llmv_shape_constants({"n_layers": 1})


def test_tensor_forms(llmv):
    assert llmv._ptr(None) is None
    assert llmv._ptr(torch.empty(0)) is None
    assert llmv._ptr(torch.zeros((0, 3)).t()) is None
    x = torch.zeros(4)
    assert llmv._ptr(x) == x.data_ptr() and llmv._ptr(x[1:]) == x.data_ptr() + 4
    with pytest.raises(ValueError):
        llmv._ptr(torch.zeros((2, 3)).t())
    with pytest.raises(TypeError):
        llmv._ptr(np.zeros(3))
