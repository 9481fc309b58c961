"""Workspace of FP32 calls whose schedule grows on [0, 1] (FP32 MFMA) against the
same calls with the l = 1e-3 schedule (fp16 planes): the same arrays, so that they
differ by less than 64 KiB of tables and partial sums and, where K is split, by
partial tiles, of which split_k = 1 has none."""
import ctypes

import numpy as np
import pytest

import paper_2505_16932_amd as pe


def _bytes(shape, abc, **kw):
    o, _keep = pe._opts(len(abc), np.asarray(abc).reshape(-1), "f32", 0, 0, 1, split_k=1, **kw)
    mat = (pe.Matrix * 1)()
    mat[0] = pe.Matrix(4096, 4096, *shape, shape[1], shape[1], pe.PE_F32, pe.PE_F32)
    return int(pe.lib().pe_workspace_size(1, mat, ctypes.byref(o)))


@pytest.mark.parametrize("kw", [dict(), dict(fast_restart=3)])
@pytest.mark.parametrize("shape", [(128, 256), (300, 1100), (1024, 4096), (2500, 2500)])
def test_workspace_does_not_depend_on_growth(shape, kw):
    plain = np.asarray(pe.coeffs(1e-3, 5).abc).reshape(5, 3)
    growing = plain.copy()
    growing[0] = (16.0, 0.0, 0.0)
    assert abs(_bytes(shape, plain, **kw) - _bytes(shape, growing, **kw)) < 65536
