"""The shortened forms of the random draws give what the plain ones give: the FP32
Box-Muller radius over all 2^23 uniforms bit for bit, and the Metropolis test, which
takes the uniform's FP32 logarithm first, the FP64 decision for thresholds from an ulp
to far from it.
"""
import ctypes
import os

import numpy as np
import pytest

from gpu_helpers import gpu_available

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import torch  # noqa: E402

from paper_2002_01184_amd import build  # noqa: E402


@pytest.fixture(scope="module")
def checks():
    if not os.path.exists(build.DEVICE_CHECK):
        build.build_device_check()
    return ctypes.CDLL(build.DEVICE_CHECK)


def test_box_muller_over_all_uniforms(checks):
    bad = torch.zeros(4, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    assert checks.check_box_muller(ctypes.c_void_p(bad.data_ptr())) == 0
    torch.cuda.synchronize()
    print("mismatches of 2^23 (uniform, radius, normals):", bad[:3].tolist())
    assert bad[:3].tolist() == [0, 0, 0]


def test_metropolis_test_decides_as_in_fp64(checks):
    mag = np.concatenate([[0.0], 10.0 ** np.arange(-17.0, 3.0), [1e-6, 3e-6, 4e-6, 5e-6, 1e-5]])
    off = np.concatenate([mag, -mag])
    fixed = np.concatenate([[0.0, -0.0, np.nan, np.inf, -np.inf, 1.0, 1e300, -1e300, -5e-324, -1e-17, -1e-8, -4e-6],
                            -np.geomspace(1e-7, 36.0, len(off) - 12)])
    o, f = (torch.from_numpy(v).cuda() for v in (off, fixed))
    bad = torch.zeros(2, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    for t in (0, 1, 12345):
        assert checks.check_below(ctypes.c_uint64(9), ctypes.c_uint32(t), ctypes.c_void_p(o.data_ptr()),
                                  ctypes.c_void_p(f.data_ptr()), len(off), ctypes.c_uint32(4096),
                                  ctypes.c_void_p(bad.data_ptr())) == 0
        torch.cuda.synchronize()
    assert bad.tolist() == [0, 0]
