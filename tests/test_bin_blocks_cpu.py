"""The degree binning's blocks cover every id once for each number of vertices that
lpa_init takes, the largest included (its rules compiled for the host)."""
import ctypes
import os
import shutil
import subprocess

import pytest

from paper_2411_19901_amd import build

SOURCE = r"""
#include "lpa_internal.h"
extern "C" int ids(int n) { return lpa::bin_ids(n); }
extern "C" int blocks(int n) { return lpa::bin_blocks(n); }
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not shutil.which(hipcc):
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("bins")
    (d / "bins.cpp").write_text(SOURCE)
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-std=c++17", "-O2", "-fPIC",
                    "-shared", f"-I{build.INCLUDE}", f"-I{build.CSRC}", str(d / "bins.cpp"), "-o",
                    str(d / "bins.so")], check=True)
    return ctypes.CDLL(str(d / "bins.so"))


@pytest.mark.parametrize("n", [1, 511, 512, 513, 1 << 18, (1 << 18) + 1, 1 << 21, (1 << 21) + 1,
                               2**31 - 4097, 2**31 - 4096, 2**31 - 4095, 2**31 - 2])
def test_blocks_cover_every_id(rules, n):
    ids, blocks = rules.ids(n), rules.blocks(n)
    assert ids % 256 == 0  # four wavefronts of whole 64-id steps
    assert (blocks - 1) * ids < n <= blocks * ids
