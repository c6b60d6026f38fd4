"""Every address that the staging of unit-weight rows can form lies in the
buffer it reads.

A range of a streamed graph (LPA_STREAM_CSR) is read through a column pointer
moved back by the range's first position, so a position outside of the range's
entries lies outside of its buffer; a lane without entries (an inactive vertex,
or none) has no position of its own.  The kernels' own position rules
(lpa_internal.h) are compiled for the host here and run over wavefronts of rows
of the ranges that lpa_init cuts, with any subset of them active.
"""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2411_19901_amd import build, inputs

SOURCE = r"""
#include "lpa_internal.h"

// Lowest and highest position that staging the rows [beg, beg + len) of a
// wavefront reads; the step widths are those of staged_rows.
template <class Pos>
static void span(const Pos *beg_, const int *len, Pos *lo, Pos *hi) {
  using namespace lpa;
  int longest = 0, filled = -1;
  for (int l = kWave - 1; l >= 0; --l) {
    longest = len[l] > longest ? len[l] : longest;
    if (len[l] > 0) filled = l;
  }
  if (longest == 0) return;
  for (int r = 0; r < kWave; ++r) {
    const Pos beg = staged_begin(beg_[r], len[r], beg_[filled]);
    for (int t0 = 0; t0 < longest;) {
      const int left = longest - t0, width = left <= 4 ? 4 : left <= 8 ? 8 : 16;
      for (int j = 0; j < width; ++j) {
        const Pos at = staged_position<Pos>(beg, len[r], t0 + j);
        if (at < *lo) *lo = at;
        if (at > *hi) *hi = at;
      }
      t0 += width;
    }
  }
}

extern "C" void span32(const int *beg, const int *len, int *lo, int *hi) { span(beg, len, lo, hi); }
extern "C" void span64(const long long *beg, const int *len, long long *lo, long long *hi) {
  span(beg, len, lo, hi);
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not shutil.which(hipcc):
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("positions")
    (d / "span.cpp").write_text(SOURCE)
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-std=c++17", "-O2", "-fPIC",
                    "-shared", f"-I{build.INCLUDE}", f"-I{build.CSRC}", str(d / "span.cpp"), "-o",
                    str(d / "span.so")], check=True)
    return ctypes.CDLL(str(d / "span.so"))


def ranges(rp, chunk_kib):
    """The id ranges of a streamed graph: rows of at most chunk_kib KiB of
    columns, or one longer row."""
    v0, n, chunk = 0, len(rp) - 1, chunk_kib * 256
    while v0 < n:
        v1 = max(v0 + 1, int(np.searchsorted(rp, rp[v0] + chunk, side="right")) - 1)
        yield v0, v1
        v0 = v1


def star(n):
    rp = np.zeros(n + 1, np.int64)
    rp[1:] = n - 1 + np.arange(n)
    return rp


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("split", [0, 64])  # rows whole, or cut into segments of 64
@pytest.mark.parametrize("graph,chunk_kib", [("sbm", 1), ("sbm", 16), ("star", 1), ("rmat", 4)])
def test_positions_lie_in_the_range(rules, graph, chunk_kib, split, wide):
    rp = {"sbm": lambda: inputs.sbm1(1).row_ptr, "star": lambda: star(5000),
          "rmat": lambda: inputs.rmat(12).row_ptr}[graph]().astype(np.int64)
    rng = np.random.default_rng(1)
    dt, ct, fn = ((np.int64, ctypes.c_int64, rules.span64) if wide
                  else (np.int32, ctypes.c_int32, rules.span32))
    count = 0
    for v0, v1 in ranges(rp, chunk_kib):
        count += 1
        beg, length = rp[v0:v1], np.diff(rp[v0:v1 + 1])
        keep = length > 0
        beg, length = beg[keep], length[keep]
        if split:
            parts = -(-length // split)
            q = np.concatenate([np.arange(p) for p in parts]) if len(parts) else parts
            beg, length = np.repeat(beg, parts) + q * split, np.repeat(length, parts)
            length = np.minimum(split, length - q * split)
        order = np.argsort(-length, kind="stable")
        for share in (0.02, 0.5, 1.0):
            for u in range(0, len(order), 64):
                rows = order[u:u + 64]
                active = rng.random(len(rows)) < share
                b, n = np.zeros(64, dt), np.zeros(64, np.int32)
                b[:len(rows)] = np.where(active, beg[rows], 0)
                n[:len(rows)] = np.where(active, length[rows], 0)
                lo, hi = ct(int(rp[v1])), ct(int(rp[v0]) - 1)
                fn(b.ctypes.data_as(ctypes.c_void_p), n.ctypes.data_as(ctypes.c_void_p),
                   ctypes.byref(lo), ctypes.byref(hi))
                assert lo.value >= rp[v0] and hi.value < rp[v1], (v0, v1, lo.value, hi.value)
    assert count > 4 or graph == "star"
