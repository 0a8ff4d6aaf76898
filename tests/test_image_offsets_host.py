"""The displacement that the pair kernels take of a row's entry against the one
its image code was made for, on the CPU from the kernels' own header: perfect
crystals in small cells that are not orthogonal, where every other pair of atoms
is exactly half a cell vector apart."""
import ctypes as C
import subprocess

import numpy as np
import pytest

from paper_2205_10046_amd import build
from tests.test_gpu_image_offsets import CELLS, _cell

SOURCE = r"""
#include "pair.h"
using namespace nep;
// walk[k], rows[k]: displacement of difference D[k] at the image `code` as the walk and as the builder take it
extern "C" void both(const double* H, const double* Hi, const int* pbc, int ortho, long n, const double* D, int code,
                     double* walk, double* rows) {
  StructInfo st{};
  for (int k = 0; k < 9; ++k) st.H[k] = H[k], st.Hi[k] = Hi[k];
  for (int k = 0; k < 3; ++k) st.pbc[k] = pbc[k];
  st.mode = kModeImages;
  st.ortho = ortho;
  const Frame fr(st);
  for (long k = 0; k < n; ++k, D += 3, walk += 3, rows += 3) {
    fr.displacement(D[0], D[1], D[2], (uint16_t)code, walk[0], walk[1], walk[2]);
    int n0, n1, n2, a, b, c;
    min_image(st, D[0], D[1], D[2], n0, n1, n2);
    split_code((uint16_t)code, a, b, c);
    image_disp(st, D[0], D[1], D[2], n0 + a, n1 + b, n2 + c, rows[0], rows[1], rows[2]);
  }
}
"""


@pytest.fixture(scope="module")
def both(tmp_path_factory):
    d = tmp_path_factory.mktemp("offsets")
    (d / "both.hip").write_text(SOURCE)
    subprocess.run([build.HIPCC, "--offload-host-only", "-std=c++17", "-O2", "-fPIC", "-shared", "-I" + build.CSRC,
                    "-I" + build.ROOT + "/include", str(d / "both.hip"), "-o", str(d / "both.so")], check=True,
                   capture_output=True)
    f = C.CDLL(str(d / "both.so")).both

    def call(box, pbc, D, code):
        H, Hi, D = box.reshape(9).copy(), np.linalg.inv(box).reshape(9).copy(), np.ascontiguousarray(D)
        out = np.empty_like(D), np.empty_like(D)
        ptr = [x.ctypes.data_as(C.POINTER(C.c_double)) for x in (H, Hi, D, *out)]
        f(ptr[0], ptr[1], (C.c_int * 3)(*pbc), int(np.count_nonzero(box - np.diag(np.diag(box))) == 0),
          C.c_long(len(D)), ptr[2], code, ptr[3], ptr[4])
        return out
    return call


@pytest.mark.parametrize("name", CELLS)
def test_walk_and_builder_take_the_same_image(name, both):
    halves = 0
    for origin in (0.0, 0.137, 3.3):
        for pbc in ((1, 1, 1), (1, 0, 1)):
            pos, _, box = _cell(name, origin)
            box = box.reshape(3, 3)
            D = (pos.T[None] - pos.T[:, None]).reshape(-1, 3)
            s = D @ np.linalg.inv(box)
            halves += np.count_nonzero(np.abs(np.abs(s) - 0.5) < 1e-9)
            for code in (0x888, 0x788, 0x97a):
                walk, rows = both(box, pbc, D, code)
                assert np.abs(walk - rows).max() < 1e-12
    assert halves > 100
