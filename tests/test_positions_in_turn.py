"""How attention's positions are dealt to a head's blocks and their waves (fkv_internal.h), compiled for the host: every position to one
wave and lane, and the last one -- the open page, whose wave has the new token to take in as well -- to a wave that has no more pages than
any other of its block."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_13109_amd", "csrc")


@pytest.fixture(scope="module")
def position(tmp_path_factory):
    d = tmp_path_factory.mktemp("positions")
    (d / "p.cpp").write_text('#include "fkv_internal.h"\n'
                             'extern "C" void positions(int n_att, int n_splits, int n_waves, int* out) {\n'
                             '  for (int s = 0; s < n_splits; ++s) for (int w = 0; w < n_waves; ++w) for (int l = 0; l < 64; ++l)\n'
                             '    *out++ = fkv::nth_position(s + fkv::nth_of_wave(w, l, n_waves) * n_splits, n_att);\n}\n')
    lib = str(d / "p.so")
    subprocess.run(["g++", "-std=c++17", "-w", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", f"-I{CSRC}", str(d / "p.cpp"), "-o", lib,
                    "-L/opt/rocm/lib", "-lamdhip64"], check=True)
    L = C.CDLL(lib)

    def run(n_att, n_splits, n_waves=8):
        out = np.empty((n_splits, n_waves, 64), dtype=np.int32)
        L.positions(n_att, n_splits, n_waves, out.ctypes.data_as(C.c_void_p))
        return out

    return run


@pytest.mark.parametrize("n_att", [1, 2, 8, 9, 16, 17, 33, 65, 129, 257, 511, 512])
@pytest.mark.parametrize("n_splits", [1, 2, 3, 7, 8, 12, 17, 32, 63])
def test_every_position_once_and_the_open_page_where_least_is_to_do(position, n_att, n_splits):
    p = position(n_att, n_splits)
    there = p < n_att
    assert (p >= 0).all() and sorted(p[there]) == list(range(n_att))
    pages = there.sum(axis=2)
    assert (there == (np.arange(64) < pages[:, :, None])).all() or n_att < 8 * n_splits      # (a wave's lanes from the first on)
    split, wave, lane = np.argwhere(p == n_att - 1)[0]
    assert (split, lane) == (0, 0) and pages[split, wave] == max(1, pages[split].min())
    assert pages.sum(axis=1).max() - pages.sum(axis=1).min() <= 1
