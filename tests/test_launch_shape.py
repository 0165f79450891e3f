"""CPU checks of the draw kernels' launch arithmetic (csrc/launch_shape.h, plain C++): compiled here with the host compiler
and gone through for every size, since a wrong share or a load past a row shows in no result that a small launch gives."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1409_5402_amd", "csrc")

SHIM = r"""
#include "launch_shape.h"
using namespace same;
extern "C" {
int t_block_len(int K) { return block_len(K); }
int t_blocks_in_use(int K) { return blocks_in_use(K); }
int t_blocks_fill_row(int K) { return blocks_fill_row(K); }
int t_scan_first_topic(int hl, int T, int nblk) { return scan_first_topic(hl, T, nblk); }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    where = tmp_path_factory.mktemp("launch_shape")
    src, so = where / "shim.cpp", where / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-I", CSRC,
                    str(src), "-o", str(so)], check=True)
    return ctypes.CDLL(str(so))


def test_scan_stays_inside_the_row(lib):
    """Loads without bounds: every lane's block lies inside the row for every number of topics that takes them, and the
    blocks in use are each some lane's."""
    unguarded = 0
    for K in range(4, 2049, 4):
        if not lib.t_blocks_fill_row(K):
            continue
        unguarded += 1
        T, nblk = lib.t_block_len(K), lib.t_blocks_in_use(K)
        first = [lib.t_scan_first_topic(hl, T, nblk) for hl in range(32)]
        assert max(first) + T <= K, (K, T, nblk)
        assert first[:nblk] == [T * l for l in range(nblk)], K
    assert unguarded > 100
