"""How the workgroups of a run share a list over the dies (gd_share.hpp),
compiled on the host: whatever the number of workgroups, every entry is taken
by exactly one of them."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = """
#include "gd_share.hpp"
extern "C" void takes(int64_t nb, int32_t nl, int32_t* count)
{
    for (int64_t id = 0; id < nb; ++id) {
        const gd::ListShare s = gd::list_share(id, nb, nl);
        for (int32_t t = s.first; t < s.end; t += s.step) ++count[t];
    }
}
"""


@pytest.fixture(scope="module")
def takes(tmp_path_factory):
    d = tmp_path_factory.mktemp("share")
    (d / "share.cpp").write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2609_35967_amd", "csrc"), str(d / "share.cpp"), "-o", str(d / "share.so")],
                   check=True)
    fn = ctypes.CDLL(str(d / "share.so")).takes
    fn.argtypes = [ctypes.c_int64, ctypes.c_int32, ctypes.c_void_p]
    return fn


@pytest.mark.parametrize("nb", [*range(1, 26), 255, 256, 257, 65536])
def test_every_entry_once(takes, nb):
    for nl in (0, 1, 5, 7, 8, 9, 63, 64, 300, 1024, 1793, 7169):
        count = np.zeros(nl + 64, np.int32)
        takes(nb, nl, count.ctypes.data)
        assert (count[:nl] == 1).all() and not count[nl:].any(), (nb, nl)
