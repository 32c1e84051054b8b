"""The binding's native calls (csrc/anszp_torch.cpp) without a GPU: what they do beside calling the library, which a stand-in takes the
place of."""
import os
import shutil
import subprocess
import sys

import pytest

from paper_2406_06237_amd import build as libbuild

STAND_IN = r"""
#include <stdint.h>
extern "C" {
int PyGILState_Check(void);
static int held = 0, calls = 0;
static int look(void) { held += PyGILState_Check(); ++calls; return 0; }
int anszp_dequant_zp(...) { return look(); }
int anszp_build_tables_device(...) { return look(); }
int anszp_pack_set_device(const void*, void*) { return look(); }
int anszp_pack_bound(uint64_t n, int, int, uint32_t chunk, uint64_t* chunks, uint64_t* words) { *chunks = (n + chunk - 1) / chunk; *words = n; return 0; }
uint64_t anszp_pack_scratch_bytes(uint32_t, int) { return 64; }
int anszp_calls_seen(void) { return calls * 100 + held; }
}
"""

CALLS = r"""
import ctypes, sys
sys.path.insert(0, sys.argv[1])
import torch
import _anszp_torch as N
seen = ctypes.CDLL(sys.argv[1] + "/libanszp.so").anszp_calls_seen
bytes_, ints = torch.zeros(64, dtype=torch.uint8), torch.zeros(256, dtype=torch.int32)
assert N.dequant_zp(bytes_, 3, 0.5, 1, 0, None, 0).shape == (64,)
assert N.build_tables_device(ints, 1, 4, 128, None, 0).shape == (128,)
assert len(N.pack_set(bytes_, ints, [30, 34], 16, 4, 8, 0, 0, 0, 0, 0, False, 0)) == 5
assert seen() == 300, seen()
"""


def test_the_interpreter_lock_is_free_while_the_library_is_called(tmp_path):
    """A launch waits where a queue is full; every Python thread would wait with it."""
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    (tmp_path / "stand_in.cpp").write_text(STAND_IN)
    subprocess.check_call(["g++", "-O1", "-fPIC", "-shared", "-o", str(tmp_path / "libanszp.so"), str(tmp_path / "stand_in.cpp")])
    shutil.copy(libbuild.HOST_LIB, tmp_path)
    r = subprocess.run([sys.executable, "-c", CALLS, str(tmp_path)], capture_output=True, text=True, timeout=300, cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    assert r.returncode == 0, r.stderr[-2000:]


def test_without_them_the_binding_takes_its_own_path(monkeypatch):
    """Not built, or built against another torch: the calls answer None once and for all, with a warning, and raise nothing."""
    from paper_2406_06237_amd import binding as B
    monkeypatch.setattr(B, "_host", None)
    monkeypatch.setitem(sys.modules, "paper_2406_06237_amd._anszp_torch", None)
    monkeypatch.delattr("paper_2406_06237_amd._anszp_torch", raising=False)
    with pytest.warns(UserWarning, match="native calls"):
        assert B._call("anszp_dequant_zp", "dequant_zp", "cuda:0") is None
    for name in ("build_tables_device", "pack_set"):
        assert B._call("", name, "cuda:0") is None
