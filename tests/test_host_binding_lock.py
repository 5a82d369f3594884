"""The native call path gives Python's lock back while it calls the library: the module is loaded in a child process
on top of a stand-in for libbmx.so whose entry points ask whether the calling thread holds the lock (and launch
nothing).  Held through a launch that waits for room in a queue, the lock would stop every other Python thread, and
with a host callback on the stream that needs it the wait would never end."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

STAND_IN = """#include <stddef.h>
#include <stdint.h>
extern "C" {
int PyGILState_Check(void);
int calls, held;
static int asked() { ++calls; held += PyGILState_Check(); return 0; }
size_t bmx_workspace_bytes(int, const int64_t*, int) { asked(); return 512; }
int64_t bmx_conv_weight_row_words(int, int, int) { return 2; }
#define ENTRY(name) int name() { return asked(); }
ENTRY(bmx_binarize_pack) ENTRY(bmx_unpack_pm1) ENTRY(bmx_xnor_gemm) ENTRY(bmx_xnor_gemm_count) ENTRY(bmx_widen_words32)
ENTRY(bmx_binary_fc_static) ENTRY(bmx_binary_fc_packed) ENTRY(bmx_pack_conv_weights) ENTRY(bmx_pack_nchw)
ENTRY(bmx_binary_conv2d_packed) ENTRY(bmx_alpha_mean_abs)
// these ask for a workspace on the first of two calls
#define LAZY(name) int name() { static int n; asked(); return n++ % 2 ? 0 : -6; }
LAZY(bmx_lazy_binary_fc) LAZY(bmx_lazy_binary_conv2d) LAZY(bmx_lazy_xnor_gemm_w32) LAZY(bmx_lazy_binary_conv2d_bits)
LAZY(bmx_lazy_quant_gemm)
}
"""

CHILD = """
import ctypes, sys
import torch
stand_in = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
from paper_1705_09864_amd import _bmx_host as h
h.set_error(RuntimeError)
f32 = lambda *s: torch.zeros(s, device="cuda")
u64 = lambda *s: torch.zeros(s, dtype=torch.int64, device="cuda")
i32 = lambda *s: torch.zeros(s, dtype=torch.int32, device="cuda")
x, w, X, W, img, pimg, n = f32(4, 64), u64(8, 1), u64(4, 1), u64(8, 2), f32(2, 64, 6, 6), u64(2, 8, 8, 1), None
CALLS = [("binarize_pack", x, 1, n, n), ("unpack_pm1", X, 64, n, n), ("xnor_gemm", X, w, 64, n, n, False),
         ("xnor_gemm", X, w, 64, n, n, True), ("widen_words32", i32(4, 2), 64, n, n),
         ("xnor_gemm_w32", i32(4, 2), i32(8, 2), 64, n, n, n), ("binary_fc", x, w, n, False, n, n, n),
         ("binary_fc_static", x, w, n, False, f32(4, 8), n), ("binary_fc_packed", X, 64, w, n, "f32", n, n, n),
         ("pack_conv_weights", f32(8, 64, 1, 1), n), ("binary_conv2d", img, W, 8, 3, 3, 1, 1, n, False, n, n, n),
         ("pack_nchw", img, 1, n, n), ("binary_conv2d_packed", pimg, 64, W, 8, 3, 3, 1, 1, n, False, n, n),
         ("binary_conv2d_bits", pimg, 64, W, 8, 3, 3, 1, 1, n, n, 1, n, n, n),
         ("quant_gemm", x, f32(8, 64), 2, 1, True, True, n, n, n, n), ("alpha_mean_abs", f32(8, 64), n)]
calls, held = ctypes.c_int.in_dll(stand_in, "calls"), ctypes.c_int.in_dll(stand_in, "held")
for name, *args in CALLS:
    calls.value = held.value = 0
    getattr(h, name)(*args)
    print(name, calls.value, held.value, flush=True)
"""


def test_library_calls_run_without_pythons_lock(tmp_path):
    (tmp_path / "stand_in.cpp").write_text(STAND_IN)
    so = str(tmp_path / "stand_in.so")
    subprocess.run(["g++", "-shared", "-fPIC", "-O1", str(tmp_path / "stand_in.cpp"), "-o", so], check=True)
    r = subprocess.run([sys.executable, "-c", CHILD, so, ROOT], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    seen = [line.split() for line in r.stdout.splitlines()]
    assert len(seen) == 16, r.stdout
    lazy = {"xnor_gemm_w32", "binary_fc", "binary_conv2d", "binary_conv2d_bits", "quant_gemm"}
    for name, calls, held in seen:
        assert int(calls) == (3 if name in lazy else 1), (name, calls)  # with a workspace: call, size, call
        assert int(held) == 0, name
