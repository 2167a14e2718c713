"""The kernels' LDS limit is set on every device that is used, once: an
attribute set with one device current says nothing about another. On the CPU,
with hipGetDevice and hipFuncSetAttribute answered by a small library loaded
before the runtime; the session creations end at their first device object."""

import subprocess
import sys

SHIM = r"""
static int device, calls;
int hipGetDevice(int* d) { *d = device; return 0; }
int hipFuncSetAttribute(const void* f, int attribute, int bytes) {
  calls += f && attribute == 8 && bytes > 65536;
  return 0;
}
int hipStreamCreateWithFlags(void** s, unsigned f) { return 100; }
void shim_device(int d) { device = d, calls = 0; }
int shim_calls(void) { return calls; }
"""

SCRIPT = r"""
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
from lpgen import tiny_lp
from paper_2506_17650_amd import capi
lib = capi.load()
a = capi._LPArrays(tiny_lp(seed=3))
for device in (0, 1, 0, 1, 5):
    shim.shim_device(device)
    got = []
    for precision in (0, 1):
        p = capi.opdhg_default_params(precision=precision)
        h = ctypes.c_void_p()
        rc = lib.opdhg_session_create(ctypes.byref(a.struct), ctypes.byref(p),
                                      ctypes.c_void_p(256), 1 << 40, None, ctypes.byref(h))
        assert rc == capi.OPDHG_ERR_DEVICE and not h.value
        got.append(shim.shim_calls())
    print(*got)
"""


def test_set_on_every_device_once(repo_root, tmp_path):
    (tmp_path / "shim.c").write_text(SHIM)
    shim = tmp_path / "shim.so"
    subprocess.run(["gcc", "-shared", "-fPIC", str(tmp_path / "shim.c"), "-o", str(shim)], check=True)
    out = subprocess.run([sys.executable, "-c", SCRIPT, str(shim)], cwd=repo_root,
                         capture_output=True, text=True)
    assert out.returncode == 0, out.stderr
    # FP64: k_one and both windowed kernels; then FP32's five
    assert out.stdout.split("\n")[:5] == ["3 8", "3 8", "0 0", "0 0", "3 8"]
