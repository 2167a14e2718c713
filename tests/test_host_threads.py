"""The host's loops ask the system for its thread count once, not in every pass:
the answer takes the system microseconds under a lock, which threads that each
prepare an LP queue for. On the CPU, with the question answered and counted by
a small library loaded first."""

import subprocess
import sys

SHIM = r"""
static int calls;
unsigned answer(void) __asm__("_ZNSt6thread20hardware_concurrencyEv");
unsigned answer(void) { ++calls; return 3; }
int shim_calls(void) { return calls; }
"""

SCRIPT = r"""
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
from lpgen import tiny_lp
from paper_2506_17650_amd import capi
capi.load()
before = shim.shim_calls()
capi.opdhg_spectral_norm(tiny_lp(seed=3), capi.opdhg_vanilla_params(0.0, power_iters=200, power_tol=0.0))
print(shim.shim_calls() - before)
"""


def test_asked_once(repo_root, tmp_path):
    (tmp_path / "shim.c").write_text(SHIM)
    shim = tmp_path / "shim.so"
    subprocess.run(["gcc", "-shared", "-fPIC", str(tmp_path / "shim.c"), "-o", str(shim)], check=True)
    out = subprocess.run([sys.executable, "-c", SCRIPT, str(shim)], cwd=repo_root,
                         capture_output=True, text=True)
    assert out.returncode == 0, out.stderr
    assert int(out.stdout) == 1
