"""The generated kernels of sixteen distinct patterns, more cases than the
compiler tracks through a kernel parameter's address, compile for gfx950.  In
a process of their own: a compiler that gives up aborts."""
import subprocess
import sys

CODE = """
from exa_modeling.generators import kernel_sweep
from paper_2608_16265_amd import ExaModel
ExaModel(kernel_sweep(16, 1000).model, host_only=True).compile_check()
print("compiled")
"""


def test_kernels_of_sixteen_patterns_compile():
    r = subprocess.run([sys.executable, "-c", CODE], capture_output=True, text=True, timeout=180)
    assert r.returncode == 0 and "compiled" in r.stdout, r.stderr[-2000:]
