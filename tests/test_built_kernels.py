"""What the built library holds (host side: the names in its symbol table)."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2104_05829_amd", "libsem.so")


def test_spread_operator_only_at_orders_that_take_it():
    """The spread form of the operator serves N <= 11; kernels beyond would
    never be launched."""
    nm = shutil.which("nm") or "/opt/rocm/llvm/bin/llvm-nm"
    if not os.path.exists(LIB) or not os.path.exists(nm):
        pytest.skip("library not built, or no nm")
    out = subprocess.run([nm, LIB], capture_output=True, text=True, timeout=120).stdout
    orders = {int(m) for m in re.findall(r"ax_split_kernelILi(\d+)E", out)}
    if not orders:
        pytest.skip("stripped library")
    assert max(orders) <= 12, sorted(orders)
