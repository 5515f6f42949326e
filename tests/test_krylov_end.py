"""How a Krylov launch learns that a vector's iteration has ended (host side,
csrc/krylov_end.h).  One block of the ending launch writes the flag while other
wavefronts of the same launch may read it before or after: whichever value they
see, they have to go the same way, and later launches have to stand down."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2104_05829_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include "krylov_end.h"
using namespace semx;
int main()
{
    const KrylovLaunch jacobi[] = {kEndOperator, kEndUpdate, kEndDecide};
    const KrylovLaunch fcg[] = {kEndUpdate, kEndDecide, kEndDirection};
    const KrylovLaunch coarse[] = {kEndUpdate};
    const struct { const KrylovLaunch *l; int n; } seq[] = {{jacobi, 3}, {fcg, 3}, {coarse, 1}};
    const int from[] = {1, 500, 1 << 28, 357913930, 715827870, 2147483600};
    long checked = 0;
    for (auto &q : seq)
        for (int first : from)
            for (int it = first; it < first + 40; ++it)
                for (int k = 0; k < q.n; ++k) {
                    const int own = end_stamp(it, q.l[k]);
                    if (own == 0 || own == 1) return std::printf("stamp %d\n", own), 1;
                    // the launch that ends the iteration: flag 0 before the write, own after
                    if (ended_before(0, own) || ended_before(own, own)) return std::printf("torn it=%d k=%d\n", it, k), 1;
                    if (!ended_before(1, own)) return std::printf("start it=%d k=%d\n", it, k), 1;
                    // every launch enqueued behind it stands down
                    for (int jt = it; jt < first + 40; ++jt)
                        for (int m = jt == it ? k + 1 : 0; m < q.n; ++m, ++checked)
                            if (!ended_before(own, end_stamp(jt, q.l[m])))
                                return std::printf("late it=%d k=%d jt=%d m=%d\n", it, k, jt, m), 1;
                }
    std::printf("ok %ld\n", checked);
    return 0;
}
"""


def test_every_reader_of_a_launch_agrees(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not found")
    src, exe = tmp_path / "end.cpp", str(tmp_path / "end")
    src.write_text(DRIVER)
    res = subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-fsanitize=undefined",
                          "-fno-sanitize-recover=all", "-I", CSRC, str(src), "-o", exe],
                         capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr[-4000:]
    res = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0 and res.stdout.startswith("ok "), res.stdout + res.stderr


def _kernels(text):
    """(name, body) of the kernels, and of the decision that one of them includes."""
    for m in re.finditer(r"^([A-Za-z_][^;{}]*?)\n\{\n(.*?)^\}\n", text, re.S | re.M):
        name = re.search(r"\b(\w+(?:_kernel|_direction))\(", m.group(1))
        if name:
            yield name.group(1), m.group(2)


def test_writers_of_the_flag_test_their_own_stamp():
    """No device function both writes the flag and leaves on its bare value
    (fin_init_kernel writes it without a test: it starts the iteration)."""
    writers = []
    for f in ("solve.hip", "ax_impl.h"):
        with open(os.path.join(CSRC, f)) as fh:
            for name, body in _kernels(fh.read()):
                if re.search(r"->done\s*=[^=]", body) and name != "fin_init_kernel":
                    writers.append(name)
                    assert "ended_before(" in body, name
                    assert not re.search(r"if \((sc->)?done\)", body), name
    assert {"coarse_step_kernel", "pcg_direction", "pcg_update_few_kernel", "pcg_update_fused_kernel",
            "fcg_update_fused_kernel", "fcg_p_fused_kernel", "fin_conv_kernel",
            "pcg_decide_kernel"} <= set(writers), writers
    with open(os.path.join(CSRC, "ax_impl.h")) as fh:
        column = dict(_kernels(fh.read()))["ax_kernel"]
    assert "dirn ? !ended_before(" in column  # the operator that decides reads the flag by wavefront
