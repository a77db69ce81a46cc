"""Where the words that a kernel waits for first lie in its arguments: in as few lines of 64 bytes as they fit."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
FIELDS = {"QflashLaunchArgs": ("Q", "K", "V", "B", "H", "N", "n_qtiles", "n_units", "units_per_xcd", "split_qtiles_inv", "split_table_lds",
                               "hc_dev", "lut_base", "one"),
          "QflashKernelArgs": ("Q", "K", "V", "B", "H", "N", "n_qtiles", "n_units", "units_per_xcd", "split_qtiles_inv", "split_table_lds",
                               "hc_dev", "lut_base", "per_head", "hw[0]")}
CONSTANTS = {"hc_dev", "lut_base", "one", "per_head", "hw[0]"}


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
@pytest.mark.parametrize("struct", sorted(FIELDS))
def test_lines(struct, tmp_path):
    rows = "".join('    std::printf("%s %%d %%d\\n", (int)((char*)&a.%s - (char*)&a), (int)sizeof a.%s);\n' % (f, f, f) for f in FIELDS[struct])
    (tmp_path / "lines.cpp").write_text('#include <cstdio>\n#include "qflash_internal.h"\nint main() {\n    static %s a;\n%s}\n' % (struct, rows))
    exe = str(tmp_path / "lines")
    subprocess.check_call(["g++", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2604_25306_amd", "csrc"),
                           str(tmp_path / "lines.cpp"), "-o", exe])
    lines = {}
    for row in subprocess.check_output([exe], text=True).splitlines():
        name, at, size = row.split()
        lines[name] = {int(at) // 64, (int(at) + int(size) - 1) // 64}
    assert len(set().union(*(lines[f] for f in lines if f in CONSTANTS))) == 1, lines      # constants: one line
    assert set().union(*(lines[f] for f in lines if f not in CONSTANTS)) == {0, 1}, lines   # tensors, shape, unit of work: two
