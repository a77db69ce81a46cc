"""What the kernels' single-precision arithmetic takes for granted of the built library, read from its own code: denormals kept,
rounding to nearest at the start of every kernel, and the change to rounding down (round_down in csrc/qflash_tile.h) ahead of what
needs it and behind what must not see it.  The compiler knows nothing of that change."""
import collections
import os
import re
import shutil
import subprocess

import pytest

from paper_2604_25306_amd import build, library_path

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
pytestmark = pytest.mark.skipif(not os.path.exists(OBJDUMP) or not os.path.exists(library_path()), reason="needs the built library and llvm-objdump")


@pytest.fixture(scope="module")
def images(tmp_path_factory):
    d = tmp_path_factory.mktemp("images")
    shutil.copy(library_path(), d / "lib.so")                 # (the parts are written beside the file)
    subprocess.check_call([OBJDUMP, "--offloading", str(d / "lib.so")], stdout=subprocess.DEVNULL)
    found = sorted(str(p) for p in d.iterdir() if p.name.endswith("gfx950"))
    assert len(found) >= 8
    return found


def test_no_option_that_changes_floats():
    flags = " ".join(build.HIPCC_FLAGS)
    for word in ("fast", "denormal", "unsafe", "finite", "ffp", "reciprocal"):
        assert word not in flags


def test_every_kernel_starts_with_denormals_and_nearest(images):
    kernels = 0
    for image in images:
        text = subprocess.check_output([OBJDUMP, "-D", "-j", ".rodata", image], text=True, stderr=subprocess.DEVNULL)
        modes = re.findall(r"\.amdhsa_float_(round|denorm)_mode_(\S+) (\d)", text)
        assert all(value == ("0" if kind == "round" else "3") for kind, _, value in modes)
        assert len(modes) == 4 * text.count("\n.amdhsa_kernel ") + (4 if text.startswith(".amdhsa_kernel ") else 0)
        kernels += len(modes) // 4
    assert kernels > 300


def test_rounding_down_ahead_of_the_floats_and_behind_the_rest(images):
    # one instruction of the float normalisation; the parts of an exact division, of the quantiser and of 64-bit divisions
    down, nearest = "v_cvt_pk_u8_f32", ("v_div_scale_f32", "v_div_fixup_f32", "v_rndne_f32", "v_trunc_f32")
    wanted = re.compile(r"^<(\S+)>:|\s(s_setreg\S*) (.*?)(?: *//|$)|\s(%s)\b" % "|".join((down,) + nearest))
    seen = collections.defaultdict(list)
    for image in images:
        with subprocess.Popen([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", image], stdout=subprocess.PIPE, text=True) as p:
            for line in p.stdout:
                m = wanted.search(line)
                if m is None:
                    continue
                if m.group(1):
                    name = m.group(1)
                elif m.group(2):
                    assert (m.group(2), m.group(3)) == ("s_setreg_imm32_b32", "hwreg(HW_REG_MODE, 0, 2), 2"), name
                    seen[name].append("mode")
                else:
                    seen[name].append(m.group(4))
        assert p.returncode == 0
    changing = {n: s for n, s in seen.items() if "mode" in s}
    assert len(changing) > 60
    for name, s in seen.items():
        if down in s:
            assert name in changing and s.index("mode") < s.index(down), name
    for name, s in changing.items():                            # (code is laid out in the order of the source here)
        last = len(s) - 1 - s[::-1].index("mode")
        assert not set(s[last:]) & set(nearest), name
