"""Vectors of floats in rows of any width are accessed as what they are, four bytes aligned: no cast and no template's parameter makes the compiler take an address for a multiple of 16."""
import os
import re
import subprocess

import pytest

from paper_2012_15469_amd import build

pytestmark = pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="no compiler here")
FLAGS = [f for f in build.HIP_FLAGS if f != "-shared"] + ["--cuda-device-only", "-I", os.path.join(build.ROOT, "include")]


def test_the_build_refuses_a_lost_alignment():
    assert "-Werror=align-mismatch" in build.HIP_FLAGS


@pytest.mark.parametrize("src", build.LIBCADA_SRC, ids=os.path.basename)
def test_no_alignment_is_lost_in_a_call(src):
    r = subprocess.run([build.HIPCC, *FLAGS, "-Werror=align-mismatch", "-fsyntax-only", src], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout


def test_rows_in_registers_are_loaded_as_four_byte_aligned(tmp_path):
    """cada_logreg_steps.hip: the rows of X are its only global accesses of four floats at a time, with the innovations that it stores."""
    out = str(tmp_path / "steps.ll")
    src = os.path.join(build.HERE, "csrc", "cada_logreg_steps.hip")
    r = subprocess.run([build.HIPCC, *FLAGS, "-S", "-emit-llvm", "-o", out, src], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout
    aligns = re.findall(r"(?:load <4 x float>|store <4 x float> [^,]+), ptr addrspace\(1\).*?align (\d+)", open(out).read())
    assert len(aligns) > 100 and set(aligns) == {"4"}, sorted(set(aligns))
