"""The short form of the fp16 quantizer (Quantizer in rowcode.h): one fma per
value instead of the exact quotient.  quant_words_check.c proves on the CPU,
over every width, every normal scale and every fp16 value a row of
that scale can hold, that the words are the same; without the replacement of
small negative values, the same check fails."""
import os
import shutil
import subprocess

import pytest

SRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "quant_words_check.c")


@pytest.mark.skipif(shutil.which("gcc") is None, reason="needs gcc")
def test_short_quantizer_equals_the_exact_words(tmp_path):
    exe = str(tmp_path / "check")
    subprocess.run(["gcc", "-O3", "-mfma", "-mavx2", "-fopenmp", "-ffp-contract=off", "-o", exe, SRC, "-lm"], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and r.stdout.strip() == "tested 7378601806", r.stdout
    assert subprocess.run([exe, "plant"], capture_output=True, timeout=600).returncode == 1
