"""The host's rules for the weight-gradient products (csrc/grad_chunks.h).  No GPU is used."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = """
#include "grad_chunks.h"
extern "C" int kernel_for(int planes, int a_bf16, int b_bf16, int P, int columns)
{
    return marl::has_product_kernel(planes, a_bf16 != 0, b_bf16 != 0, P, columns);
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("products")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-I", os.path.join(ROOT, "paper_2205_05248_amd", "csrc"),
                           str(d / "shim.cpp"), "-o", str(d / "shim.so")])
    return ctypes.CDLL(str(d / "shim.so"))


@pytest.mark.parametrize("P,columns,fits", [(1, 16, True), (128, 336, True), (128, 352, False), (129, 144, True), (129, 160, False),
                                            (256, 144, True), (257, 144, True), (384, 144, True), (385, 144, False)])
def test_a_product_is_taken_only_with_the_elements_its_kernel_reads(rules, P, columns, fits):
    """Two planes read fp32 adjoints and fp32 states; one plane bf16 adjoints, and bf16 activations from 129 rows on."""
    for planes in (1, 2):
        for a_bf16 in (0, 1):
            for b_bf16 in (0, 1):
                elements = a_bf16 == (planes == 1) and not (b_bf16 and (planes == 2 or P <= 128))
                assert bool(rules.kernel_for(planes, a_bf16, b_bf16, P, columns)) == (fits and elements), (planes, a_bf16, b_bf16)
