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
extern "C" int row_class(int P) { return marl::row_class(P); }
extern "C" int slices(int rows, int *first, int *size)
{
    const marl::EvenParts s = marl::tall_slices(rows);
    for (int i = 0; i < s.parts; ++i) { first[i] = s.first(i); size[i] = s.size(i); }
    return s.parts;
}
extern "C" void products(int rows, int state_dim, int *tall, int *flat)
{
    const marl::MixerProducts p = marl::mixer_products(rows, state_dim);
    *tall = p.tall; *flat = p.flat;
}
// the launches of a list of products: how many each holds, their chunks and the samples of one
extern "C" int launches(int count, long transitions, int *held, int *chunks, int *samples)
{
    const marl::EvenParts l = marl::even_parts(count, marl::kProductsPerLaunch);
    for (int i = 0; i < l.parts; ++i) {
        held[i] = l.size(i);
        const marl::SampleChunks c = marl::mixer_chunks(transitions, held[i]);
        chunks[i] = c.chunks; samples[i] = c.chunk;
    }
    return l.parts;
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


def test_the_tall_products_of_a_mixer_are_of_one_row_class(rules):
    """Slices follow one another, cover the rows, and differ by one block of 16 at most; a launch takes all of them."""
    first, size = (ctypes.c_int * 64)(), (ctypes.c_int * 64)()
    for rows in range(144, 64 * 64 + 1, 16):
        n = rules.slices(rows, first, size)
        assert first[0] == 0 and all(first[i + 1] == first[i] + size[i] for i in range(n - 1)) and 16 * (first[n - 1] + size[n - 1]) == rows
        assert max(size[:n]) - min(size[:n]) <= 1 and 16 * max(size[:n]) <= 384
        assert len({rules.row_class(16 * k) for k in size[:n]}) == 1, (rows, size[:n])
        assert n <= -(-rows // 384) + 1


def test_no_launch_of_the_mixers_products_leaves_half_the_chip_idle(rules):
    """As long as there are transitions to cut: 256 compute units, chunks of 64 transitions at least."""
    tall, flat = ctypes.c_int(), ctypes.c_int()
    held, chunks, samples = ((ctypes.c_int * 64)() for _ in range(3))
    counts = set()
    for N in range(1, 65):
        for M in (16, 32, 64):
            for S in (1, 48, 128, 129, 320, 321, 512, 641, 1024):
                rules.products(N * M, S, ctypes.byref(tall), ctypes.byref(flat))
                counts |= {tall.value, flat.value}
    assert {1, 2, 5, 7, 17, 24} <= counts
    for count in sorted(counts - {0}):
        for R in list(range(1, 3000, 37)) + [1025, 1089, 3265, 5441, 6400, 12800, 16385, 25600]:
            n = rules.launches(count, ctypes.c_long(R), held, chunks, samples)
            assert sum(held[:n]) == count and max(held[:n]) <= 16 and max(held[:n]) - min(held[:n]) <= 1
            for i in range(n):
                assert (chunks[i] - 1) * samples[i] < R <= chunks[i] * samples[i] and samples[i] % 64 == 0
                assert held[i] * chunks[i] <= 256
                assert held[i] * chunks[i] >= 128 or samples[i] == 64, (count, R, held[i], chunks[i])
