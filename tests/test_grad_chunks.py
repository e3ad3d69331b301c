"""The backward pass's division of samples into chunks (csrc/grad_chunks.h, host arithmetic): whichever way the slots
are walked, every sample lies in one chunk and the workspace has room for the partial sums.  No GPU is used."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = """
#include "grad_chunks.h"
extern "C" void cut(int planes, long rows, int T, long *o)
{
    const marl::GradChunks g = marl::grad_chunks(planes, rows, T);
    const marl::SampleChunks *parts[3] = {&g.whole, &g.late, &g.early};
    for (int i = 0; i < 3; ++i) { o[3 * i] = parts[i]->samples; o[3 * i + 1] = parts[i]->chunk; o[3 * i + 2] = parts[i]->chunks; }
    o[9] = g.t_mid; o[10] = g.room; o[11] = marl::kForkSlots;
    const marl::SampleChunks *gru[3] = {&g.gru_whole, &g.gru_late, &g.gru_early};
    for (int i = 0; i < 3; ++i) { o[12 + 3 * i] = gru[i]->samples; o[13 + 3 * i] = gru[i]->chunk; o[14 + 3 * i] = gru[i]->chunks; }
}
"""


@pytest.fixture(scope="module")
def cut(tmp_path_factory):
    d = tmp_path_factory.mktemp("chunks")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-I", os.path.join(ROOT, "paper_2205_05248_amd", "csrc"),
                           str(d / "shim.cpp"), "-o", str(d / "shim.so")])
    lib, out = ctypes.CDLL(str(d / "shim.so")), (ctypes.c_long * 21)()

    def call(planes, rows, T):
        lib.cut(planes, ctypes.c_long(rows), T, out)
        return [tuple(out[3 * i:3 * i + 3]) for i in range(3)], out[9], out[10], out[11]

    def call_gru(rows, T):
        lib.cut(1, ctypes.c_long(rows), T, out)
        return [tuple(out[12 + 3 * i:15 + 3 * i]) for i in range(3)], out[9], out[10], out[11]
    call.gru = call_gru
    return call


# Every row count up to 130 and beyond that odd and even ones up to more rows than the second stream is used for, with
# every slot count from the fewest that are walked in two launches (odd ones: halves of different size) to 200.
ROWS = list(range(1, 131)) + [135, 160, 185, 257, 305, 500, 777, 1024, 2048, 3071, 4099]


@pytest.mark.parametrize("planes", [1, 2])
def test_partial_sums_of_either_walk_fit_the_workspace(cut, planes):
    for rows in ROWS:
        for T in [1, 2, 15] + list(range(16, 201)):
            (whole, late, early), t_mid, room, fork_slots = cut(planes, rows, T)
            walks = [[(rows * T, whole)]]
            if planes == 1 and T >= fork_slots:
                assert 0 < t_mid < T
                walks.append([(rows * (T - t_mid), late), (rows * t_mid, early)])
            for walk in walks:
                for expected, (samples, chunk, chunks) in walk:
                    assert samples == expected and chunk % 64 == 0 and (chunks - 1) * chunk < samples <= chunks * chunk
                needed = sum(-(-samples // chunk) for _, (samples, chunk, _) in walk)
                assert needed <= room, (planes, rows, T, needed, room)
            assert room <= 256


# The same of the two GRU products of 128 units, one plane, which have chunks of their own: a partial result of either is 384 x 144
# numbers, and the workspace has `room` of each, beside those of the other two products.  Few slots, which are walked in one launch
# only, with every sample count around those where the other products' chunks grow from 64 samples to 128.
FEW_SLOTS = [(rows, T) for T in range(1, 16) for rows in range(2500 // T, 8300 // T + 2)]


@pytest.mark.parametrize("shapes", [[(rows, T) for rows in ROWS for T in range(1, 201)], FEW_SLOTS], ids=["rows", "few slots"])
def test_partial_sums_of_the_gru_products_fit_the_workspace(cut, shapes):
    for rows, T in shapes:
        (whole, late, early), t_mid, room, fork_slots = cut.gru(rows, T)
        walks = [[(rows * T, whole)]]
        if T >= fork_slots:
            walks.append([(rows * (T - t_mid), late), (rows * t_mid, early)])
        for walk in walks:
            for expected, (samples, chunk, chunks) in walk:
                assert samples == expected and chunk % 64 == 0 and (chunks - 1) * chunk < samples <= chunks * chunk
            bytes_of_a_chunk = 384 * 144 * 4
            needed = sum(-(-samples // chunk) for _, (samples, chunk, _) in walk) * bytes_of_a_chunk
            assert needed <= room * bytes_of_a_chunk, (rows, T, needed, room)


def test_few_samples_of_a_one_plane_network_are_cut_into_short_chunks(cut):
    """Up to 2560 samples a chunk's own steps are what takes time: none is longer than 64; beyond, none is shorter than 128."""
    for M in list(range(1, 4500, 7)) + [2560, 2561, 8192, 32768]:
        whole = cut(1, M, 1)[0][0]
        assert whole[1] == 64 if M <= 2560 else whole[1] >= 128
