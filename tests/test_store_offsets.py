"""Where the reverse recurrence's buffer stores go (csrc/store_offsets.h, host arithmetic): up to the largest gradient that is
accepted, a row or slot that exists is stored at its own place, and one that does not is dropped, that is, its offset is beyond
the array.  No GPU is used."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = """
#include "store_offsets.h"
extern "C" int in_range(long B, long N, long T, long H) { return marl::gradient_in_range(B, N, T, H); }
extern "C" unsigned store_offset(unsigned lane_at, unsigned slot_at, int exists) { return marl::store_offset(lane_at, slot_at, exists != 0); }
extern "C" unsigned descriptor_bytes(unsigned long bytes, int exists) { return marl::descriptor_bytes(bytes, exists != 0); }
extern "C" unsigned past() { return marl::kPast; }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("offsets")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-I", os.path.join(ROOT, "paper_2205_05248_amd", "csrc"),
                           str(d / "shim.cpp"), "-o", str(d / "shim.so")])
    so = ctypes.CDLL(str(d / "shim.so"))
    so.store_offset.restype = so.descriptor_bytes.restype = so.past.restype = ctypes.c_uint
    so.descriptor_bytes.argtypes = [ctypes.c_ulong, ctypes.c_int]
    so.in_range.argtypes = [ctypes.c_long] * 4
    so.store_offset.argtypes = [ctypes.c_uint, ctypes.c_uint, ctypes.c_int]
    return so


def most_slots(lib, B, N, H):
    """The most slots that are accepted."""
    low, high = 1, 1 << 30
    while low + 1 < high:
        mid = (low + high) // 2
        low, high = (mid, high) if lib.in_range(B, N, mid, H) else (low, mid)
    return low


# (episodes, agents): one row, rows that are and are not whole tiles of eight, the most rows that tiles of eight are taken for
BATCHES = [(1, 1), (1, 5), (8, 1), (100, 1), (409, 5), (2047, 1), (256, 8), (3, 11)]


@pytest.mark.parametrize("planes,hidden", [(1, 64), (2, 64), (1, 128)])
def test_stores_of_what_does_not_exist_are_dropped(lib, planes, hidden):
    element = 2 if planes == 1 else 4
    for B, N in BATCHES:
        most = most_slots(lib, B, N, hidden)
        assert lib.in_range(B, N, most, hidden) and not lib.in_range(B, N, most + 1, hidden)
        for T in {1, 2, 1100, min(most, 420000), most - 1, most}:
            if T > most:
                continue
            samples = B * N * T
            half = (1 << 31) // (4 * hidden * element * N)         # where a long episode's adjoints pass 2^31 bytes
            slots = [t for t in sorted({0, 1, T // 2, T - 1, half - 1, half, half + 1}) if 0 <= t < T]
            # the gates' adjoints: 4 H a sample, 16 bytes a lane
            row, slot = 4 * hidden * element, N * 4 * hidden * element
            assert lib.descriptor_bytes(samples * row, 1) == samples * row
            for b, n in {(0, 0), (0, N - 1), (B // 2, 0), (B - 1, N - 1)}:
                for piece in (0, row // 16 - 1):
                    lane = (b * T * N + n) * row + 16 * piece
                    for t in slots:
                        at = ((b * T + t) * N + n) * row + 16 * piece
                        assert lib.store_offset(lane, t * slot, 1) == at and at + 16 <= samples * row, (B, N, T, t)
                        # a row past the last one: two planes, on the first one's place behind a descriptor of its own; one, kPast
                        size, part = (lib.descriptor_bytes(samples * row, 0), 16 * piece) if planes == 2 else (samples * row, lib.past())
                        assert lib.store_offset(part, t * slot, 1) >= size and part + t * slot < 1 << 32, (B, N, T, t)
                    # the step before the first: slot T
                    assert lib.store_offset(lane, (T * slot) & 0xFFFFFFFF, 0) >= samples * row, (B, N, T)
            # the arrays in whose stores kPast takes the lane's place; a slot's part is added, by the kernel or by the hardware
            arrays = [hidden, 16, 64] + ([4 * hidden] if planes == 1 else [])
            for per_sample in arrays:
                size, slot_part = samples * per_sample * element, (T - 1) * N * per_sample * element
                assert lib.past() >= size and lib.past() + slot_part < 1 << 32, (B, N, T, per_sample)
