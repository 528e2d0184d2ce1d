"""Byte formulas of the kernels that close and sort an interval."""
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402


def test_close_reads_a_bit_per_particle_and_a_count_per_chunk():
    assert bench.algorithmic_bytes("close", 8192, 100, 8, 0) == 1024 + 4 * 8
    assert bench.algorithmic_bytes("close", 8193, 100, 4, 0) == 8193 / 8 + 4 * 9


def test_permutation_and_streaming():
    assert bench.algorithmic_bytes("perm", 1000, 100, 8, 0) == 16000
    assert bench.algorithmic_bytes("stream", 1000, 10, 8, 100) == 900 * 81 + 80
