"""What the gradient by pairs of words reserves for the largest mini-batch, against what any mini-batch up to it can need: the
functions of kernels.h compiled for the host, with the lengths of center words that make the most of each.  No GPU needed."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

from helpers import ROUNDS_CASE, rounds_stream
from paper_2211_10280_amd import build

SHIM = """
#include "kernels.h"
extern "C" {
int64_t rare(int64_t V, int tasks, int64_t n) { return tn_group_rare(V, tasks, n); }
int64_t chunk(int64_t V, int tasks, int64_t n) { return tn_group_chunk(tasks, n); }
int64_t frequent(int64_t V, int tasks, int64_t n) { return tn_group_frequent(V, tasks, n); }
int64_t chunks(int64_t V, int tasks, int64_t n) { return tn_group_chunks(V, tasks, n); }
int64_t slices(int64_t V, int tasks, int64_t n) { return tn_group_slices(V, tn_group_frequent(V, tasks, n)); }
int64_t max_vocab(int64_t, int, int64_t) { return TN_GROUP_MAX_VOCAB; }
}
"""


@pytest.fixture(scope="module")
def sizes(tmp_path_factory):
    d = tmp_path_factory.mktemp("group_sizes")
    (d / "shim.hip").write_text(SHIM)
    subprocess.check_call(["hipcc", "--cuda-host-only", "-O1", "-std=c++17", "-shared", "-fPIC", "-I" + build.CSRC, str(d / "shim.hip"),
                           "-o", str(d / "shim.so")])
    lib = C.CDLL(str(d / "shim.so"))
    for name in ("rare", "chunk", "frequent", "chunks", "slices", "max_vocab"):
        f = getattr(lib, name)
        f.restype, f.argtypes = C.c_int64, [C.c_int64, C.c_int, C.c_int64]
    return lib


def most_needed(V, n, rare, chunk):
    """(frequent center words, chunks) of n positions at their most: so many center words just frequent, and what is left over
    spent on one position more than a multiple of the chunk, word by word."""
    words = np.arange(1, min(V, n // (rare + 1)) + 1, dtype=np.int64)
    if len(words) == 0:
        return 0, 0
    base = -(-(rare + 1) // chunk)                 # chunks of a word that is just frequent, positions to its next one
    step = base * chunk + 1 - (rare + 1)
    left = n - words * (rare + 1)
    more = np.where(left >= words * step, words + (left - words * step) // chunk, left // step)
    return len(words), int((words * base + more).max())


@pytest.mark.parametrize("tasks", [128, 130, 192, 256, 258, 320, 480, 510, 512])
def test_every_mini_batch_fits_what_the_largest_reserves(sizes, tasks):
    limit = (2 ** 31 - 2) // (tasks + 1)           # occurrences and centers together fit 31 bits
    most = 65535 // tasks
    edges = [2048 * k + d for k in (1, 16, 32, 33, 64, 65, most - 1, most, most + 1) for d in (-1, 0, 1, 71)]
    sweep = np.unique(np.concatenate([np.geomspace(64, limit, 150).astype(np.int64), edges, [262_144, 262_214, 524_285, 524_288, limit]]))
    for V in (1, 4, 8, 16, 20, 50, 64, 65, 100, 200, 500, 1_000, 2_000, 5_000, 10_000, sizes.max_vocab(0, 0, 0)):
        worst = [0, 0, 0]
        for n in (int(n) for n in sweep if n <= limit):
            rare, chunk = sizes.rare(V, tasks, n), sizes.chunk(V, tasks, n)
            assert rare * tasks <= 65535 and chunk * tasks <= 65535                  # counts of 16 bits
            need = (*most_needed(V, n, rare, chunk), sizes.slices(V, tasks, n))
            worst = [max(a, b) for a, b in zip(worst, need)]
            room = [sizes.frequent(V, tasks, n), sizes.chunks(V, tasks, n), sizes.slices(V, tasks, n)]
            assert all(a <= b for a, b in zip(worst, room)), (V, tasks, n, "needed", worst, "reserved", room)
            assert worst[1] <= 65535                                                 # a chunk's number, 16 bits in the counting


def test_the_stream_of_many_frequent_words_takes_a_second_round(sizes):
    V, w, N, n, begin = ROUNDS_CASE
    tasks = 2 * w * (N + 1)
    positions = np.bincount(rounds_stream()[0][begin:begin + n], minlength=V)
    rare, slices = sizes.rare(V, tasks, n), sizes.slices(V, tasks, n)
    frequent = int((positions > rare).sum())
    assert {rare, rare + 1} <= set(positions.tolist())
    assert 16 * slices < frequent < 2 * 16 * slices and frequent % 16
