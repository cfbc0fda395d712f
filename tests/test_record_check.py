"""The records of k_fps_local (paper_2604_17720_amd/csrc/fps_record.h, compiled for the host): a chunk that holds
words of two rounds is told from a whole one by all 32 bits of its check, and the bound of the third values is
never below them, nor above the second."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2604_17720_amd", "csrc")

SOURCE = """
#include "fps_record.h"
extern "C" {
unsigned check(unsigned x, unsigned y, unsigned z, unsigned which, unsigned r) { return ffps::record_check(x, y, z, which, r); }
void words(long n, const unsigned *index, const unsigned *second, const unsigned *others, const unsigned char *picked, unsigned *word, unsigned *bound) {
    for (long i = 0; i < n; ++i) {
        word[i] = ffps::index_word(index[i], second[i], others[i], picked[i] != 0);
        bound[i] = ffps::bound_of_others(second[i], word[i]);
    }
}
unsigned tag_c() { return ffps::kTagC; }
unsigned index_mask() { return ffps::kRecordIndex; }
}
"""


@pytest.fixture(scope="module")
def rec(tmp_path_factory):
    d = tmp_path_factory.mktemp("rec")
    (d / "rec.cpp").write_text(SOURCE)
    subprocess.check_call(["g++", "-O1", "-shared", "-fPIC", "-w", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", CSRC,
                           "-o", str(d / "rec.so"), str(d / "rec.cpp")])
    return ctypes.CDLL(str(d / "rec.so"))


def test_chunks_of_two_rounds_are_told(rec):
    """Second points of a round and of two rounds later, every mixture of their four words; some coordinates are the same."""
    r = np.random.default_rng(3)
    n, tag = 20000, rec.tag_c() & 0xffffffff
    old = r.uniform(-5, 5, (n, 3)).astype(np.float32).view(np.uint32)
    new = np.where(r.random((n, 3)) < .3, old, r.uniform(-5, 5, (n, 3)).astype(np.float32).view(np.uint32))
    rounds = r.integers(3, 1000, n).astype(np.uint32)
    for i in (0, 1, 2):  # the formula below is the header's
        assert rec.check(*map(int, new[i]), tag, int(rounds[i])) & 0xffffffff == int(new[i][0] ^ new[i][1] ^ new[i][2] ^ np.uint32(tag) ^ rounds[i])
    whole = lambda p, k: np.concatenate([p, (p[:, 0] ^ p[:, 1] ^ p[:, 2] ^ np.uint32(tag) ^ k)[:, None]], 1)
    a, b = whole(old, rounds - 2), whole(new, rounds)
    for mask in range(1, 16):
        from_old = np.array([(mask >> k) & 1 for k in range(4)], bool)
        mix = np.where(from_old, a, b)
        accepted = (mix[:, 0] ^ mix[:, 1] ^ mix[:, 2] ^ mix[:, 3] ^ np.uint32(tag)) == rounds
        assert np.array_equal(mix[accepted], b[accepted]), mask  # nothing but the new chunk itself


def test_bound_of_the_third_values(rec):
    r = np.random.default_rng(5)
    n = 200000
    second = np.abs(np.concatenate([r.uniform(0, 1e6, n // 2), 10.0 ** r.uniform(-44, 38, n // 2 - 3), [0, np.inf, 3.4e38]])).astype(np.float32)
    others = (second * np.where(r.random(n) < .5, r.uniform(0, 1, n), 1 - 10.0 ** r.uniform(-8, 0, n))).astype(np.float32)
    others[~np.isfinite(others)] = 1.0
    others[: n // 10] = second[: n // 10]
    others = np.minimum(others, second)
    index = r.integers(0, 5242880, n).astype(np.uint32)
    picked = r.integers(0, 2, n).astype(np.uint8)
    word, bound = np.empty(n, np.uint32), np.empty(n, np.uint32)
    p = lambda v: v.ctypes.data_as(ctypes.c_void_p)
    rec.words(ctypes.c_long(n), p(index), p(second), p(others), p(picked), p(word), p(bound))
    assert np.array_equal(word & np.uint32(rec.index_mask()), index) and np.array_equal(word >> 31, picked)
    bound = bound.view(np.float32)
    assert (bound >= others).all() and (bound <= second).all() and np.array_equal(bound[others == second], second[others == second])
    near = (others > second * .75) & (second > 1e-30) & np.isfinite(second)
    assert near.sum() > n // 4 and (bound[near] <= others[near] * (1 + 2.0 ** -9)).all()
