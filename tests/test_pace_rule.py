"""The host's choice between bodies of two and three launches (gbsub_pace.h,
host logic, checked on the CPU): whatever word the host sees when it queues
body t (that of the body before or of the body itself), the form depends on
the dirty counts alone, and follows the count of body t - 1, back as well as
forth."""
import ctypes
import os
import random
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_18560_amd", "csrc")
SRC = """
#include "gbsub_pace.h"
extern "C" {
uint64_t word(uint32_t f, int done, int fits, int fitted) { return gbs::pace_word(f, done, fits, fitted); }
int done(uint64_t w) { return gbs::pace_done(w); }
uint32_t finished(uint64_t w) { return gbs::pace_finished(w); }
int room(uint64_t w, uint64_t t) { return gbs::pace_room(w, t); }
int two(uint64_t w, uint64_t t, int fits0) { return gbs::pace_two(w, t, fits0); }
}
"""


@pytest.fixture(scope="module")
def pace(tmp_path_factory):
    d = tmp_path_factory.mktemp("pace")
    (d / "pace.cpp").write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, "-o", str(d / "pace.so"),
                    str(d / "pace.cpp")], check=True)
    L = ctypes.CDLL(str(d / "pace.so"))
    L.word.restype = ctypes.c_uint64
    L.word.argtypes = [ctypes.c_uint32] + [ctypes.c_int] * 3
    for name in ("done", "finished"):
        getattr(L, name).argtypes = [ctypes.c_uint64]
    L.room.argtypes = [ctypes.c_uint64, ctypes.c_uint64]
    L.two.argtypes = [ctypes.c_uint64, ctypes.c_uint64, ctypes.c_int]
    return L


def test_word_fields(pace):
    for f in (0, 1, 2, 2 ** 31 - 1):
        for done in (0, 1):
            w = pace.word(f, done, 1, 0)
            assert pace.finished(w) == f and pace.done(w) == done


@pytest.mark.parametrize("seed", range(20))
def test_form_does_not_follow_the_hosts_timing(pace, seed):
    rng = random.Random(seed)
    n = 40
    fits = [rng.random() < 0.5 for _ in range(n + 1)]        # whether body t's dirty tiles fit the budget
    # the word once f bodies have ended: 0, or the counts of bodies f and f - 1
    words = [0] + [pace.word(f, 0, fits[f], fits[f - 1]) for f in range(1, n)]
    for t in range(n - 1):
        seen = [f for f in range(t + 1) if pace.room(words[f], t)]
        assert seen == ([0] if t == 0 else [t - 1, t])       # what the host can see when it queues body t
        assert {bool(pace.two(words[f], t, fits[0])) for f in seen} == {fits[max(t - 1, 0)]}
