"""The host's proof of a fused program's bounds refuses words that would lead
a kernel out of them: a plan's words are altered in one place (on the CPU;
nothing runs) and the check is asked again."""
import ctypes
import os
import subprocess

import pytest

import paper_2006_15512_amd as W
import wmc_workloads as wl

HERE = os.path.dirname(W.LIB_PATH)
SOURCE = r"""
#include <cstring>
#include "wmc_internal.h"

// Alters the first place of the wanted kind; false: the program has none.
static bool alter(FusedProgram &F, const char *what) {
    for (size_t q = 0; q < F.chains.size(); ++q) {
        const ChainTask &t = F.chains[q];
        unsigned *w = F.words.data() + t.desc;
        const unsigned L = w[CH_STAGES], end = w[CH_TILES] + (L + 2) * w[CH_TILE_BITS];
        if (!std::strcmp(what, "none")) return true;
        if (!std::strcmp(what, "lift")) {
            w[CH_WORDS + CS_LIFT] += 200;
            return true;
        }
        if (!std::strcmp(what, "list")) {  // a copy's offsets read from words that are no list
            for (unsigned s = 0; !t.big && s < L; ++s) {
                unsigned *x = w + CH_WORDS + s * CS_WORDS + CS_X;
                const unsigned n = x[CX_BITS] - x[CX_LOW];
                for (unsigned at = CH_OUT; n && at + n <= CH_WORDS; ++at) {
                    bool zero = true;
                    for (unsigned b = 0; b < n; ++b) zero = zero && w[at + b] == 0u;
                    if (!zero) continue;
                    x[CX_LIST] = at;
                    return true;
                }
            }
            continue;
        }
        for (ChainRec &r : F.recs) {
            if (r.desc != t.desc) continue;
            unsigned words = r.words;
            if (!std::strcmp(what, "big record") && t.big)  // as many as a short chain's
                words = CH_WORDS + L * CS_WORDS + (L + 2) * w[CH_TILE_BITS];
            if (!std::strcmp(what, "short record") && !t.big) words = end;  // without the copies' lists
            if (!std::strcmp(what, "long record") && q + 1 < F.chains.size()) words = F.chains[q + 1].desc - t.desc + 4;
            if (words == r.words) continue;
            r.words = words;
            return true;
        }
    }
    return false;
}

extern "C" int altered(wmc_plan_t *plan, const char *what) {
    wmc_plan_t P = *plan;
    std::string why;
    if (!alter(P.fused, what)) return -1;
    return wmc_validate_fused(P, &why) ? 1 : 0;
}
"""


@pytest.fixture(scope="module")
def altered(tmp_path_factory):
    d = tmp_path_factory.mktemp("bounds")
    src, so = d / "altered.cpp", d / "altered.so"
    src.write_text(SOURCE)
    W.lib()
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", os.path.join(HERE, "csrc"), str(src), "-o",
                    str(so), W.LIB_PATH, "-Wl,-rpath," + HERE], check=True, timeout=300)
    fn = ctypes.CDLL(str(so)).altered
    fn.argtypes = [ctypes.c_void_p, ctypes.c_char_p]
    return lambda plan, what: fn(plan._h, what.encode())


@pytest.mark.parametrize("what,accepted", [("none", 1), ("lift", 0), ("list", 0), ("short record", 0), ("big record", 0),
                                           ("long record", 0)])
def test_altered_words_are_refused(altered, what, accepted):
    plans = [W.Plan(W.Network.from_formula(f), seed=0, block=b) for f, b in
             ((wl.banded_3cnf(60, 210, 15, seed=1), 1), (wl.banded_3cnf(110, 380, 25, seed=2), 3))]
    got = [altered(p, what) for p in plans]
    assert set(got) - {-1} == {accepted}, got
