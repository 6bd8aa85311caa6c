"""How the 5-gluon amplitudes split a chunk of events into passes (CPU): the
rule of csrc/g3_pass.h compiled for the host."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2105_10529_amd", "csrc")


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("g3_pass")
    src, lib = d / "rule.cpp", d / "rule.so"
    src.write_text('#include "g3_pass.h"\n'
                   'extern "C" int shape(long b, long r, long m) { const auto p = mf::g3::pass_shape(b, r, m);'
                   " return p.states * 64 + p.per_block; }\n")
    subprocess.check_call(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(lib), str(src)])
    f = ctypes.CDLL(str(lib)).shape
    f.argtypes = [ctypes.c_long] * 3
    return lambda *a: divmod(f(*a), 64)


def _rounds(states, per_block, blocks, resident):
    """Rounds of one state each that the launches of all 32 gluon states take."""
    return 32 // states * -(-blocks * (states // per_block) // resident) * per_block


@pytest.mark.parametrize("resident,helicities,full", [(1024, 2, 131072), (512, 1, 65536)])
def test_the_pass_takes_the_fewest_rounds_of_the_real_launches(rule, resident, helicities, full):
    """Every chunk of 1 to full / 64 blocks, in FP32 and FP64: no other pass in
    the 2 GiB buffer takes fewer rounds, and none as few with less memory."""
    for blocks in range(1, full // 64 + 1):
        most = 4 * 2 * full // (helicities * blocks * 64)
        states, per_block = rule(blocks, resident, most)
        assert states == 4 or states <= most
        options = [(4, 4)] + [(s, 1) for s in (4, 8, 16, 32) if s == 4 or s <= most]
        assert (states, per_block) in options
        mine = _rounds(states, per_block, blocks, resident)
        for o in options:
            r = _rounds(*o, blocks, resident)
            assert mine < r or (mine == r and states <= o[0]), (blocks, o)
