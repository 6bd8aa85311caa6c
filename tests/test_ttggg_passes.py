"""How the 5-gluon amplitudes split a chunk of events into passes (CPU): the
rule of csrc/g3_pass.h compiled for the host."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2105_10529_amd", "csrc")
ALLOC = ctypes.CFUNCTYPE(ctypes.c_int, ctypes.c_int)


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("g3_pass")
    src, out = d / "rule.cpp", d / "rule.so"
    src.write_text('#include "g3_pass.h"\n'
                   'extern "C" int shape(long b, long r, long m) { const auto p = mf::g3::pass_shape(b, r, m);'
                   " return p.states * 64 + p.per_block; }\n"
                   'extern "C" int fitting(long b, long r, long m, int (*alloc)(int)) { mf::g3::Pass p{0, 0};'
                   " const bool ok = mf::g3::fitting_pass(b, r, m, [=](mf::g3::Pass q) { return alloc(q.states) != 0; }, p);"
                   " return ok ? p.states * 64 + p.per_block : 0; }\n")
    subprocess.check_call(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(out), str(src)])
    f = ctypes.CDLL(str(out))
    f.shape.argtypes = [ctypes.c_long] * 3
    f.fitting.argtypes = [ctypes.c_long] * 3 + [ALLOC]
    return f


def _rounds(states, per_block, blocks, resident):
    """Rounds of one state each that the launches of all 32 gluon states take."""
    return 32 // states * -(-blocks * (states // per_block) // resident) * per_block


@pytest.mark.parametrize("resident,helicities,full", [(1024, 2, 131072), (512, 1, 65536)])
def test_the_pass_takes_the_fewest_rounds_of_the_real_launches(lib, resident, helicities, full):
    """Every chunk of 1 to full / 64 blocks, in FP32 and FP64: no other pass in
    the 2 GiB buffer takes fewer rounds, and none as few with less memory."""
    for blocks in range(1, full // 64 + 1):
        most = 4 * 2 * full // (helicities * blocks * 64)
        states, per_block = divmod(lib.shape(blocks, resident, most), 64)
        assert states == 4 or states <= most
        options = [(4, 4)] + [(s, 1) for s in (4, 8, 16, 32) if s == 4 or s <= most]
        assert (states, per_block) in options
        mine = _rounds(states, per_block, blocks, resident)
        for o in options:
            r = _rounds(*o, blocks, resident)
            assert mine < r or (mine == r and states <= o[0]), (blocks, o)


@pytest.mark.parametrize("room", [0, 3, 4, 8, 15, 16, 31, 32])
@pytest.mark.parametrize("blocks", [1, 40, 200, 700, 2048])
def test_a_smaller_pass_is_taken_where_the_buffer_cannot_be_had(lib, room, blocks):
    """room: states whose buffer can be allocated.  From the preferred pass
    downwards, each size asked for at most once; refused only if not even the
    four states of the smallest pass fit, and never more than the preferred
    pass."""
    most = 4 * 131072 // (blocks * 64)
    asked = []

    def alloc(states):
        asked.append(states)
        return states <= room

    got = lib.fitting(blocks, 1024, most, ALLOC(alloc))
    assert asked[0] == lib.shape(blocks, 1024, most) // 64
    assert all(b < a for a, b in zip(asked, asked[1:]))
    if room < 4:
        assert got == 0 and asked[-1] == 4
    else:
        assert 4 <= got // 64 <= room and got // 64 == asked[-1]
