"""Every generated amplitude header is the generator's text and is used (CPU)."""
import os
import re
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2105_10529_amd", "csrc")
sys.path.insert(0, os.path.join(ROOT, "paper_2105_10529_amd", "gen"))
import gen_me  # noqa: E402


def test_generated_headers_are_current_and_used():
    made = gen_me.headers()
    assert sorted(os.listdir(os.path.join(CSRC, "gen"))) == sorted(made)
    code = ""
    for f in os.listdir(CSRC):
        if f.endswith((".h", ".hip")):
            with open(os.path.join(CSRC, f)) as fh:
                code += fh.read()
    for name, text in made.items():
        with open(os.path.join(CSRC, "gen", name)) as fh:
            assert fh.read() == text, name
        assert f'#include "gen/{name}"' in code, name
        for fn in re.findall(r"__device__ __forceinline__ \w+(?:<\w+>)? (\w+)\(", text):
            assert re.search(rf"\b{fn}\b", code), (name, fn)
