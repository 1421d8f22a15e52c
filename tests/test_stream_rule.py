"""Which weights the experts' forward loads nontemporally (csrc/stream_rule.h), against what the rule is for: those that one tile reads, of layers
whose active experts' weights do not fit the Infinity Cache."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_11005_amd", "csrc")
MB = 1 << 20


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("rule")
    (tmp / "rule.cpp").write_text('#include "stream_rule.h"\nextern "C" int cached(int d, int f) { return cached_experts(d, f); }\n'
                                  'extern "C" int streams(int a, int c, int rows, int tile) { return stream_weights(a, c, rows, tile); }\n')
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I" + CSRC, str(tmp / "rule.cpp"), "-o", str(tmp / "rule.so")], check=True)
    return ctypes.CDLL(str(tmp / "rule.so"))


# rows of every expert; 64 rows per tile (few rows) and 256
@pytest.mark.parametrize("tile", [64, 256])
@pytest.mark.parametrize("d,f,rows", [
    (2048, 768, [65] * 16), (2048, 768, [100] * 16), (2048, 768, [1000] + [16] * 15), (2048, 1408, [128] * 8),      # all of them fit
    (4096, 1536, [16] * 7 + [0] * 9), (4096, 1536, [100] * 4 + [0] * 12), (2880, 2880, [300] * 5 + [0] * 11),       # the active ones do
    (4096, 1536, [16] * 8), (4096, 1536, [64, 65, 256, 257, 512] + [1] * 11), (7168, 2048, [1] * 32), (4096, 14336, [2]), (2048, 768, [0] * 100 + [3] * 29)])
def test_weights_read_once_and_too_large_to_stay(rule, d, f, rows, tile):
    active = sum(n > 0 for n in rows)
    fit = active * 3 * 2 * d * f <= 256 * MB
    for n in rows:
        if n:
            assert bool(rule.streams(active, rule.cached(d, f), n, tile)) == (not fit and -(-n // tile) == 1), n
