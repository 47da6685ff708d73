"""The fp32 LM head takes the final norm along where that was measured to pay, by arithmetic on the sizes alone (csrc/f32_head.h, plain
C++): compiled here as it stands and held against the measurements."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2603_03251_amd", "csrc")
# width, vocabulary, rows, us of an extend of one layer on an MI355X with a norm of its own, with the norm in the head
MEASURED = [(256, 1024, 1, 27.3, 25.1), (256, 1024, 10, 30.9, 28.9), (256, 1024, 96, 39.2, 37.2), (256, 8192, 8, 33.0, 31.5),
            (256, 8192, 24, 37.6, 36.1), (256, 8192, 96, 56.8, 59.5), (256, 8192, 384, 143.5, 159.8), (256, 32000, 48, 75.1, 80.4),
            (256, 32000, 96, 117.2, 132.5), (256, 32000, 384, 371.8, 440.0), (512, 1024, 48, 40.4, 38.3), (512, 8192, 8, 38.9, 37.3),
            (512, 8192, 16, 40.6, 38.7), (512, 8192, 384, 212.0, 229.2), (512, 32000, 1, 47.3, 50.3), (512, 32000, 8, 52.6, 56.0),
            (512, 32000, 48, 113.0, 119.5), (512, 32000, 384, 664.7, 731.2), (1024, 1024, 8, 33.0, 30.8), (1024, 1024, 48, 48.5, 46.3),
            (1024, 1024, 96, 61.2, 59.1), (1024, 8192, 96, 117.8, 122.8), (1024, 8192, 384, 385.7, 408.0), (1024, 32000, 1, 62.1, 70.5),
            (1024, 32000, 8, 66.4, 75.5), (1024, 32000, 96, 339.4, 360.2), (2048, 1024, 8, 39.3, 37.5), (2048, 1024, 48, 66.4, 64.3), (2048, 1024, 96, 94.2, 92.1),
            (2048, 8192, 8, 55.5, 57.6), (2048, 8192, 16, 64.9, 63.0), (2048, 8192, 96, 216.6, 224.2), (2048, 32000, 1, 115.7, 137.0), (2048, 32000, 8, 120.4, 142.8),
            (2048, 32000, 384, 2673.0, 2741.0), (4096, 1024, 4, 49.3, 47.3), (4096, 8192, 8, 87.7, 95.0), (4096, 32000, 1, 228.9, 284.0),
            (4096, 32000, 384, 7011.0, 7455.0)]


@pytest.fixture(scope="module")
def takes_norm(tmp_path_factory):
    d = tmp_path_factory.mktemp("f32_head")
    src, so = d / "head.cpp", d / "head.so"
    src.write_text('#include "f32_head.h"\nextern "C" int takes_norm(int rows, int vocab, int d) { return ssd::f32_head_takes_norm(rows, vocab, d); }\n')
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(so), str(src)], check=True)
    return ctypes.CDLL(str(so)).takes_norm


def test_the_head_takes_the_faster_form_where_they_differ(takes_norm):
    for width, vocab, rows, apart, together in MEASURED:
        assert abs(apart / together - 1) > 0.02
        assert bool(takes_norm(rows, vocab, width)) == (together < apart), (width, vocab, rows)


def test_small_heads_and_the_largest_passes(takes_norm):
    assert not takes_norm(1, 15, 64) and takes_norm(1, 16, 64)
    assert not takes_norm(1 << 20, 128256, 8192)               # (no overflow on the way)
