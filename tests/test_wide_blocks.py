"""The blocks a linear layer of a wide pass is cut into are chosen by arithmetic on its sizes alone (csrc/wide_blocks.h, plain C++):
compiled here as it stands and checked over the sizes that passes can have, among them those of the GPU test of the blocks."""
import ctypes
import os
import subprocess

import pytest

from tests.test_gpu_prefill import BLOCK_PROMPTS, BLOCK_ROUNDS

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2603_03251_amd", "csrc")
NWG, SLICES = 256, 8


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("wide_blocks")
    src, so = d / "blocks.cpp", d / "blocks.so"
    src.write_text('#include "wide_blocks.h"\n'
                   'extern "C" int choose(int tiles, int kt, int rows, int nwg, int blocks, int slices, long long room, int width) {\n'
                   '  const auto c = ssd::choose_wide_block(tiles, kt, rows, nwg, blocks, slices, room, width); return c.block * 16 + c.S; }\n'
                   'extern "C" int count() { return ssd::kNumWideBlocks; }\n'
                   'extern "C" int tile(int i, int rows) { return rows ? ssd::kWideBlocks[i].rt : ssd::kWideBlocks[i].ft; }\n')
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(so), str(src)], check=True)
    return ctypes.CDLL(str(so))


def _choose(lib, tiles, kt, rows, nwg, head, room, width):
    c = lib.choose(tiles, kt, rows, nwg, lib.count() - (0 if head else 1), SLICES, ctypes.c_longlong(room), width)
    return c // 16, c % 16


@pytest.mark.parametrize("width,ffn", [(512, 1024), (512, 8192), (1024, 4096), (2048, 8192)])
@pytest.mark.parametrize("nwg", [256, 248, 8])
def test_choices_fit_the_layer_and_its_workspace(lib, width, ffn, nwg):
    for rows in list(range(1, 400)) + [512, 513, 768, 769, 1023, 1024]:
        room = max(8 * 384, 4 * 1024 if rows > 384 else 0)
        for tiles, kt, slices in ((width * 3 // 2 // 16, width // 32, False), (width // 16, width // 32, True), (2 * ffn // 16, width // 32, False),
                                  (width // 16, ffn // 32, True)):
            block, S = _choose(lib, tiles, kt, rows, nwg, False, room if slices else 0, width)
            assert 0 <= block < lib.count() - 1 and S in ((1, 2, 4, 8) if slices else (1,)), (rows, tiles, kt)
            assert kt % (2 * S) == 0 and S * rows <= max(room, rows), (rows, tiles, kt, S)
            if block == 0 and not slices:
                assert kt % 4 == 0                             # (its two groups of wavefronts)


def test_the_gpu_test_reaches_every_block(lib):
    seen = set()
    for width, ffn, rows in BLOCK_PROMPTS:
        seen.add(_choose(lib, 2 * ffn // 16, width // 32, rows, NWG, False, 0, width)[0])
    assert seen == set(range(lib.count() - 1)), seen
    heads = {_choose(lib, (vocab + 63) // 64 * 4, 512 // 32, nb * 3 * F, NWG, True, 0, 512)[0] for vocab, nb, F in BLOCK_ROUNDS}
    assert lib.count() - 1 in heads and len(heads) >= 4, heads
