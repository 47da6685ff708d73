"""The blocks a linear layer of a wide pass is cut into are chosen by arithmetic on its sizes alone (csrc/wide_blocks.h, plain C++):
compiled here as it stands and checked over the sizes that passes can have, among them those of the GPU tests of the blocks."""
import ctypes
import os
import subprocess

import pytest

from tests.test_gpu_prefill import BLOCK_PROMPTS, BLOCK_PROMPTS_1B, BLOCK_PROMPTS_64_HEADS, BLOCK_ROUNDS, FEW_ROW_PROMPTS, K

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2603_03251_amd", "csrc")
NWG, SLICES, ROUND_ROWS, PROMPT_ROWS = 256, 8, 384, 1024
ANY = 1 << 30                                                  # more blocks than there are


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("wide_blocks")
    src, so = d / "blocks.cpp", d / "blocks.so"
    src.write_text('#include "wide_blocks.h"\nusing namespace ssd;\n'
                   'extern "C" int choose(int tiles, int kt, int rows, int nwg, int blocks, int slices, long long room, int width) {\n'
                   '  const auto c = choose_wide_block(tiles, kt, rows, nwg, blocks < kNumWideBlocks ? blocks : kNumWideBlocks, slices, room, width);\n'
                   '  return c.block * 16 + c.S; }\n'
                   'extern "C" int few(int layer, int tiles, int kt, int rows, int nwg, int slices, long long room) {\n'
                   '  const auto c = choose_wide_few((FewLayer)layer, tiles, kt, rows, nwg, slices, room); return c.depth ? (c.mtg * 16 + c.S) * 16 + c.depth : 0; }\n'
                   'extern "C" int count(int gate_up, int head) { return head ? kNumWideBlocks : gate_up ? kGateUpBlocks : kLayerBlocks; }\n'
                   'extern "C" long long room(long long rows) { return wide_part_room(rows, %d, %d); }\n'
                   'extern "C" int tile(int i, int rows) { return rows ? kWideBlocks[i].rt : kWideBlocks[i].ft; }\n' % (ROUND_ROWS, SLICES))
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(so), str(src)], check=True)
    so = ctypes.CDLL(str(so))
    so.room.restype = ctypes.c_longlong
    return so


def _choose(lib, tiles, kt, rows, nwg, blocks, room, width):
    c = lib.choose(tiles, kt, rows, nwg, blocks, SLICES, ctypes.c_longlong(room), width)
    return c // 16, c % 16


FEW_LAYER = {"qkv": 0, "o": 1, "down": 1, "gate/up": 2}


def _few(lib, layer, tiles, kt, rows, room, nwg=NWG):
    """(row tiles of a group, slices, ring) of the kernel for few rows, or None where it is not taken."""
    c = lib.few(FEW_LAYER[layer], tiles, kt, rows, nwg, SLICES, ctypes.c_longlong(room))
    return (c // 256, c // 16 % 16, c % 16) if c else None


def _layers(width, q_heads, kv_heads, ffn):
    """(tiles, k-tiles, has slices) of the linear layers of a model."""
    return {"qkv": ((q_heads + 2 * kv_heads) * 4, width // 32, False), "o": (width // 16, q_heads * 2, True),
            "gate/up": (2 * ffn // 16, width // 32, False), "down": (width // 16, ffn // 32, True)}


def _prompt_choices(lib, model, rows, max_trunk, blocks=None):
    """What the layers of a prompt pass of one sequence take, in a context with max_trunk positions."""
    room = lib.room(ctypes.c_longlong(min(max_trunk, PROMPT_ROWS if max_trunk > ROUND_ROWS else ROUND_ROWS)))
    return {(layer,) + _choose(lib, tiles, kt, rows, NWG, blocks or lib.count(layer == "gate/up", 0), room if slices else 0, model[0])
            for layer, (tiles, kt, slices) in _layers(*model).items() if not _few(lib, layer, tiles, kt, rows, room)}


@pytest.mark.parametrize("width,ffn", [(512, 1024), (512, 8192), (1024, 4096), (2048, 8192)])
@pytest.mark.parametrize("nwg", [256, 248, 8])
def test_choices_fit_the_layer_and_its_workspace(lib, width, ffn, nwg):
    for rows in list(range(1, 400)) + [512, 513, 768, 769, 1023, 1024]:
        room = lib.room(ctypes.c_longlong(rows))
        assert room >= SLICES * min(rows, 384) and room >= rows
        for layer, (tiles, kt, slices) in _layers(width, width // 64, width // 256, ffn).items():
            blocks = lib.count(layer == "gate/up", 0)
            block, S = _choose(lib, tiles, kt, rows, nwg, blocks, room if slices else 0, width)
            assert 0 <= block < blocks and S in ((1, 2, 4, 8) if slices else (1,)), (rows, tiles, kt)
            assert kt % (2 * S) == 0 and S * rows <= max(room, rows), (rows, tiles, kt, S)
            if block == 0 and not slices:
                assert kt % 4 == 0                             # (its two groups of wavefronts)


def _fused_models():
    """Sizes of the models that fused passes take on 256 workgroups: layers of the persistent pass in one unit per workgroup, of 2, 4 or 8
    k-tiles per wavefront, o in up to two and down in up to four k-slices."""
    def cuts(groups, inputs, most):
        ks = next((k for k in (4, 2) if k <= most and groups * k <= NWG and inputs // 256 % (2 * k) == 0), 1)
        return inputs % 512 == 0 and inputs // 256 // ks in (2, 4, 8) and groups * ks <= NWG
    for width in (512, 1024, 2048):
        for q_heads in range(8, 129, 8):
            for group in (1, 2, 4, 8, 16):
                groups = (q_heads + 2 * q_heads // group) * 2
                if q_heads % group or groups > NWG or not cuts(width // 32, q_heads * 64, 2):
                    continue
                for ffn in range(512, 16385, 512):
                    if cuts(width // 32, ffn, 4):
                        yield width, q_heads, q_heads // group, ffn


def test_blocks_that_are_not_compiled_would_not_be_taken(lib):
    """Over every shape a fused pass takes: the lists that leave blocks out choose what the whole list would."""
    models = list(_fused_models())
    assert (2048, 32, 8, 8192) in models and (2048, 64, 16, 512) in models
    taken = set()
    for model in models:
        for rows in (49, 96, 150, 230, 300, 384, 385, 450, 490, 512, 640, 768, 900, 960, 1024):
            for room_rows in {rows, max(rows, 384), 1024}:
                got = _prompt_choices(lib, model, rows, room_rows)
                assert got == _prompt_choices(lib, model, rows, room_rows, 10), (model, rows)
                taken |= {(layer, block) for layer, block, _ in got}
    assert taken == {(layer, i) for layer in ("qkv", "o", "down", "gate/up") for i in range(lib.count(layer == "gate/up", 0))}


def test_few_rows_fit_the_layer_and_its_workspace(lib):
    """The kernel for few rows: its quarters of a slice are whole turns of its ring, its partial sums fit, qkv is one turn of the grid; and
    the GPU test reaches every instance that a shape takes."""
    taken, reached = set(), set()
    for model in _fused_models():
        for rows in (1, 4, 16, 17, 32, 33, 48, 49):
            room = lib.room(ctypes.c_longlong(rows))
            for layer, (tiles, kt, slices) in _layers(*model).items():
                for nwg in (NWG, 64, 8):
                    c = _few(lib, layer, tiles, kt, rows, room, nwg)
                    if c is None:
                        continue
                    mtg, S, depth = c
                    assert rows <= 48 and kt % (4 * S * depth) == 0 and S * rows <= room and (slices or S == 1), (model, rows, layer)
                    assert mtg == 1 if layer == "qkv" else mtg >= (rows + 15) // 16 and (mtg, layer) != (1, "gate/up"), (model, rows, layer)
                    assert layer != "qkv" or (tiles + 3) // 4 * ((rows + 15) // 16) <= nwg
                    if nwg == NWG:
                        taken.add((FEW_LAYER[layer], mtg, depth))
    for width, heads, kv_heads, ffn, rows in FEW_ROW_PROMPTS:
        for layer, (tiles, kt, _) in _layers(width, heads, kv_heads, ffn).items():
            c = _few(lib, layer, tiles, kt, rows, lib.room(ctypes.c_longlong(rows)))
            if c:
                reached.add((FEW_LAYER[layer], c[0], c[2]))
    assert reached == taken and len(taken) == 12


def _reached(lib):
    """(layer, block, slices) of the prompt passes that the GPU tests compare."""
    seen = set()
    for width, ffn, rows in BLOCK_PROMPTS:
        seen |= _prompt_choices(lib, (width, width // 64, 2, ffn), rows, rows + 2 * K + 8)
    for rows, trunk in BLOCK_PROMPTS_1B:
        seen |= _prompt_choices(lib, (2048, 32, 8, 8192), rows, trunk or rows + 2 * K + 8)
    for rows in BLOCK_PROMPTS_64_HEADS:
        seen |= _prompt_choices(lib, (2048, 64, 16, 512), rows, rows + 2 * K + 8)
    return seen


def test_the_gpu_tests_reach_what_the_1b_shape_takes(lib):
    """All wide passes of its layers, in contexts of every room (up to 48 rows are passes of another kind)."""
    wanted = set()
    for rows in range(49, 1025):
        for room_rows in {rows, max(rows, 300), max(rows, 384), max(rows, 385), max(rows, 512), max(rows, 700), 1024}:
            wanted |= _prompt_choices(lib, (2048, 32, 8, 8192), rows, room_rows)
    assert len(wanted) > 30 and wanted <= _reached(lib), wanted - _reached(lib)


def test_the_gpu_tests_reach_every_block(lib):
    seen = _reached(lib)
    for layers in (("qkv",), ("o", "down"), ("gate/up",)):        # (o and down share their kernels)
        assert {block for at, block, _ in seen if at in layers} == set(range(lib.count(layers[0] == "gate/up", 0))), layers
    assert {S for _, _, S in seen} == {1, 2, 4, 8}
    heads = {_choose(lib, (vocab + 63) // 64 * 4, 512 // 32, nb * 3 * F, NWG, ANY, 0, 512)[0] for vocab, nb, F in BLOCK_ROUNDS if nb * 3 * F > 96}
    assert heads == set(range(lib.count(0, 1))), heads
