"""The RMSNorm of the persistent pass down to the bits: a row's sum of squares adds up in one order, whatever instructions carry it."""
import numpy as np
import pytest

import ssd_inputs as I
from tests.gpu_util import dev_f32, dev_i32

pytestmark = pytest.mark.gpu
F32 = np.float32


def _row_scales(h, eps, nearest_first=True):
    """1/rms of the rows of h [M][d] as the pass adds it up: four features of a lane, the four lanes of a 16-feature tile, every eighth
    tile in one of eight lanes, and those; pairs of neighbours first.  (The squares of bf16 values are exact in fp32, so a fused
    multiply-add rounds as an addition does.)"""
    M, d = h.shape
    sq = (h * h).reshape(M, d // 16, 4, 4)
    s = np.zeros((M, d // 16, 4), F32)
    for i in range(4):
        s = s + sq[..., i]
    tiles = (s[..., 0] + s[..., 1]) + (s[..., 2] + s[..., 3]) if nearest_first else (s[..., 0] + s[..., 2]) + (s[..., 1] + s[..., 3])
    v = np.zeros((M, 8), F32)
    for j in range(0, d // 16, 8):
        v = v + tiles[:, j:j + 8]
    for o in ((1, 2, 4) if nearest_first else (4, 2, 1)):
        v = v + v[:, np.arange(8) ^ o]
    return (F32(1) / np.sqrt(v[:, 0] / F32(d) + F32(eps))).astype(F32)


@pytest.mark.parametrize("width", [512, 1024, 2048])
def test_row_scales_add_up_in_their_order(width):
    """Without o and down projections the residual stream is the embedding: the hidden states are its rows times 1/rms, which numpy
    follows operation by operation."""
    from paper_2603_03251_amd import binding as B
    shape = I.ModelShape(n_layers=1, d_model=width, n_q_heads=width // 64, n_kv_heads=2 if width == 512 else width // 256, head_dim=64, d_ffn=512,
                         vocab=512, dtype="bf16", rope_theta=500000.0, tie_embeddings=True)
    w = I.make_weights(shape, 3)
    for name in w:
        if name.endswith(("wo", "w_down")):
            w[name] = np.zeros_like(w[name])
    K, F, P = 5, 4, 40
    model = B.ssd_model_create(shape, w)
    ctx = B.ssd_ctx_create(model, 1, K, F, P + 2 * K + 8)
    try:
        assert B.ssd_ctx_views(ctx).fused_pass == 2
        B.ssd_ctx_fill_synthetic_kv(ctx, [P], 3)
        rng = np.random.default_rng(width)
        pending = rng.integers(0, shape.vocab, (1, K + 1))
        keys = rng.permutation(shape.vocab)[:(K + 1) * F][None]
        tokens = rng.integers(0, shape.vocab, (1, (K + 1) * F, K))
        d_keys, d_tokens, d_pending, d_temps = dev_i32(keys), dev_i32(tokens), dev_i32(pending), dev_f32(np.zeros(1))
        B.ssd_ctx_set_forced(ctx, d_keys, d_tokens)
        B.ssd_prespeculate(ctx, d_pending, d_temps, 1)
        got = {k: v.cpu().numpy() for k, v in B.read_cache(ctx).items()}
        fed = np.concatenate([keys[0][:, None], tokens[0][:, :-1]], axis=1).reshape(-1)       # row by row, step by step
        embed = w["embed"].astype(F32)
        differ = 0
        for hidden, ids in ((got["glue_hidden"].reshape(-1, width), pending[0]), (got["hidden"].reshape(-1, width), fed)):
            h = embed[ids]
            scale = _row_scales(h, shape.rms_eps)
            differ += int((scale != _row_scales(h, shape.rms_eps, nearest_first=False)).sum())
            assert np.array_equal(hidden, h * scale[:, None])
        assert differ > 0                                      # (else these rows could not tell one order from another)
    finally:
        B.ssd_ctx_destroy(ctx)
        B.ssd_model_destroy(model)
