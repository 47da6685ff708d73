"""Prompts prefilled in wide passes (many tokens of a sequence per pass) against the same prompts prefilled in chunks of K+1
tokens through narrow passes, and against the float64 oracle.  Sizes: one token, one chunk, the edges of what a pass takes of a
sequence, several passes, several short prompts in one pass."""
import numpy as np
import pytest
import torch

import ssd_inputs as I
from oracle import ssd_oracle as O
from tests.gpu_util import TOL_BF16_OWN_PREFILL, TOL_WIDE_BF16, dev_f32, dev_i32, row_rel_err

pytestmark = pytest.mark.gpu

SHAPE = I.ModelShape(n_layers=2, d_model=512, n_q_heads=8, n_kv_heads=2, head_dim=64, d_ffn=1024, vocab=4112, dtype="bf16",
                     rope_theta=500000.0, tie_embeddings=True)
K, F = 3, 2


@pytest.fixture(scope="module")
def B():
    from paper_2603_03251_amd import binding
    return binding


def _trunk(B, ctx, lens, max_trunk, shape=SHAPE):
    """Keys and values of the verified positions, [layer][sequence] arrays [len][Hkv][64]."""
    v = B.ssd_ctx_views(ctx)
    T, hkv = (max_trunk + 63) // 64 * 64, shape.n_kv_heads
    ks, vs = [], []
    for l in range(shape.n_layers):
        k = B.device_copy(v.h_trunk_k[l], (len(lens), hkv, T, 64), torch.bfloat16).float().cpu().numpy()
        vt = B.device_copy(v.h_trunk_v[l], (len(lens), hkv, T // 32, 64, 32), torch.bfloat16).float().cpu().numpy()
        vt = vt.transpose(0, 1, 2, 4, 3).reshape(len(lens), hkv, T, 64)
        ks.append([k[b, :, :n].transpose(1, 0, 2) for b, n in enumerate(lens)])
        vs.append([vt[b, :, :n].transpose(1, 0, 2) for b, n in enumerate(lens)])
    return ks, vs


@pytest.mark.parametrize("lens", [[1], [6], [64], [65], [144], [145], [191], [192], [193], [384], [385], [700], [129, 130], [40, 300, 7], [33] * 15],
                         ids=lambda x: "-".join(map(str, x[:3])) + ("x%d" % len(x) if len(x) > 3 else ""))
def test_wide_prefill_equals_narrow_chunks(B, lens):
    nb, max_trunk, seed = len(lens), max(lens) + 2 * K + 8, 7 + sum(lens)
    print(f"[case] prefill of {lens}", flush=True)
    model = B.ssd_model_create(SHAPE, I.make_weights(SHAPE, 11))
    prompt = dev_i32(I.make_prompt(SHAPE, nb, max(lens), seed))
    pending, temps = dev_i32(I.make_pending(SHAPE, nb, K, seed)), dev_f32(np.zeros(nb))
    ctxs = [B.ssd_ctx_create(model, nb, K, F, max_trunk, flags) for flags in (0, B.SSD_CTX_NARROW_PASSES)]
    try:
        assert all(B.ssd_ctx_views(c).fused_pass for c in ctxs)
        got = []
        for ctx in ctxs:
            B.ssd_ctx_prefill(ctx, prompt, lens)
            kv = _trunk(B, ctx, lens, max_trunk)
            B.ssd_prespeculate(ctx, pending, temps, 1)
            got.append((kv, B.read_cache(ctx)["glue_logits"].cpu().numpy()))
        # each side is within TOL_BF16_OWN_PREFILL of the exact keys, values and logits
        for part in (0, 1):
            for l in range(SHAPE.n_layers):
                for b in range(nb):
                    assert row_rel_err(got[0][0][part][l][b], got[1][0][part][l][b]) < 2 * TOL_BF16_OWN_PREFILL, (part, l, b)
        assert row_rel_err(got[0][1], got[1][1]) < 2 * TOL_BF16_OWN_PREFILL
        assert max(lens) <= K + 1 or not np.array_equal(got[0][1], got[1][1])      # (the prompts did go through another pass)
        # one slot prefilled alone gives what it gets beside the others
        b = nb - 1
        B.ssd_ctx_prefill_sequence(ctxs[0], b, prompt[b, :lens[b]].contiguous())
        again = _trunk(B, ctxs[0], lens, max_trunk)
        for part in (0, 1):
            for l in range(SHAPE.n_layers):
                assert row_rel_err(again[part][l][b], got[0][0][part][l][b]) < 2 * TOL_BF16_OWN_PREFILL
    finally:
        for ctx in ctxs:
            B.ssd_ctx_destroy(ctx)
        B.ssd_model_destroy(model)


@pytest.mark.parametrize("width,lens", [(1024, [512]), (1024, [513]), (512, [896]), (1024, [897]), (512, [1024]), (1024, [1025]),
                                        (512, [1409]), (512, [1124]), (1024, [1168]), (1024, [500, 512, 30])], ids=lambda x: str(x) if isinstance(x, int) else "-".join(map(str, x)))
@pytest.mark.parametrize("paged", [False, True])
def test_prompt_passes_at_the_edges_of_their_row_groups(B, width, lens, paged):
    """Passes of 385 to 1024 rows: whole groups of 8 row tiles, one row more, the most a pass takes and what is left behind it (1 row;
    100, 144, whose keys the units stage beside stored ones; 385), the row count from which o and down have room for fewer slices (512 | 513), a pass of two sequences."""
    print(f"[case] width {width}, prefill of {lens}, paged {paged}", flush=True)
    nb, max_trunk, seed = len(lens), max(lens) + 2 * K + 8, 3 + sum(lens)
    shape = I.ModelShape(n_layers=2, d_model=width, n_q_heads=width // 64, n_kv_heads=width // 256, head_dim=64, d_ffn=2 * width, vocab=4112,
                         dtype="bf16", rope_theta=500000.0, tie_embeddings=True)
    model = B.ssd_model_create(shape, I.make_weights(shape, 17))
    prompt = dev_i32(I.make_prompt(shape, nb, max(lens), seed))
    pending, temps = dev_i32(I.make_pending(shape, nb, K, seed)), dev_f32(np.zeros(nb))
    pages = 1 + nb * ((max_trunk + 63) // 64 * 2) if paged else 0
    ctxs = [B.ssd_ctx_create(model, nb, K, F, max_trunk, flags, n) for flags, n in ((0, pages), (B.SSD_CTX_NARROW_PASSES, 0))]
    try:
        assert all(B.ssd_ctx_views(c).fused_pass for c in ctxs)
        got = []
        for ctx in ctxs:
            B.ssd_ctx_prefill(ctx, prompt, lens)
            kv = None if paged else _trunk(B, ctx, lens, max_trunk, shape)
            B.ssd_prespeculate(ctx, pending, temps, 1)
            torch.cuda.synchronize()
            B.ssd_ctx_status(ctx)
            got.append((kv, B.read_cache(ctx)["glue_logits"].cpu().numpy()))
        # each side is within TOL_BF16_OWN_PREFILL of the exact keys, values and logits
        for part in (0, 1) if not paged else ():
            for l in range(shape.n_layers):
                for b in range(nb):
                    assert row_rel_err(got[0][0][part][l][b], got[1][0][part][l][b]) < 2 * TOL_BF16_OWN_PREFILL, (part, l, b)
        assert row_rel_err(got[0][1], got[1][1]) < 2 * TOL_BF16_OWN_PREFILL
        assert not np.array_equal(got[0][1], got[1][1])
    finally:
        for ctx in ctxs:
            B.ssd_ctx_destroy(ctx)
        B.ssd_model_destroy(model)


@pytest.mark.parametrize("lens,pages", [([340, 10, 10], 13), ([250, 1, 1, 1], 11), ([500, 300], 26), ([470, 510], 31), ([190, 180, 10, 12], 14),
                                        ([60] * 6 + [20], 13), ([130, 130, 100, 90], 17)],
                         ids=lambda x: "-".join(map(str, x[:4])) if isinstance(x, list) else str(x))
def test_unequal_prompts_take_no_pages_for_rows_that_only_pad(B, lens, pages):
    """Prompts of different lengths in a pool that holds them and no more: rows that pad a large pass to its longest prompt are not
    stored (attention units that append themselves, up to 144 rows per sequence, and the pass that appends first)."""
    print(f"[case] prefill of {lens} in {pages} pages", flush=True)
    nb, max_trunk, seed = len(lens), max(lens) + 2 * K + 8, 13 + sum(lens)
    assert pages == sum((n + 31) // 32 for n in lens)
    model = B.ssd_model_create(SHAPE, I.make_weights(SHAPE, 11))
    prompt, last = dev_i32(I.make_prompt(SHAPE, nb, max(lens), seed)), dev_i32(np.arange(nb).reshape(nb, 1))
    ctxs = [B.ssd_ctx_create(model, nb, K, F, max_trunk, flags, n) for flags, n in ((0, 1 + pages), (B.SSD_CTX_NARROW_PASSES, 0), (0, 0))]
    try:
        assert all(B.ssd_ctx_views(c).fused_pass for c in ctxs)
        got = []
        for ctx in ctxs:
            B.ssd_ctx_prefill(ctx, prompt, lens)
            z = torch.zeros((nb, 1, SHAPE.vocab), dtype=torch.float32, device="cuda")
            B.ssd_ctx_extend(ctx, last, 0, z)
            torch.cuda.synchronize()
            B.ssd_ctx_status(ctx)
            got.append(z.cpu().numpy())
        assert B.ssd_ctx_kv_pages(ctxs[0]) == (1 + pages, 0)
        assert np.array_equal(got[0], got[2])                  # the same passes as over a contiguous trunk
        assert row_rel_err(got[0], got[1]) < 2 * TOL_BF16_OWN_PREFILL
    finally:
        for ctx in ctxs:
            B.ssd_ctx_destroy(ctx)
        B.ssd_model_destroy(model)


@pytest.mark.parametrize("lens", [[1], [K], [K + 1], [K + 1, 1], [2, K, 1]], ids=lambda x: "-".join(map(str, x)))
def test_prompts_of_one_chunk_take_the_narrow_pass(B, lens):
    """Where the rounds are narrow passes and a chunk of K+1 tokens holds the prompts, the prefill is that one narrow pass, to
    the bit: for the whole batch and for a slot of its own."""
    nb, max_trunk, seed = len(lens), 2 * K + 12, 9 + sum(lens)
    print(f"[case] prefill of {lens}", flush=True)
    model = B.ssd_model_create(SHAPE, I.make_weights(SHAPE, 13))
    prompt = dev_i32(I.make_prompt(SHAPE, nb, max(lens), seed))
    ctxs = [B.ssd_ctx_create(model, nb, K, F, max_trunk, flags) for flags in (0, B.SSD_CTX_NARROW_PASSES)]
    try:
        assert all(B.ssd_ctx_views(c).fused_pass for c in ctxs)
        for alone in (False, True):
            got = []
            for ctx in ctxs:
                if alone:
                    B.ssd_ctx_prefill_sequence(ctx, nb - 1, prompt[nb - 1, :lens[-1]].contiguous())
                else:
                    B.ssd_ctx_prefill(ctx, prompt, lens)
                got.append(_trunk(B, ctx, lens, max_trunk))
            for part in (0, 1):
                for l in range(SHAPE.n_layers):
                    for b in range(nb):
                        assert np.array_equal(got[0][part][l][b], got[1][part][l][b]), (alone, part, l, b)
    finally:
        for ctx in ctxs:
            B.ssd_ctx_destroy(ctx)
        B.ssd_model_destroy(model)


@pytest.mark.parametrize("pages", [0, 16])
def test_wide_prefill_against_the_oracle(B, pages):
    lens, max_trunk, seed = [210, 60], 240, 5
    w = I.make_weights(SHAPE, seed)
    om = O.Model.from_weights(SHAPE, w)
    model = B.ssd_model_create(SHAPE, w)
    prompt = I.make_prompt(SHAPE, 2, max(lens), seed)
    pending = I.make_pending(SHAPE, 2, K, seed)
    ctx = B.ssd_ctx_create(model, 2, K, F, max_trunk, 0, pages)
    try:
        assert B.ssd_ctx_views(ctx).fused_pass
        B.ssd_ctx_prefill(ctx, dev_i32(prompt), lens)
        B.ssd_prespeculate(ctx, dev_i32(pending), dev_f32(np.zeros(2)), 1)
        got = B.read_cache(ctx)["glue_logits"].cpu().numpy()
        for b, n in enumerate(lens):
            _, trunk = O.prefill(om, prompt[b, :n])
            want, _, _ = O.glue_extend(om, trunk, pending[b])
            err = row_rel_err(got[b], want)
            print(f"[parity] prefill of {n} tokens, glue logits {err:.2e}", flush=True)
            assert err < TOL_BF16_OWN_PREFILL
    finally:
        B.ssd_ctx_destroy(ctx)
        B.ssd_model_destroy(model)


@pytest.mark.parametrize("heads,lens", [(16, [384]), (16, [340, 1]), (32, [770]), (32, [90] * 4)])
def test_wide_attention_units_of_two_and_three_query_tiles(B, heads, lens):
    """8 KV heads and groups of 2 and 4: 384 and 768 query tiles per pass, more than there are compute units, so that a unit
    takes two or three of them (the last unit of a head an incomplete set); appended prompts and, 90 rows of 4 sequences,
    their last chunk.  Against the narrow passes, whose units take one tile each."""
    shape = I.ModelShape(n_layers=2, d_model=512, n_q_heads=heads, n_kv_heads=8, head_dim=64, d_ffn=1024, vocab=2064, dtype="bf16",
                         rope_theta=500000.0, tie_embeddings=True)
    nb, seed = len(lens), 3 + heads
    print(f"[case] prefill of {lens} with {heads} query heads", flush=True)
    model = B.ssd_model_create(shape, I.make_weights(shape, 12))
    prompt = dev_i32(I.make_prompt(shape, nb, max(lens), seed))
    pending, temps = dev_i32(I.make_pending(shape, nb, K, seed)), dev_f32(np.zeros(nb))
    ctxs = [B.ssd_ctx_create(model, nb, K, F, max(lens) + 2 * K + 8, flags) for flags in (0, B.SSD_CTX_NARROW_PASSES)]
    try:
        assert all(B.ssd_ctx_views(c).fused_pass for c in ctxs)
        got = []
        for ctx in ctxs:
            B.ssd_ctx_prefill(ctx, prompt, lens)
            B.ssd_prespeculate(ctx, pending, temps, 1)
            got.append(B.read_cache(ctx)["glue_logits"].cpu().numpy())
        # each side is within TOL_BF16_OWN_PREFILL of the exact logits
        assert row_rel_err(got[0], got[1]) < 2 * TOL_BF16_OWN_PREFILL
    finally:
        for ctx in ctxs:
            B.ssd_ctx_destroy(ctx)
        B.ssd_model_destroy(model)


@pytest.mark.parametrize("pages", [0, 420])
@pytest.mark.parametrize("kv_heads,lens", [(1, [6000]), (2, [4100, 2500]), (1, [4500])])
def test_appended_prompts_with_key_splits(B, kv_heads, lens, pages):
    """8 query heads on one or two KV heads: some 190 query tiles per pass of up to 384 tokens, which from about 3500 stored
    keys on run as units of two or three tiles with the keys in two to four splits.  The last splits hold no keys for the first tiles of a pass, and a merge
    launch follows.  Keys, values and glue logits against the narrow passes' chunks of K+1 tokens."""
    shape = I.ModelShape(n_layers=2, d_model=512, n_q_heads=8, n_kv_heads=kv_heads, head_dim=64, d_ffn=1024, vocab=2064,
                         dtype="bf16", rope_theta=500000.0, tie_embeddings=True)
    nb, seed, max_trunk = len(lens), 5 + kv_heads, max(lens) + 2 * K + 8
    print(f"[case] prefill of {lens}, {kv_heads} KV heads, {pages} pages", flush=True)
    model = B.ssd_model_create(shape, I.make_weights(shape, 14))
    prompt = dev_i32(I.make_prompt(shape, nb, max(lens), seed))
    pending, temps = dev_i32(I.make_pending(shape, nb, K, seed)), dev_f32(np.zeros(nb))
    ctxs = [B.ssd_ctx_create(model, nb, K, F, max_trunk, flags, pages) for flags in (0, B.SSD_CTX_NARROW_PASSES)]
    try:
        assert all(B.ssd_ctx_views(c).fused_pass for c in ctxs)
        got, kv = [], []
        for ctx in ctxs:
            B.ssd_ctx_prefill(ctx, prompt, lens)
            if not pages:
                kv.append(_trunk(B, ctx, lens, max_trunk, shape))
            B.ssd_prespeculate(ctx, pending, temps, 1)
            got.append(B.read_cache(ctx)["glue_logits"].cpu().numpy())
        for part in (0, 1) if kv else ():
            for l in range(shape.n_layers):
                for b in range(nb):
                    e = row_rel_err(kv[0][part][l][b], kv[1][part][l][b])
                    assert e < 2 * TOL_BF16_OWN_PREFILL, (part, l, b, e)
        e = row_rel_err(got[0], got[1])
        print(f"[splits] glue logits {e:.2e}", flush=True)
        assert e < 2 * TOL_BF16_OWN_PREFILL
    finally:
        for ctx in ctxs:
            B.ssd_ctx_destroy(ctx)
        B.ssd_model_destroy(model)


@pytest.mark.parametrize("pages", [0, 700])
@pytest.mark.parametrize("lens", [[6000, 3500, 6000, 100], [700] * 4, [3000] * 3])
def test_wide_rounds_over_long_trunks(B, lens, pages):
    """24 branch rows of 3 or 4 sequences, 8 KV heads: 144 and 192 query tiles.  Over a short trunk a unit takes one of them;
    over thousands of keys units of two (3000) and three (6000) with the keys split are the shorter ones.  Against the narrow
    passes."""
    shape = I.ModelShape(n_layers=2, d_model=512, n_q_heads=32, n_kv_heads=8, head_dim=64, d_ffn=1024, vocab=2064, dtype="bf16",
                         rope_theta=500000.0, tie_embeddings=True)
    nb, k5, f4, seed = len(lens), 5, 4, 15
    print(f"[case] wide rounds over {lens} keys, {pages} pages", flush=True)
    model = B.ssd_model_create(shape, I.make_weights(shape, seed))
    pending, temps = dev_i32(I.make_pending(shape, nb, k5, seed)), dev_f32(np.zeros(nb))
    keys = dev_i32(np.arange(nb * 24).reshape(nb, 6, 4))
    toks = dev_i32(I.make_prompt(shape, nb * 24, k5, seed).reshape(nb, 6, 4, k5))
    got = []
    try:
        for flags in (0, B.SSD_CTX_NARROW_PASSES):
            ctx = B.ssd_ctx_create(model, nb, k5, f4, max(lens) + 2 * k5 + 8, flags, pages)
            try:
                assert B.ssd_ctx_views(ctx).pass_rows == (48 if flags else 384)
                B.ssd_ctx_fill_synthetic_kv(ctx, lens, seed)
                B.ssd_ctx_set_forced(ctx, keys, toks)
                B.ssd_prespeculate(ctx, pending, temps, 1)
                c = B.read_cache(ctx)
                got.append([c[n].cpu().numpy() for n in ("glue_logits", "logits", "hidden")])
            finally:
                B.ssd_ctx_destroy(ctx)
    finally:
        B.ssd_model_destroy(model)
    for name, a, b in zip(("glue_logits", "logits", "hidden"), *got):
        e = row_rel_err(a, b)
        print(f"[wide] {name} {e:.2e}", flush=True)
        assert e < 2 * TOL_WIDE_BF16


@pytest.mark.parametrize("nb,T", [(16, 1), (16, 3), (12, 4), (13, 4)])
@pytest.mark.parametrize("paged", [False, True])
def test_extends_of_few_rows_in_a_context_of_wide_passes(B, nb, T, paged):
    """Up to 48 rows such a context takes the persistent pass of the narrow contexts: the same bits, also between rounds of wide
    passes; beyond (13 x 4 rows) it stays with wide passes."""
    print(f"[case] {nb} sequences, extend of {T} tokens, paged {paged}", flush=True)
    P, seed = 75, 5 + nb
    pages = 1 + nb * 4 if paged else 0
    SHAPE = I.ModelShape(n_layers=2, d_model=1024, n_q_heads=16, n_kv_heads=4, head_dim=64, d_ffn=2048, vocab=4112, dtype="bf16",
                         rope_theta=500000.0, tie_embeddings=True)     # (narrower models keep the wide passes)
    model = B.ssd_model_create(SHAPE, I.make_weights(SHAPE, 3))
    ctxs = [B.ssd_ctx_create(model, nb, K, F, P + 4 * K + 8, flags, pages) for flags in (0, B.SSD_CTX_NARROW_PASSES)]
    try:
        assert [B.ssd_ctx_views(c).pass_rows for c in ctxs] == [384, 48]
        g = np.random.default_rng(seed)
        tokens = dev_i32(g.integers(0, SHAPE.vocab, (nb, T)))
        pending, temps = dev_i32(I.make_pending(SHAPE, nb, K, seed)), dev_f32(np.zeros(nb))
        got = []
        for ctx in ctxs:
            z = [torch.zeros((nb, T, SHAPE.vocab), dtype=torch.float32, device="cuda") for _ in range(2)]
            B.ssd_ctx_fill_synthetic_kv(ctx, [P - b for b in range(nb)], seed)
            B.ssd_ctx_extend(ctx, tokens, 0, z[0])
            B.ssd_prespeculate(ctx, pending, temps, 1)
            B.ssd_ctx_extend(ctx, tokens, 0, z[1])
            torch.cuda.synchronize()
            B.ssd_ctx_status(ctx)
            got.append([x.cpu().numpy() for x in z])
        assert np.array_equal(got[0][0], got[0][1])
        if nb * T <= 48:
            assert np.array_equal(got[0][0], got[1][0])
        else:
            assert row_rel_err(got[0][0], got[1][0]) < 2 * TOL_WIDE_BF16
    finally:
        for ctx in ctxs:
            B.ssd_ctx_destroy(ctx)
        B.ssd_model_destroy(model)


@pytest.mark.parametrize("nb,T,P,small", [(8, 6, 1500, True), (8, 6, 32768, False), (3, 16, 1500, True), (3, 16, 65536, False), (16, 3, 32768, True)])
def test_few_rows_over_long_trunks_take_the_pass_that_reads_their_keys_once(B, nb, T, P, small):
    """Sequences of several query tiles pull the same keys once per tile in the persistent pass: over long trunks they stay with the
    wide pass (the bits of a context without the persistent kernel), over short ones and with one query tile (16 x 3 rows) they
    take the persistent pass (the bits of a context of narrow passes)."""
    print(f"[case] {nb} sequences of {P} keys, extend of {T} tokens", flush=True)
    K, F, seed = max(T - 1, 3), 2, 5 + nb
    shape = I.ModelShape(n_layers=2, d_model=1024, n_q_heads=16, n_kv_heads=4, head_dim=64, d_ffn=2048, vocab=4112, dtype="bf16",
                         rope_theta=500000.0, tie_embeddings=True)
    model = B.ssd_model_create(shape, I.make_weights(shape, 3))
    ctxs = [B.ssd_ctx_create(model, nb, K, F, P + 2 * K + 8, flags) for flags in (0, B.SSD_CTX_FUSED_PHASES, B.SSD_CTX_NARROW_PASSES)]
    try:
        assert all(B.ssd_ctx_views(c).fused_pass for c in ctxs)
        tokens, got = dev_i32(np.random.default_rng(seed).integers(0, shape.vocab, (nb, T))), []
        for ctx in ctxs:
            z = torch.zeros((nb, T, shape.vocab), dtype=torch.float32, device="cuda")
            B.ssd_ctx_fill_synthetic_kv(ctx, [P - b for b in range(nb)], seed)
            B.ssd_ctx_extend(ctx, tokens, 0, z)
            torch.cuda.synchronize()
            B.ssd_ctx_status(ctx)
            got.append(z.cpu().numpy())
        assert row_rel_err(got[1], got[2]) < 2 * TOL_WIDE_BF16
        assert np.array_equal(got[0], got[2 if small else 1])
        assert not np.array_equal(got[1], got[2])
    finally:
        for ctx in ctxs:
            B.ssd_ctx_destroy(ctx)
        B.ssd_model_destroy(model)


@pytest.mark.parametrize("heads_kv,base,F,paged", [(4, 1024, 2, False), (4, 1024, 16, True), (4, 4096, 2, True), (8, 4096, 16, False), (1, 4096, 2, False), (1, 1024, 16, True)])
def test_remainders_of_prompts_on_the_persistent_pass(B, heads_kv, base, F, paged):
    """What full passes of 1024 rows leave of a prompt, 16 to 48 rows of ONE sequence, in one persistent launch: one and two blocks of
    the pass's own keys, 2 to 48 query tiles per head, key splits over the longer prompts; 49 rows are a wide pass.  In contexts of
    narrow and of wide rounds, against chunks of K+1 tokens."""
    shape = I.ModelShape(n_layers=2, d_model=1024, n_q_heads=16, n_kv_heads=heads_kv, head_dim=64, d_ffn=2048, vocab=4112, dtype="bf16",
                         rope_theta=500000.0, tie_embeddings=True)
    model, max_trunk = B.ssd_model_create(shape, I.make_weights(shape, 17)), base + 49 + 2 * K + 8
    prompt, last = dev_i32(I.make_prompt(shape, 1, base + 49, 23)), dev_i32([[7]])
    pages = 1 + (max_trunk + 31) // 32 if paged else 0
    ctxs = [B.ssd_ctx_create(model, 1, K, f, max_trunk, flags, n)
            for flags, f, n in ((0, F, pages), (B.SSD_CTX_FUSED_PHASES, F, pages), (B.SSD_CTX_NARROW_PASSES, 2, 0))]
    try:
        assert all(B.ssd_ctx_views(c).fused_pass for c in ctxs)
        for r in (16, 17, 32, 33, 47, 48, 49):
            print(f"[case] {base} + {r} tokens, {heads_kv} KV heads, F {F}, paged {paged}", flush=True)
            got = []
            for ctx in ctxs:
                B.ssd_ctx_prefill(ctx, prompt, [base + r])
                z = torch.zeros((1, 1, shape.vocab), dtype=torch.float32, device="cuda")
                B.ssd_ctx_extend(ctx, last, 0, z)
                torch.cuda.synchronize()
                B.ssd_ctx_status(ctx)
                ks, vs = ([], []) if paged else _trunk(B, ctx, [base + r], max_trunk, shape)
                got.append((z.cpu().numpy(), [x[0][base:] for x in ks + vs]))
            assert row_rel_err(got[0][0], got[2][0]) < 2 * TOL_BF16_OWN_PREFILL, r
            for a, b in zip(got[0][1], got[2][1]):
                assert row_rel_err(a, b) < 2 * TOL_BF16_OWN_PREFILL, r
            if not paged:                                      # the pass that the remainder takes: its keys' bits
                same = all(np.array_equal(a, b) for a, b in zip(got[0][1], got[1][1]))
                assert same == (r > 48), r
    finally:
        for ctx in ctxs:
            B.ssd_ctx_destroy(ctx)
        B.ssd_model_destroy(model)


def test_expired_wait_and_recovery_in_a_context_of_wide_passes(B):
    """The glue extend of a small batch is a persistent launch also where the rounds are wide passes: with a limit of one poll its
    bounded waits expire and every workgroup leaves the kernel.  The context reports it, refuses the hot calls, and computes the
    same bits again after ssd_ctx_recover."""
    nb, P, F, seed = 4, 75, 4, 9
    shape = I.ModelShape(n_layers=2, d_model=1024, n_q_heads=16, n_kv_heads=4, head_dim=64, d_ffn=2048, vocab=4112, dtype="bf16",
                         rope_theta=500000.0, tie_embeddings=True)
    model = B.ssd_model_create(shape, I.make_weights(shape, 3))
    ctx = B.ssd_ctx_create(model, nb, K, F, P + 4 * K + 8)
    try:
        assert B.ssd_ctx_views(ctx).pass_rows == 384
        pending, temps = dev_i32(I.make_pending(shape, nb, K, seed)), dev_f32(np.zeros(nb))
        B.ssd_ctx_fill_synthetic_kv(ctx, [P] * nb, seed)
        B.ssd_prespeculate(ctx, pending, temps, 1)
        good = {k: v.cpu().numpy() for k, v in B.read_cache(ctx).items()}
        B.ssd_ctx_status(ctx)
        B.ssd_ctx_debug_set(ctx, B.SSD_DEBUG_SPIN_LIMIT, 1)
        print("[fault] launching one extend whose bounded waits expire after one poll", flush=True)
        B.ssd_ctx_extend(ctx, pending, 0, None)
        torch.cuda.synchronize()
        for call in (lambda: B.ssd_ctx_status(ctx), lambda: B.ssd_prespeculate(ctx, pending, temps, 1), lambda: B.ssd_ctx_extend(ctx, pending, 0, None)):
            with pytest.raises(B.SsdError) as e:
                call()
            assert e.value.status == B.SSD_EHIP
        B.ssd_ctx_debug_set(ctx, B.SSD_DEBUG_SPIN_LIMIT, 0)
        B.ssd_ctx_recover(ctx)
        B.ssd_ctx_fill_synthetic_kv(ctx, [P] * nb, seed)
        B.ssd_prespeculate(ctx, pending, temps, 1)
        again = {k: v.cpu().numpy() for k, v in B.read_cache(ctx).items()}
        B.ssd_ctx_refresh_bounds(ctx)
        for name in ("keys", "tokens", "logits", "hidden", "glue_logits"):
            assert np.array_equal(good[name], again[name]), name
    finally:
        B.ssd_ctx_destroy(ctx)
        B.ssd_model_destroy(model)


def test_captured_extend_of_few_rows_takes_the_wide_pass(B):
    """Persistent launches take turns by events, which a replay would not see: inside a stream capture the extend of a context of wide
    passes is wide launches (the bits of a context without the persistent kernel).  Replayed with eager work in between."""
    nb, T, P, F, seed = 4, 4, 200, 4, 9
    shape = I.ModelShape(n_layers=2, d_model=1024, n_q_heads=16, n_kv_heads=4, head_dim=64, d_ffn=2048, vocab=4112, dtype="bf16",
                         rope_theta=500000.0, tie_embeddings=True)
    model = B.ssd_model_create(shape, I.make_weights(shape, 3))
    ctx, wide = (B.ssd_ctx_create(model, nb, K, F, P + 4 * K + 8, flags) for flags in (0, B.SSD_CTX_FUSED_PHASES))
    try:
        assert all(B.ssd_ctx_views(c).fused_pass for c in (ctx, wide))
        sets = [dev_i32(np.random.default_rng(i).integers(0, shape.vocab, (nb, T))) for i in range(4)]
        tokens, z = sets[0].clone(), torch.zeros((nb, T, shape.vocab), dtype=torch.float32, device="cuda")
        eager = torch.zeros_like(z)
        for c in (ctx, wide):
            B.ssd_ctx_fill_synthetic_kv(c, [P - b for b in range(nb)], seed)
        want = []
        for t in sets:
            B.ssd_ctx_extend(wide, t, 0, z)
            want.append(z.clone())
        B.ssd_ctx_extend(ctx, tokens, 0, eager)                # (first launches outside the capture)
        torch.cuda.synchronize()
        graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        with torch.cuda.graph(graph, stream=stream):
            B.ssd_ctx_extend(ctx, tokens, 0, z, stream=stream)
        for t, w in zip(sets, want):
            tokens.copy_(t)
            z.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(z, w)
            B.ssd_ctx_extend(ctx, t, 0, eager)                 # eager work between the replays: the persistent pass
            torch.cuda.synchronize()
            assert not torch.equal(eager, w)
            assert row_rel_err(eager.cpu().numpy(), w.cpu().numpy()) < 2 * TOL_WIDE_BF16
        B.ssd_ctx_status(ctx)
    finally:
        for c in (ctx, wide):
            B.ssd_ctx_destroy(c)
        B.ssd_model_destroy(model)


# (width, d_ffn, prompt rows): gate/up takes another block at each, with whole and with partly filled row groups, and o and down two, four
# and eight slices
BLOCK_PROMPTS = [(512, 8192, 20), (512, 8192, 32), (512, 2048, 100), (512, 8192, 64), (512, 8192, 65), (512, 8192, 96), (512, 8192, 128), (512, 8192, 190),
                 (512, 8192, 250), (512, 8192, 256), (512, 8192, 384), (512, 8192, 500), (512, 8192, 513), (512, 8192, 768), (512, 8192, 1000),
                 (2048, 2048, 300)]
# (prompt rows, trunk positions) at the layers of the 1B shape: every block and number of slices that qkv, o, gate/up and down of a wide
# pass take there, row groups whole and partly filled (the trunk's room decides how many rows of partial sums o and down may write)
BLOCK_PROMPTS_1B = [(58, 0), (64, 0), (74, 0), (128, 0), (160, 0), (256, 0), (384, 0), (450, 1100), (490, 0), (512, 0), (700, 0), (768, 0),
                    (1003, 0)]
# prompt rows at a width of 2048 under 64 query and 16 KV heads and a d_ffn of 512: larger blocks of qkv, o and down in one slice
BLOCK_PROMPTS_64_HEADS = [500, 900, 1003]
# (width, query heads, KV heads, d_ffn, prompt rows): the kernel of passes of up to 48 rows, every instance of it and the first that is not
FEW_ROW_PROMPTS = [(512, 8, 2, 8192, n) for n in (5, 16, 17, 32, 33, 48, 49)] + [(1024, 16, 4, 1024, n) for n in (16, 31, 48)] + [
    (2048, 32, 8, 2048, 20), (2048, 32, 8, 8192, 48), (2048, 64, 16, 512, 48), (512, 8, 2, 512, 30)]
# (vocabulary, sequences, F) with K = 2: the LM head's blocks, the last of them with features behind the vocabulary
BLOCK_ROUNDS = [(66016, 16, 3), (66016, 16, 4), (66016, 16, 6), (66016, 16, 8), (20016, 16, 8), (4112, 11, 3), (4112, 16, 8),
                (2000, 5, 7), (2592, 14, 8), (5552, 11, 8), (8512, 13, 8), (10288, 11, 8), (32784, 9, 8), (128256, 14, 5)]


def _layer_shape(q_heads, kv_heads, ffn, width=2048):
    return I.ModelShape(n_layers=2, d_model=width, n_q_heads=q_heads, n_kv_heads=kv_heads, head_dim=64, d_ffn=ffn, vocab=4112, dtype="bf16",
                        rope_theta=500000.0, tie_embeddings=True)


@pytest.fixture(scope="module")
def layer_models(B):
    """Models of two layers, made once per shape."""
    made = {}

    def model_of(*sizes):
        if sizes not in made:
            shape = _layer_shape(*sizes)
            made[sizes] = (shape, B.ssd_model_create(shape, I.make_weights(shape, 17)))
        return made[sizes]
    yield model_of
    for _, model in made.values():
        B.ssd_model_destroy(model)


def _compare_with_narrow_chunks(B, shape, model, rows, max_trunk, flags=0):
    """One prompt in a wide pass against the narrow passes' own kernels."""
    prompt, lens = dev_i32(I.make_prompt(shape, 1, rows, 5 + rows)), [rows]
    ctxs = [B.ssd_ctx_create(model, 1, K, F, max_trunk, f) for f in (flags, B.SSD_CTX_NARROW_PASSES)]
    try:
        got = []
        for ctx in ctxs:
            B.ssd_ctx_prefill(ctx, prompt, lens)
            got.append(_trunk(B, ctx, lens, max_trunk, shape))
        # each side is within TOL_BF16_OWN_PREFILL of the exact keys and values
        for part in (0, 1):
            for l in range(shape.n_layers):
                assert row_rel_err(got[0][part][l][0], got[1][part][l][0]) < 2 * TOL_BF16_OWN_PREFILL, (part, l)
        assert not np.array_equal(got[0][0][1][0], got[1][0][1][0])          # (the prompt did go through another pass)
    finally:
        for ctx in ctxs:
            B.ssd_ctx_destroy(ctx)


@pytest.mark.parametrize("rows,trunk", BLOCK_PROMPTS_1B)
def test_blocks_of_prompt_passes_at_the_1b_layers(B, layer_models, rows, trunk):
    print(f"[case] 1B layers, {rows} rows, trunk {trunk}", flush=True)
    _compare_with_narrow_chunks(B, *layer_models(32, 8, 8192), rows, trunk or rows + 2 * K + 8)


@pytest.mark.parametrize("width,heads,kv_heads,ffn,rows", FEW_ROW_PROMPTS)
def test_wide_passes_of_few_rows(B, layer_models, width, heads, kv_heads, ffn, rows):
    """(One launch per phase: a context that may launch the persistent kernel takes that for so few rows from a width of 1024 on.)"""
    print(f"[case] width {width}, {heads} heads, d_ffn {ffn}, {rows} rows", flush=True)
    _compare_with_narrow_chunks(B, *layer_models(heads, kv_heads, ffn, width), rows, rows + 2 * K + 8, B.SSD_CTX_FUSED_PHASES)


@pytest.mark.parametrize("rows", BLOCK_PROMPTS_64_HEADS)
def test_blocks_of_prompt_passes_under_64_heads(B, layer_models, rows):
    print(f"[case] 64 heads, {rows} rows", flush=True)
    _compare_with_narrow_chunks(B, *layer_models(64, 16, 512), rows, rows + 2 * K + 8)


@pytest.mark.parametrize("width,ffn,rows", BLOCK_PROMPTS)
def test_blocks_of_prompt_passes(B, width, ffn, rows):
    """Every block that the linear layers of wide passes are cut into, against the narrow passes' own kernels."""
    print(f"[case] width {width}, d_ffn {ffn}, {rows} rows", flush=True)
    shape = I.ModelShape(n_layers=2, d_model=width, n_q_heads=width // 64, n_kv_heads=2, head_dim=64, d_ffn=ffn, vocab=4112, dtype="bf16",
                         rope_theta=500000.0, tie_embeddings=True)
    model = B.ssd_model_create(shape, I.make_weights(shape, 17))
    try:
        _compare_with_narrow_chunks(B, shape, model, rows, rows + 2 * K + 8)
    finally:
        B.ssd_model_destroy(model)


@pytest.mark.parametrize("vocab,nb,F_", BLOCK_ROUNDS)
def test_blocks_of_the_head(B, vocab, nb, F_):
    print(f"[case] vocabulary {vocab}, {nb} sequences, F {F_}", flush=True)
    K_, P = 2, 40
    shape = I.ModelShape(n_layers=1, d_model=512, n_q_heads=8, n_kv_heads=2, head_dim=64, d_ffn=1024, vocab=vocab, dtype="bf16",
                         rope_theta=500000.0, tie_embeddings=True)
    model = B.ssd_model_create_random(shape, 3)
    R = (K_ + 1) * F_
    pending = dev_i32(I.make_pending(shape, nb, K_, 3))
    rng = np.random.default_rng(vocab + nb)
    keys = dev_i32(np.stack([rng.permutation(vocab)[:R] for _ in range(nb)]))
    tokens, temps = dev_i32(rng.integers(0, vocab, (nb, R, K_))), dev_f32(np.zeros(nb))
    out = []
    try:
        for flags in (0, B.SSD_CTX_NARROW_PASSES):
            ctx = B.ssd_ctx_create(model, nb, K_, F_, P + 2 * K_ + 8, flags)
            try:
                B.ssd_ctx_fill_synthetic_kv(ctx, [P] * nb, 4)
                B.ssd_ctx_set_forced(ctx, keys, tokens)
                B.ssd_prespeculate(ctx, pending, temps, 1)
                out.append(B.read_cache(ctx)["logits"].reshape(-1, vocab).float())
                B.ssd_ctx_refresh_bounds(ctx)
            finally:
                B.ssd_ctx_destroy(ctx)
        err = ((out[0] - out[1]).abs().amax(dim=1) / out[1].abs().amax(dim=1)).max().item()
        print(f"[head] {err:.2e}", flush=True)
        assert err < 2 * TOL_WIDE_BF16                         # each side is within TOL_WIDE_BF16 of the exact logits
    finally:
        B.ssd_model_destroy(model)
