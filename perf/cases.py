"""The calls that a serving loop around this library makes, as cases to be timed: pre-speculation rounds of the draft,
prompt prefill, the target's verification forward, just-in-time drafting after a cache miss, and verification alone.

Shapes are those of the repository's own workloads (`ssd_inputs`): the tiny fp32 pair, the Llama-3.2-1B-shaped bf16 draft,
and layers of the Llama-3.1-70B-shaped bf16 target.  Weights, prefix KV, prompts and logits are random and made on the
GPU from the seed.

Two things keep the outputs of two correct implementations comparable.  The tokens the branches feed are given
(`ssd_ctx_set_forced`; the drafting loop feeds given tokens too): the library still selects, draws and stores its own, so the
kernels and the work are the same, but a near-tie early in a branch cannot turn the rest of it into another text.  And where a
greedy argmax or a top-F over 128256 random bf16-model logits decides (its ranks are 0.04 to 0.2 apart and the logits carry
errors of 1e-3, so that near-ties are common), the choice comes back as the logits it selected, which two correct
implementations share to rounding, beside all the logits.  fp32 and sampled choices come back as token ids."""
import math

import torch

import ssd_inputs as I
from paper_2603_03251_amd import binding as B

MODELS = {
    "tiny": I.TINY,
    "1b": I.LLAMA_1B,
    # the 70B-shaped target's layers (4 of its 80) under a 16384-token vocabulary: every kernel at its real layer shape
    "70b_layers": I.ModelShape(n_layers=4, d_model=8192, n_q_heads=64, n_kv_heads=8, head_dim=128, d_ffn=28672, vocab=16384,
                               dtype="bf16", rope_theta=500000.0, tie_embeddings=False),
}
VOCAB = I.LLAMA_1B.vocab


def listed():
    return [
        # ---- pre-speculation rounds: one per verification of the target
        # the smallest model: fp32, ten branches, everything is launches and latency
        dict(name="round_tiny_f32", kind="round", model="tiny", B=1, P=128, K=4, F=2, T=0.0),
        # a short chat turn with few branches: one row tile
        dict(name="round_1b_p211_k3_f2", kind="round", model="1b", B=1, P=211, K=3, F=2, T=0.0),
        # the headline workload as bench.py runs it: the round, the verification on a second stream, the cache lookup
        dict(name="round_1b_p1024_k5_f4", kind="round", model="1b", B=1, P=1024, K=5, F=4, T=0.0, verify=True),
        # a long context, sampled, wide fan-out
        dict(name="round_1b_p8192_k5_f8_t1", kind="round", model="1b", B=1, P=8192, K=5, F=8, T=1.0),
        # a small serving batch with prompts of different lengths, paged trunk, the Saguaro sampling scheme
        dict(name="round_1b_b4_paged_t07", kind="round", model="1b", B=4, P=1500, ragged=True, K=5, F=4, T=0.7, C=0.7, paged=True),
        # the large serving batch
        dict(name="round_1b_b16_p2048_k5_f4", kind="round", model="1b", B=16, P=2048, K=5, F=4, T=0.0),
        # ---- a request arrives: its prompt into an empty trunk, then the extend that gives the first logits
        dict(name="prefill_1b_p1021", kind="prefill", model="1b", B=1, P=1021, K=5, F=4),
        # a new request joins a running batch: its slot is prefilled while the others keep their state
        dict(name="join_1b_b8_p300", kind="join", model="1b", B=8, P=300, K=5, F=4),
        # ---- the target: one forward over the pending block, then rejection sampling
        dict(name="target_70b_layers_p4096", kind="target", model="70b_layers", B=1, P=4096, K=5, T=1.0),
        # ---- a cache miss: the next speculation is drafted token by token
        dict(name="draft_1b_p1500_k5", kind="draft", model="1b", B=1, P=1500, K=5, F=4),
        # ---- verification alone: one sequence, and a batch of greedy and sampled sequences
        dict(name="verify_b1_k5", kind="verify", B=1, K=5, V=VOCAB, T=1.0),
        dict(name="verify_b16_k5_mixed", kind="verify", B=16, K=5, V=VOCAB, T=0.8, mixed=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    most = 0.8 * max(_cost(c) for c in listed())
    while True:
        kind = rng.choice(["round", "round", "round", "round", "prefill", "join", "target", "draft", "verify", "verify"])
        K = rng.randint(2, 7)
        if kind == "round" and rng.random() < 0.2:
            c = dict(kind=kind, model="tiny", B=rng.randint(1, 3), P=_log_int(rng, 16, 400), K=min(K, 5), F=rng.randint(1, 4), T=0.0)
        elif kind == "round":
            c = dict(kind=kind, model="1b", B=_log_int(rng, 1, 16), P=_log_int(rng, 100, 8192), K=K, F=rng.randint(1, 8),
                     T=rng.choice([0.0, 0.0, 0.8, 1.0]))
            if c["B"] > 1 and rng.random() < 0.6:
                c["ragged"] = True
            if rng.random() < 0.25:
                c["paged"] = True
            if c["B"] * (K + 1) * c["F"] > 384:
                continue
        elif kind == "prefill":
            c = dict(kind=kind, model="1b", B=rng.randint(1, 4), P=_log_int(rng, 60, 1000), K=rng.randint(5, 7), F=rng.randint(1, 5))
        elif kind == "join":
            c = dict(kind=kind, model="1b", B=rng.randint(2, 10), P=_log_int(rng, 60, 800), K=rng.randint(4, 7), F=rng.randint(1, 4))
        elif kind == "target":
            c = dict(kind=kind, model="70b_layers", B=rng.randint(1, 3), P=_log_int(rng, 200, 4096), K=K, T=rng.choice([0.0, 1.0]))
        elif kind == "draft":
            c = dict(kind=kind, model="1b", B=rng.randint(1, 4), P=_log_int(rng, 100, 4096), K=K, F=rng.randint(1, 4))
        else:
            c = dict(kind=kind, B=_log_int(rng, 1, 16), K=K, V=rng.choice([VOCAB, VOCAB, 32003, 50257]), T=rng.choice([0.0, 0.6, 1.0]),
                     mixed=rng.random() < 0.4)
        if _cost(c) <= most:
            return c


# ------------------------------------------------------------------------------------------------ what a pass needs

def _weights(s):
    """Elements of the linear layers of one forward, without and with the LM head."""
    layer = (s.n_q_heads + 2 * s.n_kv_heads) * s.head_dim * s.d_model + s.d_model * s.n_q_heads * s.head_dim + 3 * s.d_model * s.d_ffn
    return s.n_layers * layer, s.n_layers * layer + s.vocab * s.d_model


def _forward(s, rows, kv_positions, attended, logit_rows):
    """Bytes and flops of one forward: weights once, stored KV once, the rows' own KV, fp32 logits."""
    es = 2 if s.dtype == "bf16" else 4
    body, full = _weights(s)
    kvd = s.n_kv_heads * s.head_dim
    w = full if logit_rows else body
    nbytes = w * es + s.n_layers * (kv_positions + rows) * 2 * kvd * es + logit_rows * s.vocab * 4
    flops = 2.0 * rows * body + 2.0 * logit_rows * s.vocab * s.d_model + 4.0 * s.n_layers * s.n_q_heads * s.head_dim * attended
    return nbytes, flops


def _lens(c):
    """Prefix length of every sequence: the same, or spread from a tenth of P to P."""
    if not c.get("ragged"):
        return [c["P"]] * c["B"]
    return [max(8, int(c["P"] * (1.0 - 0.9 * ((7 * b) % c["B"]) / c["B"]))) for b in range(c["B"])]


def work(case):
    c = case
    K = c["K"]
    if c["kind"] == "verify":
        sampled = [t > 0 for t in _temperatures(c)]
        rows = sum(2 * K + 1 if s else K + 1 for s in sampled)
        return {"bytes": rows * c["V"] * 4.0, "flops": 10.0 * rows * c["V"]}
    s = MODELS[c["model"]]
    nb, lens = c["B"], _lens(c)
    pos = sum(lens)
    if c["kind"] == "round":
        rows = nb * (K + 1) * c["F"]
        by, fl = _forward(s, nb * (K + 1), pos, (K + 1) * pos, nb * (K + 1))
        b2, f2 = _forward(s, rows, pos, (K + 1) * c["F"] * pos, rows)
        by, fl = by + K * b2, fl + K * f2
        if c.get("verify"):
            by += nb * (K + 1) * s.vocab * 4.0
        return {"bytes": float(by), "flops": fl}
    if c["kind"] in ("prefill", "join"):
        n = nb if c["kind"] == "prefill" else 1
        by, fl = _forward(s, n * c["P"], 0, n * c["P"] * c["P"] / 2.0, 0)
        b2, f2 = _forward(s, nb, nb * c["P"], nb * c["P"], nb)
        return {"bytes": float(by + b2), "flops": fl + f2}
    if c["kind"] == "target":
        by, fl = _forward(s, nb * (K + 1), pos, (K + 1) * pos, nb * (K + 1))
        return {"bytes": by + nb * (2 * K + 1) * s.vocab * 4.0, "flops": fl}
    by, fl = _forward(s, nb, pos, pos, nb)
    return {"bytes": float(K * by), "flops": K * fl}


def _cost(c):
    w = work(c)
    if c["kind"] in ("prefill", "join"):
        # a prompt is counted by the rows it brings, not by the one pass over the weights it could be
        w = {"bytes": w["bytes"] * (1 if c["kind"] == "join" else c["B"]) * c["P"] / 48.0, "flops": w["flops"]}
    return max(w["bytes"], w["flops"] / 50.0)


def tolerance(case):
    """Measured between the library's own paths for the same weights (fused passes with one and with two activation planes,
    narrow and wide passes, one kernel per operator), times about four: through 16 bf16 layers logits and hidden states differ by
    1.8e-3 (2-norm; largest element 1.1e-2), stored bf16 keys and values after a prefill by 2.5e-3 (1.4e-2); fp32 by 3e-7.  Sampled
    ids: the two best scores of a draw are about 1 apart and the logits carry 2e-3; 1 of 240 differed."""
    if case["kind"] == "verify":
        return "exact"
    if case["model"] == "tiny":
        return {"rel": 2e-6, "max": 2e-5}
    t = {"rel": 1e-2 if case["kind"] in ("prefill", "join") else 7e-3, "max": 0.06}
    if case.get("T", 0.0) > 0.0:
        t["differ"] = 0.01
        if case.get("C", 1.0) < 1.0:
            # the scheme lowers the top-F logits of a row by T log C: a near-tie at rank F lowers another one
            t["max"] = 0.4
    return t


# ------------------------------------------------------------------------------------------------ states

class _Handles:
    """A model and a context; gives the library's memory back when nothing refers to it any more."""
    model = None
    ctx = None

    def __del__(self):
        try:
            torch.cuda.synchronize()
            if self.ctx is not None:
                B.ssd_ctx_destroy(self.ctx)
            if self.model is not None:
                B.ssd_model_destroy(self.model)
        except Exception:   # at interpreter exit the modules may be gone
            pass


class _Foreign:
    """Library-owned device memory as torch sees it.  A tensor made from this keeps it, and with it the memory's owner, alive."""

    def __init__(self, owner, ptr, shape, typestr):
        self.owner = owner
        self.__cuda_array_interface__ = {"data": (int(ptr), False), "shape": tuple(shape), "typestr": typestr, "version": 2}


def _view(owner, ptr, shape, dtype):
    typestr = {torch.float32: "<f4", torch.int32: "<i4", torch.bfloat16: "<i2"}[dtype]
    t = torch.as_tensor(_Foreign(owner, ptr, shape, typestr), device="cuda")
    return t.view(torch.bfloat16) if dtype == torch.bfloat16 else t


class _State:
    """What the program around a pass holds: handles, inputs, output buffers."""


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) & 0x7FFFFFFF)


def _tokens(g, shape, vocab):
    return torch.randint(0, vocab, shape, generator=g, device="cuda", dtype=torch.int32)


def _temperatures(c):
    T = c.get("T", 0.0)
    return [0.0 if c.get("mixed") and b % 2 else T for b in range(c["B"])]


def _verify_inputs(g, nb, K, V):
    """Logits of a target and of a draft that is close to it (spread of 2.5 nats, differences of 0.7), and K tokens drawn from
    the draft's distribution: some positions are accepted, some rejected."""
    base = torch.randn((nb, K + 1, V), generator=g, device="cuda") * 2.5
    zt = base + 0.5 * torch.randn((nb, K + 1, V), generator=g, device="cuda")
    zd = (base[:, :K] + 0.5 * torch.randn((nb, K, V), generator=g, device="cuda")).contiguous()
    spec = torch.multinomial(torch.softmax(zd.reshape(nb * K, V), dim=1), 1, generator=g).reshape(nb, K).to(torch.int32)
    return zt, zd, spec.contiguous()


def _verify_outputs(nb, K):
    return (torch.zeros(nb, dtype=torch.int32, device="cuda"), torch.zeros(nb, dtype=torch.int32, device="cuda"),
            torch.empty(B.ssd_verify_workspace_bytes(nb, K), dtype=torch.uint8, device="cuda"))


def prepare(case, seed):
    c, s = case, _State()
    s.case, s.seed = c, int(seed)
    g = _generator(seed)
    nb, K = c["B"], c["K"]
    s.temps = torch.tensor(_temperatures(c), dtype=torch.float32, device="cuda")
    if c["kind"] == "verify":
        s.zt, s.zd, s.spec = _verify_inputs(g, nb, K, c["V"])
        s.k_out, s.t_out, s.ws = _verify_outputs(nb, K)
        return s

    shape = s.shape = MODELS[c["model"]]
    V = shape.vocab
    lens = _lens(c)
    F = c.get("F", 1)
    room = max(lens) + 2 * K + 2
    # paged: pages for every sequence's positions of a round, and the shared zero page
    pages = 1 + sum((n + K + 1 + 31) // 32 for n in lens) if c.get("paged") else 0
    s.handles = own = _Handles()
    own.model = B.ssd_model_create_random(shape, 1 + (int(seed) & 0xFFFFFF))
    own.ctx = s.ctx = B.ssd_ctx_create(own.model, nb, K, F, room, 0, pages)
    v = B.ssd_ctx_views(s.ctx)
    R = (K + 1) * F
    if c["kind"] in ("prefill", "join"):
        # the KV store of a fused context: keys [B][Hkv][T][64], values [B][Hkv][T/32][64][32]
        T = (room + 63) // 64 * 64
        hkv, hd, P = shape.n_kv_heads, shape.head_dim, c["P"]
        s.kv = []
        for l in range(shape.n_layers):
            k = _view(own, v.h_trunk_k[l], (nb, hkv, T, hd), torch.bfloat16)
            vt = _view(own, v.h_trunk_v[l], (nb, hkv, T // 32, hd, 32), torch.bfloat16)
            b0, b1 = (0, nb) if c["kind"] == "prefill" else (nb // 2, nb // 2 + 1)
            # (positions behind the prompt are not part of the result)
            s.kv += [k[b0:b1, :, :P - 1], vt[b0:b1, :, :(P - 1) // 32]]
        s.prompt = _tokens(g, (nb, P - 1), V)
        s.last = _tokens(g, (nb, 1), V)
        s.logits = torch.empty((nb, 1, V), dtype=torch.float32, device="cuda")
        if c["kind"] == "join":
            B.ssd_ctx_fill_synthetic_kv(s.ctx, [P - 1] * nb, s.seed + 3)
            s.prompt = s.prompt[nb // 2].contiguous()
        return s

    B.ssd_ctx_fill_synthetic_kv(s.ctx, lens, s.seed + 3)
    if c["kind"] == "target":
        s.pending = _tokens(g, (nb, K + 1), V)
        s.logits = torch.empty((nb, K + 1, V), dtype=torch.float32, device="cuda")
        _, s.zd, _ = _verify_inputs(g, nb, K, V)
        s.spec = s.pending[:, 1:].contiguous()
        s.k_out, s.t_out, s.ws = _verify_outputs(nb, K)
        return s
    if c["kind"] == "draft":
        s.feed = [_tokens(g, (nb, 1), V) for _ in range(K)]
        s.logits = [torch.empty((nb, 1, V), dtype=torch.float32, device="cuda") for _ in range(K)]
        s.drawn = torch.zeros((K, nb), dtype=torch.int32, device="cuda")
        return s

    # ---- round
    s.pending = _tokens(g, (nb, K + 1), V)
    s.forced_keys = torch.stack([torch.randperm(V, generator=g, device="cuda")[:R] for _ in range(nb)]).to(torch.int32).contiguous()
    s.forced_tokens = _tokens(g, (nb, R, K), V)
    B.ssd_ctx_set_forced(s.ctx, s.forced_keys, s.forced_tokens)
    if c.get("C", 1.0) < 1.0:
        B.ssd_ctx_set_saguaro(s.ctx, c["C"])
    s.out = {
        "glue_logits": _view(own, v.d_glue_logits, (nb, K + 1, V), torch.float32),
        "glue_hidden": _view(own, v.d_glue_hidden, (nb, K + 1, shape.d_model), torch.float32),
        "logits": _view(own, v.d_logits, (nb, R, K, V), torch.float32),
        "hidden": _view(own, v.d_hidden, (nb, R, K, shape.d_model), torch.float32),
    }
    s.keys = _view(own, v.d_keys, (nb, K + 1, F), torch.int32)
    s.tokens = _view(own, v.d_tokens, (nb, R, K), torch.int32)
    if c.get("verify"):
        s.zt, s.zd, s.spec = _verify_inputs(g, nb, K, V)
        s.k_out, s.t_out, s.ws = _verify_outputs(nb, K)
        s.hit = torch.zeros(nb, dtype=torch.uint8, device="cuda")
        s.branch = torch.zeros(nb, dtype=torch.int32, device="cuda")
        s.next = torch.zeros((nb, K), dtype=torch.int32, device="cuda")
        s.side = torch.cuda.Stream()
    return s


# ------------------------------------------------------------------------------------------------ passes

def _run_round(s, c):
    if c.get("verify"):
        main = torch.cuda.current_stream()
        s.side.wait_stream(main)
        B.ssd_prespeculate(s.ctx, s.pending, s.temps, s.seed)
        B.ssd_verify(s.zt, None, s.spec, s.temps, s.seed, s.k_out, s.t_out, s.ws, stream=s.side)
        main.wait_stream(s.side)
        B.ssd_cache_lookup(s.ctx, s.k_out, s.t_out, s.hit, s.branch, s.next)
        out = dict(s.out, outcome=(s.k_out, s.t_out, s.hit, s.branch, s.next))
    else:
        B.ssd_prespeculate(s.ctx, s.pending, s.temps, s.seed)
        out = dict(s.out)
    if c["model"] == "tiny":
        out.update(keys=s.keys, tokens=s.tokens)
        return out
    out["key_logits"] = torch.gather(s.out["glue_logits"], 2, s.keys.long())
    if c.get("T", 0.0) > 0.0:
        out["tokens"] = s.tokens
    else:
        out["token_logits"] = torch.gather(s.out["logits"], 3, s.tokens.long().unsqueeze(3))
    return out


def run(state):
    s, c = state, state.case
    kind = c["kind"]
    if kind == "round":
        return _run_round(s, c)
    if kind == "verify":
        B.ssd_verify(s.zt, s.zd, s.spec, s.temps, s.seed, s.k_out, s.t_out, s.ws)
        return {"accept_len": s.k_out, "bonus": s.t_out}
    if kind == "prefill":
        B.ssd_ctx_prefill(s.ctx, s.prompt, [c["P"] - 1] * c["B"])
        B.ssd_ctx_extend(s.ctx, s.last, 0, s.logits)
        return {"logits": s.logits, "kv": s.kv}
    if kind == "join":
        B.ssd_ctx_prefill_sequence(s.ctx, c["B"] // 2, s.prompt)
        B.ssd_ctx_extend(s.ctx, s.last, 0, s.logits)
        return {"logits": s.logits, "kv": s.kv}
    if kind == "target":
        B.ssd_ctx_extend(s.ctx, s.pending, 0, s.logits)
        B.ssd_verify(s.logits, s.zd, s.spec, s.temps, s.seed, s.k_out, s.t_out, s.ws)
        return {"logits": s.logits, "outcome": (s.k_out, s.t_out)}
    # just-in-time drafting: K single-token extends, the next token drawn after each
    for i in range(c["K"]):
        B.ssd_ctx_extend(s.ctx, s.feed[i], i, s.logits[i])
        B.ssd_sample(s.logits[i].reshape(c["B"], -1), s.temps, s.seed, 0, i, s.drawn[i])
    scores = [torch.gather(z.reshape(c["B"], -1), 1, t.long().unsqueeze(1)) for z, t in zip(s.logits, s.drawn)]
    return {"logits": s.logits, "drawn_logits": scores}
