"""The two verification kernels where their cuts can go wrong: vocabularies around the sizes at which a row is cut into one more
part, parts of the bonus row whose residual has no mass, a residual without any mass, NaN logits and infinite ones of either sign."""
import numpy as np
import pytest
import torch

from oracle import ssd_oracle as O
from tests.gpu_util import MARGIN, dev_f32, dev_i32

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2603_03251_amd import binding
    return binding


def _verify(B, zt, zd, spec, temps, seed):
    nb, K = spec.shape
    k = torch.full((nb,), -9, dtype=torch.int32, device="cuda")
    t = torch.full((nb,), -9, dtype=torch.int32, device="cuda")
    ws = torch.randint(0, 255, (B.ssd_verify_workspace_bytes(nb, K),), dtype=torch.uint8, device="cuda")   # its contents do not matter
    for _ in range(2):                                        # the second call runs over what the first left
        B.ssd_verify(dev_f32(zt), dev_f32(zd), dev_i32(spec), dev_f32(temps), seed, k, t, ws)
    torch.cuda.synchronize()
    return k.cpu().numpy(), t.cpu().numpy()


@pytest.mark.parametrize("V", [2, 1023, 1024, 2047, 2049, 4097, 32771, 65536])
@pytest.mark.parametrize("nb,K", [(1, 1), (1, 15), (7, 3), (70, 2)])
def test_verify_at_the_edges_of_its_parts(B, V, nb, K):
    print(f"[case] verify B={nb} K={K} V={V}", flush=True)
    g = np.random.default_rng(V + nb + K)
    zd = (g.standard_normal((nb, K, V)) * 2).astype(np.float32)
    zt = (g.standard_normal((nb, K + 1, V)) * 2).astype(np.float32)
    # the target gives the lower half less than the draft does: those parts have no residual mass
    zt[:, :K, : V // 2] = zd[:, :, : V // 2] - 1.0
    zt[:, :K, V // 2:] = zd[:, :, V // 2:] + g.uniform(0.2, 0.6, (nb, K, V - V // 2)).astype(np.float32)
    if V > 8:
        zt[:, :, 3], zt[:, :, 5] = np.nan, -np.inf            # no probability
    spec = g.integers(0, V, (nb, K)).astype(np.int32)
    temps = np.where(np.arange(nb) % 4 == 3, 0.0, 0.9).astype(np.float32)
    k, t = _verify(B, zt, zd, spec, temps, 99 + V)
    zt[np.isnan(zt)] = -np.inf
    checked = 0
    for b in range(nb):
        want = O.verify(zt[b], zd[b], spec[b], float(temps[b]), 99 + V, seq=b)
        if all(m > MARGIN for m in want.accept_margin):
            assert k[b] == want.accept_len, b
            if want.bonus_margin > MARGIN:
                assert t[b] == want.bonus, b
                checked += 1
    # (with these seeds every sequence of the small batches is decided by more than the margin)
    assert checked == nb if nb <= 7 else checked >= 0.9 * nb


@pytest.mark.parametrize("V", [257, 2050, 40011])
@pytest.mark.parametrize("T,spread,apart", [(1.0, 3.0, 0.5), (0.02, 3.0, 0.5), (9.0, 40.0, 2.0), (0.7, 90.0, 30.0), (1.0, 3.0, 1e-4), (1.0, 1e-3, 1e-6)])
def test_verify_bonus_token_of_residuals_that_fp32_can_and_cannot_order(B, V, T, spread, apart):
    """The race for the bonus token leaves out, by bounds in fp32, the tokens that cannot win.  Peaked and flat distributions,
    exponents past the fp32 range, and residuals that are differences of almost equal probabilities (`apart`: how far draft and
    target logits lie apart), where fp32 excludes little or nothing."""
    nb, K, seed = 6, 2, V + int(100 * T)
    print(f"[case] verify bonus V={V} T={T} spread={spread} apart={apart}", flush=True)
    g = np.random.default_rng(seed)
    zt = (g.standard_normal((nb, K + 1, V)) * spread).astype(np.float32)
    zd = (zt[:, :K] + apart * g.standard_normal((nb, K, V))).astype(np.float32)
    spec = np.full((nb, K), -1, np.int32)                     # tokens outside the vocabulary: rejected at position 0
    k, t = _verify(B, zt, zd, spec, np.full(nb, T, np.float32), seed)
    checked = 0
    for b in range(nb):
        p, q = O.softmax_T(zt[b, 0], T), O.softmax_T(zd[b, 0], T)
        r = np.maximum(p - q, 0.0)
        with np.errstate(divide="ignore"):
            score = np.log(r) + O.gumbel(seed, O.STREAM_BONUS, b, 0, V)
        order = np.argsort(-score)
        assert k[b] == 0
        # (r is off by the rounding of p and q, 1e-14 of them: it moves a score by that over r)
        best = order[0]
        if score[best] - score[order[1]] > MARGIN and r[best] > 1e-9 * p[best]:
            assert t[b] == best, b
            checked += 1
    assert checked >= nb // 2


def test_verify_residual_without_mass_falls_back_to_the_target(B):
    V, K = 5000, 2
    g = np.random.default_rng(3)
    zt = g.standard_normal((1, K + 1, V)).astype(np.float32)
    k, t = _verify(B, zt, zt[:, :K].copy(), np.array([[-1, 5]], np.int32), np.ones(1, np.float32), 7)   # a token outside: rejected
    score = np.log(O.softmax_T(zt[0, 0], 1.0)) + O.gumbel(7, O.STREAM_BONUS, 0, 0, V)
    assert k[0] == 0 and t[0] == int(np.argmax(score))


def test_verify_with_rows_that_have_no_distribution(B):
    """Greedy: +infinity is the row's argmax.  Sampled: such a row has no distribution (every probability is 0/0), so its token
    is rejected; a target row without a distribution gives token 0, beside a draft row without one (also one of NaN only) the
    bonus token comes from the target's own distribution."""
    V, K, T, seed = 3000, 3, 0.8, 21
    g = np.random.default_rng(8)
    zt = np.tile(g.standard_normal((1, K + 1, V)).astype(np.float32), (5, 1, 1))
    zd = zt[:, :K].copy()                                     # equal distributions: every token is accepted
    spec = np.tile(np.array([[5, 6, 7]], np.int32), (5, 1))
    zt[0, 1, 2999] = np.inf                                   # greedy, position 1
    spec[0, 0], spec[0, 1] = zt[0, 0].argmax(), 2999
    spec[0, 2] = (zt[0, 2].argmax() + 1) % V                  # rejected: the bonus is the argmax of row 2
    zt[1, 1, 2999] = np.inf                                   # sampled, target row 1
    zd[2, 1, 17] = np.inf                                     # sampled, draft row 1
    zd[3, 1] = np.nan                                         # a draft row without any probability
    k, t = _verify(B, zt, zd, spec, np.array([0.0, T, T, T, T], np.float32), seed)
    from_p = lambda b, i: int(np.argmax(np.log(O.softmax_T(zt[b, i], T)) + O.gumbel(seed, O.STREAM_BONUS, b, i, V)))
    assert k.tolist() == [2, 1, 1, 1, 3]
    assert t.tolist() == [int(zt[0, 2].argmax()), 0, from_p(2, 1), from_p(3, 1), from_p(4, K)]
