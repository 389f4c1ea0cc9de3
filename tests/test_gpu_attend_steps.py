"""The matrix-core attention kernel's step sequence against the oracle: every number of tiles a wave can be left with
around its two-steps-per-trip loop (none, one, ..., seven), a last tile of one token, of all but one and a full one, and
keys that grow along the context, so that rows keep moving their softmax reference."""
import numpy as np
import pytest

from oracle import polykv_oracle as O
from paper_2604_24971_amd import workloads as W
from test_gpu_parity import Case, _pk, _pu

pytestmark = pytest.mark.gpu


def _case(d, T, growing, **kw):
    rng = np.random.default_rng(1000 * d + T)
    K = rng.standard_normal((1, 2, T, d))
    if growing:
        K *= np.linspace(0.2, 9.0, T)[None, None, :, None]
    V = rng.standard_normal((1, 2, T, d))
    cfg = W.PoolConfig(0, "steps", 1, 2, 8, d, T, 10, 1)
    Q = rng.standard_normal((1, 10, 1, 8, d)).astype(np.float16)
    return Case(cfg, K.astype(np.float16), V.astype(np.float16), **kw), Q


# with one split a wave's tile count is ceil(tiles / 4): 1 .. 7, the waves of a workgroup differing by one
@pytest.mark.parametrize("tiles", [1, 4, 5, 8, 12, 13, 16, 20, 25, 28])
@pytest.mark.parametrize("d,rows", [(64, 8), (64, 40), (128, 8), (128, 40), (256, 40)])
def test_tiles_per_wave(tiles, d, rows):
    pk = _pk()
    T = 32 * tiles - {0: 0, 1: 31, 2: 1}[tiles % 3]
    case, Q = _case(d, T, growing=tiles % 2 == 0)
    Q = Q[:, :rows // 4]
    case.attend_check(Q, splits=1, kernel=pk.KERNEL_MATRIX)
    if tiles > 4:
        case.attend_check(Q, splits=3)


@pytest.mark.parametrize("codec", [dict(int8_values=True), dict(scaled_values=True), dict(scaled_values=True, value_bits=4),
                                   dict(value_bits=2), dict(key_per_tensor=True)])
@pytest.mark.parametrize("d", [64, 128, 256])
def test_codecs_over_growing_keys(codec, d):
    case, Q = _case(d, 32 * 21 + 5, growing=True, **codec)
    case.attend_check(Q, splits=1)
    case.attend_check(Q[:, :3], splits=2)


@pytest.mark.parametrize("heads,agents,splits", [(1, 33, 1), (3, 33, 1), (3, 17, 2), (9, 33, 3)])
def test_row_blocks_and_streams_that_do_not_fill_the_dies(heads, agents, splits):
    """Row blocks times (head, split) streams: the launch rounds the streams up to the eight dies."""
    rng = np.random.default_rng(heads * 100 + agents)
    T, d = 32 * 9 + 3, 64
    cfg = W.PoolConfig(0, "blocks", 1, heads, 4 * heads, d, T, agents, 1)
    case = Case(cfg, rng.standard_normal((1, heads, T, d)).astype(np.float16),
                rng.standard_normal((1, heads, T, d)).astype(np.float16))
    case.attend_check(rng.standard_normal((1, agents, 1, 4 * heads, d)).astype(np.float16), splits=splits)


# Many rows over KV heads enough to fill the CUs more than once: the waves have rows of their own.  One tile, a few, a
# ragged end; a last wave of one row and waves with none; a split token range (65 heads, 256 rows); private tails.
@pytest.mark.parametrize("d,heads,T,agents,q,group,tails", [
    (64, 40, 20, 33, 4, 4, False), (64, 40, 300, 57, 3, 3, False), (64, 65, 2300, 64, 1, 4, False), (128, 40, 131, 33, 4, 4, True),
    (128, 40, 33, 57, 3, 3, False), (256, 40, 129, 43, 2, 3, True), (256, 40, 64, 65, 4, 1, False)])
@pytest.mark.parametrize("codec", [dict(), dict(scaled_values=True), dict(key_per_tensor=True)])
def test_waves_with_rows_of_their_own(d, heads, T, agents, q, group, tails, codec):
    rng = np.random.default_rng(d + heads + T)
    half = lambda *s: rng.standard_normal(s).astype(np.float16)
    cfg = W.PoolConfig(0, "rows", 1, heads, heads * group, d, T, agents, q)
    K = half(1, heads, T, d) * np.linspace(0.2, 4.0, T)[None, None, :, None].astype(np.float16)
    case = Case(cfg, K, half(1, heads, T, d), **codec)
    kw = {}
    if tails:
        lens = [(7 * a) % 20 for a in range(agents)]
        kw = dict(tails_np=[(half(1, heads, 20, d), half(1, heads, 20, d)) for _ in lens], tails_len=lens)
    Q = half(1, agents, q, heads * group, d)
    assert case.pool.attend_plan(_pu().dev(Q)).own_rows == 1
    case.attend_check(Q, **kw)


@pytest.mark.parametrize("growing", [True, False])
@pytest.mark.parametrize("tiles", [2, 3, 4, 5, 6, 7])
def test_references_from_the_last_tiles(tiles, growing):
    """A wave's first tile and its last three set references, in waves of up to seven tiles, over keys that grow (references
    move up) and shrink (they move down, or lie too far below)."""
    rng = np.random.default_rng(tiles)
    heads, agents, q, group, d, T = 40, 33, 4, 4, 64, 32 * tiles - (tiles % 3)
    half = lambda *s: rng.standard_normal(s).astype(np.float16)
    size = np.linspace(0.1, 6.0, T)
    K = half(1, heads, T, d) * (size if growing else size[::-1])[None, None, :, None].astype(np.float16)
    case = Case(W.PoolConfig(0, "references", 1, heads, heads * group, d, T, agents, q), K, half(1, heads, T, d))
    Q = half(1, agents, q, heads * group, d)
    choice = case.pool.attend_plan(_pu().dev(Q))
    assert choice.own_rows == 1 and choice.references == 4
    case.attend_check(Q)


OTHER_CODECS = [dict(int8_values=True), dict(value_bits=2), dict(value_bits=2, scaled_values=True), dict(value_bits=4),
                dict(value_bits=4, scaled_values=True), dict(value_bits=4, key_per_tensor=True)]


# (int8 values at head_dim 256 are the vector kernel's)
@pytest.mark.parametrize("d,codec", [(d, c) for d in (64, 128, 256) for c in OTHER_CODECS if d != 256 or "int8_values" not in c])
def test_waves_with_rows_of_their_own_and_the_other_codecs(d, codec):
    rng = np.random.default_rng(d + len(codec))
    heads, T, agents, q, group = 40, 32 * 6 + 9, 33, 4, 4     # 528 rows: a last workgroup of one wave, six tiles and a few tokens
    half = lambda *s: rng.standard_normal(s).astype(np.float16)
    cfg = W.PoolConfig(0, "rows", 1, heads, heads * group, d, T, agents, q)
    K = half(1, heads, T, d) * np.linspace(0.2, 4.0, T)[None, None, :, None].astype(np.float16)
    case = Case(cfg, K, half(1, heads, T, d), **codec)
    Q = half(1, agents, q, heads * group, d)
    assert case.pool.attend_plan(_pu().dev(Q)).own_rows == 1
    case.attend_check(Q)


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("bf16,fp16_keys,causal", [(True, False, False), (False, True, False), (True, True, True), (False, False, True)])
def test_waves_with_rows_of_their_own_and_the_other_options(d, bf16, fp16_keys, causal):
    pk, pu = _pk(), _pu()
    rng = np.random.default_rng(d + 2 * bf16 + fp16_keys)
    heads, T, agents, q, group, cap = 40, 32 * 5 + 30, 40, 4, 3, 35
    rnd = (lambda x: W.bf16_round(x.astype(np.float32))) if bf16 else (lambda x: x.astype(np.float16))
    draw = lambda *s: rnd(rng.standard_normal(s))
    K, V, Q = draw(1, heads, T, d), draw(1, heads, T, d), draw(1, agents, q, heads * group, d)
    pool = pu.gpu_pool(K, V, bf16=bf16)
    ref = O.pool_encode(K, V)
    pu.compare_codes(pool, ref)
    Kh, Vh = O.pool_decode(ref)
    if fp16_keys and d != 256:       # (exact keys at head_dim 256 whatever is asked for)
        Kh = O.keys_as_fp16(Kh)
    lens = [(11 * a) % (cap + 1) for a in range(agents)]
    tails = [(draw(1, heads, cap, d), draw(1, heads, cap, d)) for _ in lens] if causal else None
    gpu = [(pu.dev(k, bf16), pu.dev(v, bf16), n) for (k, v), n in zip(tails, lens)] if causal else None
    cut = [(k[:, :, :n], v[:, :, :n]) for (k, v), n in zip(tails, lens)] if causal else None
    kw = dict(key_precision=pk.KEY_PRECISION_FP16 if fp16_keys else pk.KEY_PRECISION_EXACT, tails=gpu, tail_causal=causal)
    assert pool.attend_plan(pu.dev(Q, bf16), **kw).own_rows == 1
    out = pool.attend(pu.dev(Q, bf16), **kw)
    pu.compare_attend(out, O.pool_attend(Kh, Vh, Q, tails=cut, tail_causal=causal), heads)


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("codec", [dict(), dict(value_bits=4), dict(value_bits=2, scaled_values=True)])
def test_splits_that_are_merged(d, codec):
    """(Small pools are no longer split by themselves.)"""
    case, Q = _case(d, 32 * 13 + 6, growing=True, **codec)
    for splits in (2, 3):
        assert case.pool.attend_plan(_pu().dev(Q), splits=splits).splits == splits
        case.attend_check(Q, splits=splits)


# Queries with large sums over the key blocks, and references beyond what fp16 holds (60,000), in some of a wave's rows: their
# neighbours do not notice.
@pytest.mark.parametrize("d,heads,agents,q,block_rows,own", [
    (64, 2, 5, 1, 32, 0), (64, 2, 12, 1, 32, 0), (64, 256, 12, 1, 64, 0), (128, 2, 5, 1, 32, 0), (128, 2, 12, 1, 32, 0),
    (128, 256, 12, 1, 64, 0), (256, 2, 5, 1, 32, 0), (64, 40, 33, 4, 64, 1), (128, 40, 33, 4, 64, 1), (256, 40, 33, 4, 32, 1)])
@pytest.mark.parametrize("what", ["sums", "references"])
def test_rows_beyond_the_corrections_range(d, heads, agents, q, block_rows, own, what):
    rng = np.random.default_rng(d + agents)
    T, group = 32 * 9 + 5, 4
    cfg = W.PoolConfig(0, "range", 1, heads, heads * group, d, T, agents, q)
    K, V = rng.standard_normal((1, heads, T, d)), rng.standard_normal((1, heads, T, d)).astype(np.float16)
    Q = rng.standard_normal((1, agents, q, heads * group, d))
    far = np.zeros(agents, bool)
    far[1::3] = True
    if what == "sums":             # 300 in every coordinate: |W| = 128 * qscale * 9,600, scores of ordinary size over small keys
        K *= 0.01
        Q[:, far] += 300.0
    else:                          # scores of 10^5 and more; the six largest 10^4 apart (an ulp of them in fp32 is 0.016)
        K[:, :, 7::50] += 20.0 + 3.0 * np.arange(6)[:, None]
        Q[:, far] = 200.0 * np.abs(Q[:, far]) + 500.0
    case = Case(cfg, K.astype(np.float16), V)
    Q = Q.astype(np.float16)
    choice = case.pool.attend_plan(_pu().dev(Q))
    assert (choice.block_rows, choice.own_rows) == (block_rows, own)
    case.attend_check(Q)
    out = case.pool.attend(_pu().dev(Q))
    # the other agents' rows do not notice
    Q2 = Q.copy()
    Q2[:, far] = 0.0
    near = np.flatnonzero(~far)
    assert bool((case.pool.attend(_pu().dev(Q2))[:, near] == out[:, near]).all())


# References beyond 60,000 of rows whose block sums are zero: queries of one size and alternating sign, over keys of which a few
# lie along them.  In the 32-row form, the one with 64 shared rows and the one with rows of their own, and with the tails in the
# pool's launch.
@pytest.mark.parametrize("d,heads,agents,q,block_rows,own,tails", [
    (64, 2, 5, 1, 32, 0, False), (128, 2, 5, 1, 32, 0, False), (256, 2, 5, 1, 32, 0, False), (64, 2, 5, 1, 32, 0, True),
    (128, 2, 5, 1, 32, 0, True), (64, 256, 12, 1, 64, 0, False), (128, 256, 12, 1, 64, 0, False), (64, 40, 33, 4, 64, 1, False),
    (128, 40, 33, 4, 64, 1, False), (256, 40, 33, 4, 32, 1, False)])
def test_large_references_alone(d, heads, agents, q, block_rows, own, tails):
    rng = np.random.default_rng(3 * d + agents)
    T, group = 32 * 9 + 5, 4
    half = lambda *s: rng.standard_normal(s).astype(np.float16)
    sign = np.where(np.arange(d) % 2 == 0, 1.0, -1.0)
    K = rng.standard_normal((1, heads, T, d))
    K[:, :, 7::50] += (20.0 + 3.0 * np.arange(6))[:, None] * sign
    Q = rng.standard_normal((1, agents, q, heads * group, d))
    far = np.zeros(agents, bool)
    far[1::3] = True
    Q[:, far] = 200.0 * sign
    K, Q = K.astype(np.float16), Q.astype(np.float16)
    base2 = d ** -0.5 / np.log(2.0)
    assert np.abs(128.0 * base2 * Q[:, far].astype(np.float64).reshape(-1, d // 32, 32).sum(-1)).max() == 0.0
    assert (200.0 * sign * K[0, 0, 257].astype(np.float64)).sum() * base2 > 60000.0     # (the largest of the six)
    case = Case(W.PoolConfig(0, "references", 1, heads, heads * group, d, T, agents, q), K, half(1, heads, T, d))
    kw, gpu_kw = {}, {}
    if tails:
        lens = [3 + 2 * a for a in range(agents)]
        pairs = [(half(1, heads, 20, d), half(1, heads, 20, d)) for _ in lens]
        kw = dict(tails_np=pairs, tails_len=lens, splits=2)
        gpu_kw = dict(tails=[(_pu().dev(k), _pu().dev(v), n) for (k, v), n in zip(pairs, lens)], splits=2)
    choice = case.pool.attend_plan(_pu().dev(Q), **gpu_kw)
    assert (choice.block_rows, choice.own_rows, choice.tails_in_pool_launch) == (block_rows, own, int(tails))
    case.pool.attend(_pu().dev(Q + np.float16(300.0)), **gpu_kw)    # (leaves other numbers in the LDS)
    case.attend_check(Q, **kw)
    out = case.pool.attend(_pu().dev(Q), **gpu_kw)
    # the other agents' rows do not notice
    Q2 = Q.copy()
    Q2[:, far] = 0.0
    near = np.flatnonzero(~far)
    assert bool((case.pool.attend(_pu().dev(Q2), **gpu_kw)[:, near] == out[:, near]).all())


@pytest.mark.parametrize("codec", [dict(), dict(value_bits=2), dict(key_per_tensor=True)])
@pytest.mark.parametrize("d,heads,agents,q,block_rows,own", [
    (64, 2, 5, 1, 32, 0), (64, 256, 12, 1, 64, 0), (128, 256, 12, 1, 64, 0), (256, 256, 5, 1, 32, 0), (64, 40, 33, 4, 64, 1)])
def test_other_agents_references_do_not_show(d, heads, agents, q, block_rows, own, codec):
    """Some agents' rows outgrow their reference in every tile, and the wave forms the tile's probabilities and sums anew; the
    others' rows come out bit for bit as they do beside rows that never move theirs."""
    rng = np.random.default_rng(d + agents)
    T, group = 32 * (9 if own else 25) + 7, 4
    K = rng.standard_normal((1, heads, T, d))
    K[..., 0] = 0.05 * np.arange(T)
    Q = 3.0 * rng.standard_normal((1, agents, q, heads * group, d))     # sums of large and small terms, whose order shows
    Q[..., 0] = 0.17 * d ** 0.5
    far = np.zeros(agents, bool)
    far[1::3] = True
    Q[:, far, ..., 0] = 20.0 * d ** 0.5         # by 46 in 32 tokens
    half = lambda x: _pu().dev(x.astype(np.float16))
    pool = _pu().gpu_pool(K.astype(np.float16), rng.standard_normal(K.shape).astype(np.float16), **codec)
    choice = pool.attend_plan(half(Q), splits=1 if own == 0 else 0)
    assert (choice.block_rows, choice.own_rows) == (block_rows, own)
    out = pool.attend(half(Q), splits=1 if own == 0 else 0)
    Q[:, far] = 0.0
    near = np.flatnonzero(~far)
    assert bool((pool.attend(half(Q), splits=1 if own == 0 else 0)[:, near] == out[:, near]).all())


# The 64-row form with shared rows at head_dim 64, of which two workgroups share a CU: it takes 256 workgroups and more.
def _two_a_cu(T, growing, **codec):
    rng = np.random.default_rng(T)
    K = rng.standard_normal((1, 256, T, 64))
    if growing:
        K *= np.linspace(0.2, 9.0, T)[None, None, :, None]
    V = rng.standard_normal((1, 256, T, 64))
    case = Case(W.PoolConfig(0, "two", 1, 256, 1024, 64, T, 10, 1), K.astype(np.float16), V.astype(np.float16), **codec)
    return case, rng.standard_normal((1, 10, 1, 1024, 64)).astype(np.float16)


def _plan_of(case, Q, **kw):
    choice = case.pool.attend_plan(_pu().dev(Q), **kw)
    return choice.block_rows, choice.own_rows, choice.splits


@pytest.mark.parametrize("tiles", [1, 4, 5, 8, 13, 16, 20, 25, 28])
def test_tiles_per_wave_with_two_workgroups_a_cu(tiles):
    case, Q = _two_a_cu(32 * tiles - {0: 0, 1: 31, 2: 1}[tiles % 3], growing=tiles % 2 == 0)
    assert _plan_of(case, Q) == (64, 0, 1)
    case.attend_check(Q)


@pytest.mark.parametrize("codec", [dict(), dict(value_bits=2), dict(key_per_tensor=True), dict(value_bits=2, key_per_tensor=True)])
def test_codecs_with_two_workgroups_a_cu(codec):
    case, Q = _two_a_cu(32 * 17 + 5, growing=True, **codec)
    for splits in (1, 2):
        assert _plan_of(case, Q, splits=splits) == (64, 0, splits)
        case.attend_check(Q, splits=splits)
    case.attend_check(Q[:, :9], splits=1)      # 36 rows


def test_fp16_keys_with_two_workgroups_a_cu():
    pk, pu = _pk(), _pu()
    case, Q = _two_a_cu(32 * 17 + 5, growing=True)
    kw = dict(key_precision=pk.KEY_PRECISION_FP16)
    assert _plan_of(case, Q, **kw) == (64, 0, 1)
    Kh, Vh = case.decoded()
    pu.compare_attend(case.pool.attend(pu.dev(Q), **kw), O.pool_attend(O.keys_as_fp16(Kh), Vh, Q), 256)
