"""Private tails against the oracle at the edges of the wave's blocks: lengths around its 16-token tiles and 64- (head_dim
256: 32-) token rounds, agents with more and with fewer rows than the four of a wave, causal steps, with the token range
whole (tails in a launch of their own), split (tails in the pool's launch) and on the vector kernel; what lies past a
tail's end is NaN and must not be seen."""
import numpy as np
import pytest

from oracle import polykv_oracle as O
from paper_2604_24971_amd import workloads as W
from test_gpu_parity import Case, _pk, _pu

pytestmark = pytest.mark.gpu

LENGTHS = [0, 1, 15, 16, 17, 31, 32, 33, 48, 63, 64, 65, 95, 128, 130]


@pytest.mark.parametrize("d,group,nq,codec", [
    (64, 1, 1, {}), (64, 3, 2, {}), (128, 4, 1, {}), (128, 5, 1, dict(scaled_values=True)), (128, 2, 4, dict(int8_values=True)),
    (256, 2, 1, {}), (256, 3, 2, {})])
def test_tail_lengths_and_rows(d, group, nq, codec):
    pk, pu = _pk(), _pu()
    rng = np.random.default_rng(d + 10 * group + nq)
    H, T, A, cap = 2, 32 * 33 + 7, len(LENGTHS), 133
    cfg = W.PoolConfig(0, "tails", 2, H, H * group, d, T, A, nq)
    half = lambda *s: rng.standard_normal(s).astype(np.float16)
    # (few pool tokens matter: their keys are short, so that the tails carry most of the weight)
    case = Case(cfg, (0.1 * half(2, H, T, d)).astype(np.float16), half(2, H, T, d), **codec)
    tails = []
    for n in LENGTHS:
        K, V = half(2, H, cap, d) * np.float16(2), half(2, H, cap, d)
        K[:, :, n:] = V[:, :, n:] = np.nan
        tails.append((K, V))
    Q = half(2, A, nq, H * group, d)
    for kw in (dict(), dict(splits=1), dict(splits=3), dict(kernel=pk.KERNEL_VECTOR)):
        case.attend_check(Q, tails_np=tails, tails_len=LENGTHS, **kw)
    case.attend_check(Q[1:], tails_np=tails, tails_len=LENGTHS, layer_begin=1, layer_end=2)
    if nq > 1:
        Kh, Vh = case.decoded()
        ref = [(k[:, :, :n], v[:, :, :n]) for (k, v), n in zip(tails, LENGTHS)]
        gpu = [(pu.dev(k), pu.dev(v), n) for (k, v), n in zip(tails, LENGTHS)]
        want = O.pool_attend(Kh, Vh, Q, tails=ref, tail_causal=True)
        atol = pu.attend_row_atol(Kh, Vh, Q, tails=ref) if codec else pu.ATTEND_ATOL
        for splits in (1, 3):
            out = case.pool.attend(pu.dev(Q), tails=gpu, tail_causal=True, splits=splits)
            pu.compare_attend(out, want, H, case.dirty, 0, atol=atol)


@pytest.mark.parametrize("d,group,nq,bf16,fp16_keys", [
    (64, 1, 1, True, False), (64, 3, 2, True, True), (64, 2, 1, False, True), (128, 4, 1, True, False), (128, 2, 3, True, True),
    (128, 4, 1, False, True), (256, 2, 1, True, False), (256, 3, 2, True, False)])
def test_tails_of_bfloat16_and_beside_keys_as_fp16(d, group, nq, bf16, fp16_keys):
    pk, pu = _pk(), _pu()
    rng = np.random.default_rng(d + 10 * group + nq + bf16)
    H, T, A, cap = 2, 32 * 33 + 7, len(LENGTHS), 133
    rnd = (lambda x: W.bf16_round(x.astype(np.float32))) if bf16 else (lambda x: x.astype(np.float16))
    draw = lambda *s: rng.standard_normal(s)
    K, V, Q = rnd(0.1 * draw(2, H, T, d)), rnd(draw(2, H, T, d)), rnd(draw(2, A, nq, H * group, d))
    pool = pu.gpu_pool(K, V, bf16=bf16)
    ref = O.pool_encode(K, V)
    pu.compare_codes(pool, ref)
    Kh, Vh = O.pool_decode(ref)
    if fp16_keys:
        Kh = O.keys_as_fp16(Kh)
    tails = []
    for n in LENGTHS:
        k, v = rnd(2 * draw(2, H, cap, d)), rnd(draw(2, H, cap, d))
        k[:, :, n:] = v[:, :, n:] = np.nan
        tails.append((k, v))
    gpu = [(pu.dev(k, bf16), pu.dev(v, bf16), n) for (k, v), n in zip(tails, LENGTHS)]
    cut = [(k[:, :, :n], v[:, :, :n]) for (k, v), n in zip(tails, LENGTHS)]
    for causal in (False, True) if nq > 1 else (False,):
        want = O.pool_attend(Kh, Vh, Q, tails=cut, tail_causal=causal)
        for splits in (1, 3):     # in a launch of their own, in the pool's
            kw = dict(tails=gpu, tail_causal=causal, splits=splits,
                      key_precision=pk.KEY_PRECISION_FP16 if fp16_keys else pk.KEY_PRECISION_EXACT)
            assert pool.attend_plan(pu.dev(Q, bf16), **kw).tails_in_pool_launch == (splits > 1 and d != 256)
            out = pool.attend(pu.dev(Q, bf16), **kw)
            pu.compare_attend(out, want, H)
