"""The matrix-core attention kernel's step sequence against the oracle: every number of tiles a wave can be left with
around its two-steps-per-trip loop (none, one, ..., seven), a last tile of one token, of all but one and a full one, and
keys that grow along the context, so that rows keep moving their softmax reference."""
import numpy as np
import pytest

from paper_2604_24971_amd import workloads as W
from test_gpu_parity import Case, _pk

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
