"""he_add_share and he_mask_extract word for word against the oracle at the
edges of their reduction mod t and of their index arithmetic: the smallest and
largest t, odd ones, int64's extremes; tiles of one column or row, one output
position, counts just off a whole workgroup."""
import numpy as np
import pytest

import oracle
import synth
from synth import Stream
from tests.gpu_util import empty_words, to_dev, to_host
from tests.test_gpu_protocol import ctx_and_prm, _desc

pytestmark = pytest.mark.gpu

I64 = np.iinfo(np.int64)
TS = [2, 3, 65537, 2 ** 37 - 1, 2 ** 61 + 1, 2 ** 62 - 57, 2 ** 62]
SHAPES = [(1, 1, 1, 1, 1, 1, 0), (2, 16, 16, 1, 3, 1, 1), (1, 3, 257, 2, 1, 1, 0), (3, 65, 1, 2, 1, 2, 0),
          (2, 5, 51, 3, 3, 2, 1)]


def values(seed, n, t):
    v = Stream(seed, synth.SHARE).words(n).view(np.int64).copy()
    edge = np.array([I64.min, I64.max, I64.min + 1, 0, -1, t, -t, t - 1, 1 - t, 2 * t - 1, I64.max // t * t,
                     -(I64.max // t * t)], dtype=object)
    edge = np.clip(edge, I64.min, I64.max).astype(np.int64)
    v[: min(n, len(edge))] = edge[:n]
    return v


@pytest.mark.parametrize("t,shape", [(t, SHAPES[1]) for t in TS] + [(2 ** 37, s) for s in SHAPES])
def test_protocol_edges(t, shape):
    ctx, prm = ctx_and_prm(1024, 2, 50, t)
    d, cv = _desc(ctx, shape)
    g = oracle.geometry(cv, d.Cw, d.Hw, d.Ww)
    B = 3
    ct = synth.uniform_mod(Stream(61, synth.UNIFORM), (B, g.CB, g.S, 2, prm.L, prm.N), prm.q)
    xs = values(61, B * cv.C * cv.H * cv.W, t).reshape(B, cv.C, cv.H, cv.W)
    dev = to_dev(ct)
    ctx.add_share(d, B, dev, to_dev(xs))
    got = to_host(dev).reshape(ct.shape)
    out = synth.uniform_mod(Stream(62, synth.UNIFORM), (B, cv.M, g.S, 2, prm.L, prm.N), prm.q)
    R = values(62, B * cv.M * g.Ho * g.Wo, t).reshape(B, cv.M, g.Ho, g.Wo)
    e = values(63, R.size, prm.q[0]).reshape(R.shape)
    y = empty_words(R.size * prm.L)
    ctx.mask_extract(d, B, to_dev(out), to_dev(R), to_dev(e), y)
    got_y = to_host(y).reshape(B, cv.M, prm.L, g.Ho, g.Wo)
    for b in range(B):
        assert np.array_equal(got[b], oracle.add_share(ct[b], xs[b], cv, g, prm)), b
        assert np.array_equal(got_y[b], oracle.mask_extract(out[b], R[b], e[b], cv, g, prm)), b
