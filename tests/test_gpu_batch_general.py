"""The batch executor and the fused layer with primes outside the signed
transforms' form, word for word against the oracle: 8 and 16 words per thread,
one and two chains."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import empty_words, require_gpu, to_dev, to_host
from tests.libload import ensure_built
from tests.test_gpu_batch import make_jobs
from tests.test_gpu_ntt_forms import context

pytestmark = pytest.mark.gpu

SHAPES = [((4, 12, 12, 5, 3, 3, 1, 1), 2), ((9, 7, 7, 9, 1, 1, 1, 0), 3), ((3, 15, 15, 4, 5, 5, 2, 2), 1)]


def general(N, bits):
    if bits == 40:  # 2^40 - delta with delta * 2^20 above 2^31
        require_gpu()
        ensure_built()
        from paper_2506_11586_amd import heconv
        q = oracle.find_primes(N, 40, 2)
        return heconv.Context(N, q), oracle.Params(N, 2, 40, 2 ** 20, q=q)
    return context("outside", N)


@pytest.mark.parametrize("loge", [3, 4])
@pytest.mark.parametrize("N,bits", [(2048, 40), (1024, 60), (8192, 60)])
def test_batch_and_fused_layer(N, bits, loge):
    from paper_2506_11586_amd import heconv
    ctx, prm = general(N, bits)
    ctx.set_tuning(ntt_loge_small=loge, ntt_loge_large=loge, ntt_fp64=0)
    jobs, host = make_jobs(ctx, prm, SHAPES, 300)
    wants = []
    for (d, B, *_), (cv, _, _, x, K) in zip(jobs, host):
        g = oracle.geometry(cv, d.Cw, d.Hw, d.Ww)
        w_ntt = oracle.encode_weights(K, cv, g, prm)
        wants.append(oracle.conv_layer_ntt(x.reshape(B, g.CB, g.S, 2, prm.L, prm.N), w_ntt, B, g, cv.M, prm))
    for schedule in (1, 2):
        for (_, _, d_in, _, _), (*_, x, _) in zip(jobs, host):
            d_in.copy_(to_dev(x).reshape(d_in.shape))
        b = heconv.Batch(ctx, jobs, schedule=schedule)
        b.launch()
        b.status()
        for (*_, d_out), want in zip(jobs, wants):
            assert np.array_equal(to_host(d_out).reshape(want.shape), want), schedule
        b.close()
    ctx.set_tuning(layer_fused=1)
    for (d, B, _, wntt, _), (*_, x, _), want in zip(jobs, host, wants):
        out = empty_words(want.size)
        ctx.conv_layer(d, B, to_dev(x), wntt, out)
        assert np.array_equal(to_host(out).reshape(want.shape), want)
