"""GPU parity of both forms of the integer transforms: the signed one (every
prime 2^b - delta, delta < 2^24) and the general one, which a single prime
outside the form selects for its whole context.  NTT, inverse NTT (one grid
with 8 and 16 words per thread, two grids) and rotation, word for word
against the oracle, with words at the ends of their ranges."""
import numpy as np
import pytest

import oracle
import synth
from synth import Stream
from tests import workload as wl
from tests.gpu_util import empty_words, require_gpu, to_dev, to_host
from tests.libload import ensure_built

pytestmark = pytest.mark.gpu


def prime_below(top, N, skip=0):
    """The largest prime at most `top` that is 1 mod 2N, after `skip` others."""
    c = (top - 1) // (2 * N) * (2 * N) + 1
    while True:
        if oracle.is_prime(c):
            if skip == 0:
                return c
            skip -= 1
        c -= 2 * N


def primes_of(kind, N):
    if kind == "near":  # the signed form at its common end
        return oracle.find_primes(N, 60, 3)
    if kind == "delta24":  # the largest delta it takes, beside the smallest
        return [prime_below(2 ** 60 - 2 ** 23 - 2 ** 22, N), prime_below(2 ** 60, N), prime_below(2 ** 55, N)]
    if kind == "outside":  # one prime outside the form: the whole context is general
        return [prime_below(2 ** 60, N), prime_below(2 ** 60 - 2 ** 24, N), prime_below(2 ** 59 + 2 ** 57, N)]
    raise ValueError(kind)


def context(kind, N):
    require_gpu()
    ensure_built()
    from paper_2506_11586_amd import heconv
    q = primes_of(kind, N)
    return heconv.Context(N, q), oracle.Params(N, len(q), 60, 2 ** 37, q=q)


@pytest.mark.parametrize("kind", ["near", "delta24", "outside"])
@pytest.mark.parametrize("N", [1024, 2048, 4096, 8192, 16384])
def test_transforms_in_both_forms(N, kind):
    ctx, prm = context(kind, N)
    n = 3
    x = synth.uniform_mod(Stream(N, synth.UNIFORM), (n, prm.L, N), prm.q)
    top = np.array(prm.q, dtype=np.uint64)[:, None] - np.uint64(1)
    x[0] = top
    x[1, :, ::2], x[1, :, 1::2] = top, 0  # alternating ends: the largest differences
    fwd, inv = oracle.ntt(x, prm), oracle.intt(x, prm)
    for loge in (3, 4):
        for split in (0, 1 << 30):
            ctx.set_tuning(ntt_loge_small=loge, ntt_loge_large=loge, ntt_fp64=0, ntt_split_below=split,
                           ntt_inv_split_below=split)
            d = to_dev(x)
            ctx.ntt_fwd(d, n)
            assert np.array_equal(to_host(d).reshape(x.shape), fwd), (loge, split)
            ctx.ntt_inv(d, n)
            assert np.array_equal(to_host(d).reshape(x.shape), x), (loge, split)
            d = to_dev(x)
            ctx.ntt_inv(d, n)
            assert np.array_equal(to_host(d).reshape(x.shape), inv), (loge, split)


@pytest.mark.parametrize("bits", [50, 40])
@pytest.mark.parametrize("N", [1024, 2048, 4096, 8192, 16384])
def test_double_precision_transforms(N, bits):
    """The fp64 transforms on words whose sums and differences are the
    largest: all at the top, alternating ends in runs of every length."""
    require_gpu()
    ensure_built()
    from paper_2506_11586_amd import heconv
    q = oracle.find_primes(N, bits, 2)
    ctx, prm = heconv.Context(N, q), oracle.Params(N, 2, bits, 2 ** 20, q=q)
    top = np.array(q, dtype=np.uint64)[:, None] - np.uint64(1)
    runs = [0, 1, 2, 3, N.bit_length() - 2]
    x = synth.uniform_mod(Stream(N + 1, synth.UNIFORM), (len(runs) + 2, 2, N), q)
    x[0] = top
    for i, r in enumerate(runs):
        x[i + 1] = np.where((np.arange(N) >> r) & 1, np.uint64(0), top)
    n = x.shape[0]
    fwd, inv = oracle.ntt(x, prm), oracle.intt(x, prm)
    for loge in (3, 4):
        ctx.set_tuning(ntt_loge_small=loge, ntt_loge_large=loge, ntt_fp64=1)
        d = to_dev(x)
        ctx.ntt_fwd(d, n)
        assert np.array_equal(to_host(d).reshape(x.shape), fwd), loge
        ctx.ntt_inv(d, n)
        assert np.array_equal(to_host(d).reshape(x.shape), x), loge
        d = to_dev(x)
        ctx.ntt_inv(d, n)
        assert np.array_equal(to_host(d).reshape(x.shape), inv), loge


@pytest.mark.parametrize("kind", ["near", "delta24", "outside"])
@pytest.mark.parametrize("g,fused", [(3, 1), (1, 1), (2 * 1024 - 1, 2)])
def test_rotation_in_both_forms(kind, g, fused):
    """Digits of one prime enter the transforms of the others (with the
    signed form as they are, also where the prime is the smaller)."""
    N = 1024
    ext, prm_all = context(kind, N)
    q, P = prm_all.q[:2], prm_all.q[2]
    prm = oracle.Params(N, 2, 60, 2 ** 37, q=q)
    sk = wl.secret_key(5, N)
    ex = oracle.ext_params(prm, P)
    a = synth.uniform_mod(Stream(6, synth.UNIFORM), (2, 3, N), ex.q)
    e = Stream(6, synth.ERROR).cbd(2 * N, wl.ETA).reshape(2, N)
    ksk = oracle.galois_key(sk, g, a, e, prm, P)
    n = 9
    ct = synth.uniform_mod(Stream(7, synth.UNIFORM), (n, 2, 2, N), q)
    ct[0, 0] = np.array(q, dtype=np.uint64)[:, None] - np.uint64(1)
    dk = to_dev(ksk)
    ext.ntt_fwd(dk, 4)
    ext.set_tuning(ks_fused=fused)
    out = empty_words(ct.size)
    ext.rotate(g, n, to_dev(ct), dk, out, empty_words(ext.keyswitch_work_words(n)))
    assert np.array_equal(to_host(out).reshape(ct.shape), oracle.rotate(ct, g, ksk, prm, P))


@pytest.mark.parametrize("g", [1, 5])
def test_division_by_P_inside_the_transform(g):
    """A call large enough for the fused division by P: every ciphertext
    against the same words rotated in a call too small for it, and the first
    and the last against the oracle (digits and b words at their ends too)."""
    N = 1024
    ext, prm_all = context("near", N)
    q, P = prm_all.q[:2], prm_all.q[2]
    prm = oracle.Params(N, 2, 60, 2 ** 37, q=q)
    sk = wl.secret_key(15, N)
    a = synth.uniform_mod(Stream(16, synth.UNIFORM), (2, 3, N), prm_all.q)
    e = Stream(16, synth.ERROR).cbd(2 * N, wl.ETA).reshape(2, N)
    ksk = oracle.galois_key(sk, g, a, e, prm, P)
    n = 64 + 3  # from 64 on the division rides on the transform (256 workgroups of two digits and components)
    ct = synth.uniform_mod(Stream(17, synth.UNIFORM), (n, 2, 2, N), q)
    top = np.array(q, dtype=np.uint64)[:, None] - np.uint64(1)
    ct[0] = top
    ct[-1, 0], ct[-1, 1] = 0, top
    dk = to_dev(ksk)
    ext.ntt_fwd(dk, 4)
    dct, out = to_dev(ct), empty_words(ct.size)
    ext.rotate(g, n, dct, dk, out, empty_words(ext.keyswitch_work_words(n)))
    got = to_host(out).reshape(ct.shape)
    step = 32
    for i in range(0, n, step):
        m = min(step, n - i)
        part, small = to_dev(ct[i:i + m]), empty_words(ct[i:i + m].size)
        ext.rotate(g, m, part, dk, small, empty_words(ext.keyswitch_work_words(m)))
        assert np.array_equal(got[i:i + m], to_host(small).reshape(ct[i:i + m].shape)), i
    ends = [0, n - 1]
    assert np.array_equal(got[ends], oracle.rotate(ct[ends], g, ksk, prm, P))
    # rotate-and-add on the same path
    ext.zp_fold(g, n, dct, dk, out, empty_words(ext.keyswitch_work_words(n)))
    fold = to_host(out).reshape(ct.shape).astype(object)
    want = (got.astype(object) + ct.astype(object)) % np.array(q, dtype=object)[:, None]
    assert np.array_equal(fold, want)


@pytest.mark.parametrize("kind", ["near", "delta24", "outside"])
@pytest.mark.parametrize("C,M,B,grid", [(3, 5, 1, 0), (8, 9, 4, 1), (9, 8, 5, 1), (17, 17, 4, 0)])
def test_mac_folds(kind, C, M, B, grid):
    """The streamed MAC with each of its folds: channel blocks below, at and
    above one chunk, the wave grid and the per-wave form, remainders of rows
    and channels, words at their ends."""
    N = 1024
    ctx, prm = context(kind, N)
    ctx.set_tuning(mac_grid=grid)
    cv = wl.conv_of((C, 8, 8, M, 3, 3, 1, 1))
    d = ctx.plan((C, 8, 8, M, 3, 3, 1, 1), batch=B, packing=(1, 10, 10))
    g = oracle.geometry(cv, 1, 10, 10)
    assert g.CB == C and g.S == 1
    top = np.array(prm.q, dtype=np.uint64)[:, None] - np.uint64(1)
    x = synth.uniform_mod(Stream(31, synth.UNIFORM), (B * C * 2, 3, N), prm.q)
    w = synth.uniform_mod(Stream(32, synth.UNIFORM), (M * C, 3, N), prm.q)
    x[:C * 2], w[:C] = top, top  # image 0 and channel 0: every product the largest
    out = empty_words(B * M * 2 * 3 * N)
    ctx.conv_ntt_mac(d, B, to_dev(x), to_dev(w), out)
    want = oracle.conv_mac(x.reshape(B, C, 1, 2, 3, N), w.reshape(M, C, 3, N), B, g, M, prm)
    assert np.array_equal(to_host(out).reshape(want.shape), want)
