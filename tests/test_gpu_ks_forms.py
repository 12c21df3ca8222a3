"""The forms of key switching that larger calls take, word for word: the inner
product with two and with eight steps of loads in flight, the division by P
inside the transform, and general primes; with one to seven digits, without any
(the first step of a Z_P chain) and with the plaintext term, for several chains
that share their inputs.

The Z_P reference composes the oracle's rotation with products by arbitrary
NTT-form words, the plaintext term being x*w*(-P)^-1 mod q; x, w and the keys
have words at their ends.  At N = 1024 every call takes one workgroup a
polynomial, and the count of ciphertexts alone chooses the form: workgroups of
the inner product up to 256 (eight steps ahead), the sums mod the q_l from 256
on (the division inside)."""
import numpy as np
import pytest

import oracle
import synth
from synth import Stream
from tests.gpu_util import empty_words, require_gpu, to_dev, to_host
from tests.libload import ensure_built
from tests.test_gpu_ntt_forms import context, prime_below

pytestmark = pytest.mark.gpu
N = 1024


def setup(kind, L):
    """Extended context of L + 1 primes, oracle parameters of the first L, P."""
    if kind == "outside":
        ext, prm_all = context(kind, N)
        q = prm_all.q
        assert L + 1 == len(q)
    else:
        require_gpu()
        ensure_built()
        from paper_2506_11586_amd import heconv
        q = [prime_below(2 ** 60, N, i) for i in range(L + 1)]
        ext = heconv.Context(N, q)
    return ext, oracle.Params(N, L, 60, 2 ** 20, q=q[:L]), q[L]


def key(L, qs, seed):
    """A key of arbitrary NTT-form words, one component's rows all at the top,
    and its coefficient form for the oracle."""
    k = synth.uniform_mod(Stream(seed, synth.UNIFORM), (L, 2, L + 1, N), qs)
    k[:, 0, :, : N // 2] = np.array(qs, dtype=np.uint64)[:, None] - np.uint64(1)
    return k


def reference(x, w, per, G, g, ksk, g2, ksk2, prm, P):
    """One input ciphertext x [2][L][N] (NTT form) through the chains."""
    q = np.array(prm.q, dtype=object)[:, None]
    inv = np.array([pow(-P, -1, v) for v in prm.q], dtype=object)[:, None]
    add = lambda a, b: ((a.astype(object) + b.astype(object)) % q).astype(np.uint64)

    def term(i):
        return oracle.intt((x.astype(object) * w[i].astype(object) * inv % q).astype(np.uint64), prm)[None]

    chains = []
    for c in range(G):
        acc = term(c * per + per - 1)
        for i in range(per - 2, -1, -1):
            acc = add(oracle.rotate(acc, g, ksk, prm, P), term(c * per + i))
        chains.append(acc)
    acc = chains[G - 1]
    for c in range(G - 2, -1, -1):
        acc = add(oracle.rotate(acc, g2, ksk2, prm, P), chains[c])
    return acc[0]


# (L, n, groups, steps): n * groups ciphertexts in each step
ZP = [(2, 10, 4, 3),   # 40: eight steps ahead
      (2, 13, 4, 3),   # 52: two
      (2, 17, 4, 3),   # 68: the division inside, three terms
      (3, 8, 4, 2),    # 32: exactly 256 workgroups
      (3, 10, 4, 2),   # 40
      (3, 11, 4, 3),   # 44: four terms
      (1, 32, 4, 3),   # 128: two terms, one digit
      (1, 21, 4, 2),   # 84
      (4, 8, 4, 2),    # 32: five terms
      (4, 5, 2, 2),    # 10
      (7, 10, 2, 2),   # 20: eight terms
      (7, 2, 2, 2)]    # 4


def run_zp(kind, L, n, G, per):
    ext, prm, P = setup(kind, L)
    qs = prm.q + [P]
    D, g, g2 = per * G, 5, 25
    top = np.array(prm.q, dtype=np.uint64)[:, None] - np.uint64(1)
    x = synth.uniform_mod(Stream(201, synth.UNIFORM), (n, 2, L, N), prm.q)
    w = synth.uniform_mod(Stream(202, synth.UNIFORM), (D, L, N), prm.q)
    x[0], w[0], w[-1, :, ::2] = top, top, 0
    k1, k2 = key(L, qs, 203), key(L, qs, 204)
    dx, dw, d1, d2 = to_dev(x), to_dev(w), to_dev(k1), to_dev(k2)
    out = empty_words(x.size)
    ext.zp_matvec_grouped(g, n, dx, dw, D, G, d1, g2, d2, out, empty_words(ext.zp_grouped_work_words(n, G)))
    got = to_host(out).reshape(x.shape)
    ex = oracle.ext_params(prm, P)
    c1, c2 = oracle.intt(k1, ex), oracle.intt(k2, ex)
    for j in sorted({0, n - 1}):
        assert np.array_equal(got[j], reference(x[j], w, per, G, g, c1, g2, c2, prm, P)), j
    # every other ciphertext as it comes out alone
    one = empty_words(x[0].size)
    for j in range(n):
        ext.zp_matvec_grouped(g, 1, to_dev(x[j]), dw, D, G, d1, g2, d2, one,
                              empty_words(ext.zp_grouped_work_words(1, G)))
        assert np.array_equal(to_host(one).reshape(x[0].shape), got[j]), j


@pytest.mark.parametrize("L,n,G,per", ZP)
def test_zp_chains_in_every_form(L, n, G, per):
    run_zp("near", L, n, G, per)


@pytest.mark.parametrize("n,G,per", [(1, 1, 3), (10, 4, 2), (17, 4, 3)])
def test_zp_chains_with_general_primes(n, G, per):
    run_zp("outside", 2, n, G, per)


@pytest.mark.parametrize("L,n", [(1, 127), (1, 128), (2, 63), (3, 43), (4, 31), (4, 33), (5, 26), (7, 18), (7, 19)])
def test_rotation_in_every_form(L, n):
    """Rotation, rotate-and-add and a key switch in place against the separate
    steps, the first and the last ciphertext against the oracle."""
    ext, prm, P = setup("near", L)
    k = key(L, prm.q + [P], 205)
    dk = to_dev(k)
    ct = synth.uniform_mod(Stream(206, synth.UNIFORM), (n, 2, L, N), prm.q)
    ct[0] = np.array(prm.q, dtype=np.uint64)[:, None] - np.uint64(1)
    work = empty_words(ext.keyswitch_work_words(n))
    outs = []
    for mode in (1, 0):
        ext.set_tuning(ks_fused=mode)
        dct, rot, fold = to_dev(ct), empty_words(ct.size), empty_words(ct.size)
        ext.rotate(5, n, dct, dk, rot, work)
        ext.zp_fold(2 * N - 1, n, dct, dk, fold, work)
        ext.keyswitch(n, dct, dk, dct, work)
        outs.append([to_host(t).reshape(ct.shape).copy() for t in (rot, fold, dct)])
    for a, b in zip(*outs):
        assert np.array_equal(a, b)
    ends = [0, n - 1]
    want = oracle.rotate(ct[ends], 5, oracle.intt(k, oracle.ext_params(prm, P)), prm, P)
    assert np.array_equal(outs[0][0][ends], want)


@pytest.mark.parametrize("n8,L,n,G", [(8192, 3, 8, 8), (8192, 3, 8, 4), (4096, 2, 9, 4), (2048, 2, 10, 4)])
def test_zp_at_served_sizes(n8, L, n, G):
    """64-bit words of larger rings: n inputs through G chains at once (the
    division inside from 64 ciphertexts at N = 8192 on, else the plain inner
    product), each input as it comes out alone, where N >= 4096 takes the small
    grids."""
    require_gpu()
    ensure_built()
    from paper_2506_11586_amd import heconv
    per = 3
    q = heconv.gen_primes(n8, 60, L + 1)
    ext = heconv.Context(n8, q)
    x = synth.uniform_mod(Stream(211, synth.UNIFORM), (n, 2, L, n8), q[:L])
    dw = to_dev(synth.uniform_mod(Stream(212, synth.UNIFORM), (per * G, L, n8), q[:L]))
    d1, d2 = (to_dev(synth.uniform_mod(Stream(s, synth.UNIFORM), (L, 2, L + 1, n8), q)) for s in (213, 214))
    out, one = empty_words(x.size), empty_words(x[0].size)
    ext.zp_matvec_grouped(5, n, to_dev(x), dw, per * G, G, d1, 25, d2, out, empty_words(ext.zp_grouped_work_words(n, G)))
    got = to_host(out).reshape(x.shape)
    for j in range(n):
        ext.zp_matvec_grouped(5, 1, to_dev(x[j]), dw, per * G, G, d1, 25, d2, one,
                              empty_words(ext.zp_grouped_work_words(1, G)))
        assert np.array_equal(to_host(one).reshape(x[0].shape), got[j]), j
