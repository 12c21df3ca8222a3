"""Encryption and decryption at N = 2^14 on both sides of the line between the
split transforms in separate steps and the one-kernel product, word for word
against the oracle.  Which form ran shows in the scratch buffer: the steps leave
a*sk there; the one-kernel form leaves it alone in encryption and b - a*sk in
decryption.  With a few limb polynomials the one-kernel form took 1.4 to 1.5
times as long."""
import numpy as np
import pytest

import oracle
import synth
from synth import Stream
from tests import workload as wl
from tests.gpu_util import empty_words, to_dev, to_host
from tests.test_gpu_client import ctx_and_prm, key_ntt

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,n,steps", [(2, 1, True), (4, 10, True), (3, 14, False)])
def test_forms_at_ring_16384(L, n, steps):
    N = 16384
    ctx, prm = ctx_and_prm(N, L, 60)
    sk = wl.secret_key(71, N)
    msgs = Stream(71, synth.INPUT).below(n * N, prm.t).reshape(n, N)
    a = synth.uniform_mod(Stream(71, synth.UNIFORM), (n, L, N), prm.q)
    e = Stream(71, synth.ERROR).cbd(n * N, wl.ETA).reshape(n, N)
    want = oracle.bfv_encrypt(msgs, sk, a, e, prm)
    skn = key_ntt(ctx, prm, sk)
    zero = np.zeros((n, N), dtype=np.int64)
    a_sk = oracle.bfv_encrypt(zero.astype(np.uint64), sk, a, zero, prm)[:, 1]
    ct, work, dec = empty_words(want.size), to_dev(np.zeros((n, L, N), dtype=np.int64)), empty_words(n * N)
    ctx.encrypt(n, to_dev(msgs.astype(np.int64)), to_dev(a), to_dev(e), skn, ct, work)
    assert np.array_equal(to_host(ct).reshape(want.shape), want)
    assert np.array_equal(to_host(work).reshape(a_sk.shape), a_sk if steps else np.zeros_like(a_sk))
    ctx.decrypt(n, ct, skn, dec, work)
    assert np.array_equal(dec.cpu().numpy().reshape(n, N), oracle.centre_mod(msgs.astype(object), prm.t).astype(np.int64))
    q = np.array(prm.q, dtype=object)[:, None]
    phase = ((want[:, 1].astype(object) - a_sk.astype(object)) % q).astype(np.uint64)
    assert np.array_equal(to_host(work).reshape(a_sk.shape), a_sk if steps else phase)
