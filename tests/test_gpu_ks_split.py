"""Key switching of a few ciphertexts (the three small grids), word for word:
against the oracle at one and two ciphertexts, for every ring the grids take
and 1 to 7 digits, with the addend; and against the separate-steps form (itself
checked against the oracle) in place, for the reversing automorphism and around
the count where the one-workgroup transforms take over."""
import numpy as np
import pytest

import oracle
import synth
from synth import Stream
from tests import workload as wl
from tests.gpu_util import empty_words, to_dev, to_host
from tests.test_gpu_rotation import contexts, key_to_dev, make_key

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,L,bits,n", [(4096, 2, 60, 1), (4096, 3, 60, 2), (8192, 2, 60, 2), (8192, 4, 55, 1),
                                        (4096, 7, 60, 1), (4096, 1, 54, 2), (16384, 2, 60, 1)])
def test_few_ciphertexts_match_oracle(N, L, bits, n):
    base, ext, prm, P = contexts(N, L, bits)
    ext.set_tuning(ks_fused=1)
    sk = wl.secret_key(171, N)
    ksk = make_key(prm, P, sk, 5, 172)
    dk = key_to_dev(ext, prm, ksk)
    ct = synth.uniform_mod(Stream(173, synth.UNIFORM), (n, 2, L, N), prm.q)
    ct[0, 0, :, :3] = np.array(prm.q, dtype=np.uint64)[:, None] - 1  # largest digits
    ct[-1, 0, :, 3:9] = 0
    work = empty_words(ext.keyswitch_work_words(n))
    out = empty_words(ct.size)
    ext.rotate(5, n, to_dev(ct), dk, out, work)
    rot = oracle.rotate(ct, 5, ksk, prm, P)
    assert np.array_equal(to_host(out).reshape(rot.shape), rot)
    ext.zp_fold(5, n, to_dev(ct), dk, out, work)
    q = np.array(prm.q, dtype=object)[:, None]
    assert np.array_equal(to_host(out).reshape(rot.shape), ((ct.astype(object) + rot) % q).astype(np.uint64))
    got = []
    for mode in (1, 0):
        ext.set_tuning(ks_fused=mode)
        ext.rotate(2 * N - 1, n, to_dev(ct), dk, out, work)
        got.append(to_host(out).copy())
        dct = to_dev(ct)
        ext.keyswitch(n, dct, dk, dct, work)
        got.append(to_host(dct).copy())
    ext.set_tuning(ks_fused=1)
    assert np.array_equal(got[0], got[2]) and np.array_equal(got[1], got[3])


@pytest.mark.parametrize("N,L,bits", [(4096, 2, 50), (8192, 3, 60), (8192, 4, 55), (16384, 2, 60)])
def test_counts_match_separate_steps(N, L, bits):
    base, ext, prm, P = contexts(N, L, bits)
    dk = to_dev(synth.uniform_mod(Stream(181, synth.UNIFORM), (L, 2, L + 1, N), prm.q + [P]))
    for n in (1, 3, 7, 8, 9, 15, 16, 17, 31, 33):
        ct = to_dev(synth.uniform_mod(Stream(182 + n, synth.UNIFORM), (n, 2, L, N), prm.q))
        work = empty_words(ext.keyswitch_work_words(n))
        outs = []
        for mode in (1, 0):
            ext.set_tuning(ks_fused=mode)
            o = empty_words(ct.numel())
            ext.rotate(25, n, ct, dk, o, work)
            outs.append(to_host(o))
        ext.set_tuning(ks_fused=1)
        assert np.array_equal(outs[0], outs[1]), n
