"""Timed workloads of the library's public entry points.

listed() gives the fixed workloads, draw() more of the same kinds and ranges;
prepare() builds what a program keeps before the call (context, key,
NTT-form weights, batch, buffers) and its inputs, all from the seed; run() is
one pass and returns every output word.  Calls that transform their input in
place first copy the received ciphertexts into the launch buffer, as the
request server does.  Ciphertext words are uniform residues, as those of
fresh RLWE ciphertexts; weights and messages are small integers.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2506_11586_amd import heconv

T37 = 1 << 37  # the layers' plaintext modulus (37-bit fixed point)

# One bottleneck block of three stages of the batch-16 CNN (1x1 reduce, 3x3, 1x1 expand; the
# last without its expand layer): channels, spatial size, width.
BOTTLENECK = [(256, 56, 64, True), (1024, 14, 256, True), (2048, 7, 512, False)]
# The fire modules of the batch-1 CNN: input channels, spatial size, squeeze, expand.
FIRES = [(64, 55, 16, 64), (128, 55, 16, 64), (128, 27, 32, 128), (256, 27, 32, 128),
         (256, 13, 48, 192), (384, 13, 48, 192), (384, 13, 64, 256), (512, 13, 64, 256)]


def _cnn(net):
    """Layer shapes (C, H, W, M, kh, kw, stride, pad) of a batched network."""
    out = []
    if net == "fire":
        out.append((3, 224, 224, 64, 3, 3, 2, 1))
        for c, hw, sq, ex in FIRES:
            out += [(c, hw, hw, sq, 1, 1, 1, 0), (sq, hw, hw, ex, 1, 1, 1, 0), (sq, hw, hw, ex, 3, 3, 1, 1)]
        out.append((512, 13, 13, 1000, 1, 1, 1, 0))
    elif net == "bottleneck":
        for c, hw, w, expand in BOTTLENECK:
            out += [(c, hw, hw, w, 1, 1, 1, 0), (w, hw, hw, w, 3, 3, 1, 1)]
            if expand:
                out.append((w, hw, hw, c, 1, 1, 1, 0))
    else:  # "CxHxM": one bottleneck block of that width
        c, hw, w = (int(v) for v in net.split("x"))
        out += [(c, hw, hw, w, 1, 1, 1, 0), (w, hw, hw, w, 3, 3, 1, 1), (w, hw, hw, c, 1, 1, 1, 0)]
    return out


def _layer(name, C, HW, M, k, stride=1, B=1, N=8192, L=3, bits=60, kind="layer"):
    return dict(name=name, kind=kind, N=N, L=L, bits=bits, C=C, HW=HW, M=M, k=k, stride=stride, B=B)


def listed():
    return [
        # the smallest layer: latency and launches (double-precision transforms)
        _layer("layer_4ch_16px_n4096", 4, 16, 4, 3, N=4096, L=2, bits=50),
        # one image of a 3x3 layer at 56x56: the single-layer benchmark
        _layer("layer_64ch_56px", 64, 56, 64, 3),
        # a 3x3 layer of the batch-16 CNN in one call of 16 images
        _layer("layer_128ch_28px_b16", 128, 28, 128, 3, B=16),
        # the other parameter sets: ring 2^14, and 50-bit primes at ring 2^12, odd image counts
        _layer("layer_48ch_27px_n16384_b3", 48, 27, 96, 3, N=16384, L=4, B=3),
        _layer("layer_96ch_14px_n4096_b5", 96, 14, 64, 3, N=4096, L=2, bits=50, B=5),
        # a served request group: shares folded in, layer, masked extraction
        _layer("server_step_fire_27px_b7", 32, 27, 128, 3, B=7, kind="server"),
        # whole networks through the batch executor, one graph launch each
        dict(name="batch_fire_cnn_b1", kind="batch", N=8192, L=3, bits=60, net="fire", B=1),
        dict(name="batch_bottleneck_blocks_b16", kind="batch", N=8192, L=3, bits=60, net="bottleneck", B=16),
        # rotation of one ciphertext (latency) and of many (throughput)
        dict(name="rotate_1", kind="rotate", N=8192, L=3, bits=60, n=1, g=5),
        dict(name="rotate_256", kind="rotate", N=8192, L=3, bits=60, n=256, g=5),
        # the Z_P fully connected layer, 2048 -> 1000 on 16 images as 8 chains
        dict(name="zp_fc_2048_1000_b16", kind="zp", N=8192, L=3, bits=60, rows=1000, cols=2048, n=16, groups=8),
        # client side: encrypt and decrypt a batch of messages
        dict(name="client_64", kind="client", N=8192, L=3, bits=60, n=64),
    ]


def _logint(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


PARAMS = [(8192, 3, 60), (8192, 3, 60), (8192, 2, 60), (8192, 4, 55), (4096, 2, 50), (4096, 2, 60), (2048, 1, 54),
          (16384, 4, 60), (16384, 5, 50), (8192, 3, 49)]


def draw(rng):
    kind = rng.choice(["layer", "layer", "layer", "server", "batch", "rotate", "zp", "client"])
    N, L, bits = rng.choice(PARAMS)
    if kind in ("rotate", "client"):
        n = _logint(rng, 1, 256)
        c = dict(kind=kind, N=N, L=max(L, 2), bits=bits, n=n)
        if kind == "rotate":
            c["g"] = pow(5, rng.randrange(1, N // 2), 2 * N)
        return c
    if kind == "zp":
        rows = _logint(rng, 40, 600)
        return dict(kind=kind, N=8192, L=3, bits=60, rows=rows, cols=_logint(rng, rows, 2048), n=_logint(rng, 1, 16),
                    groups=rng.choice([1, 2, 4, 8]))
    while True:
        if kind == "batch":
            hw = _logint(rng, 6, 40)
            w = _logint(rng, 12, 200)
            c = dict(kind=kind, N=8192, L=3, bits=60, net="%dx%dx%d" % (w * rng.choice([2, 3, 4]), hw, w),
                     B=_logint(rng, 1, 16))
        else:
            hw, k = _logint(rng, 6, 60), rng.choice([1, 3, 3, 5])
            c = dict(kind=kind, N=N, L=L, bits=bits, C=_logint(rng, 3, 300), HW=hw, M=_logint(rng, 3, 300), k=k,
                     stride=rng.choice([1, 1, 2]), B=_logint(rng, 1, 16))
        w = work(c)
        if w["bytes"] < 3e9 and w["flops"] < 3e10:
            return c


def _shapes(c):
    if c["kind"] == "batch":
        return _cnn(c["net"])
    return [(c["C"], c["HW"], c["HW"], c["M"], c["k"], c["k"], c["stride"], c["k"] // 2)]


def _planned(c, shape):
    """The planned descriptor with its channel blocks and spatial tiles."""
    C, H, W, M, kh, kw, stride, pad = shape
    d = heconv.plan_host(c["N"], c["L"], shape, c["B"])
    He, We = H + 2 * pad, W + 2 * pad
    if kh == 1 and kw == 1 and stride > 1:
        He, We = -(-He // stride), -(-We // stride)
    S = -(-(He - kh + 1) // (d.Hw - kh + 1)) * -(-(We - kw + 1) // (d.Ww - kw + 1))
    return d, -(-C // d.Cw), S


def work(case):
    c = case
    N, L = c["N"], c["L"]
    poly, ntt = N * 8, 3.0 * (N // 2) * math.log2(N)  # bytes; multiply, add and subtract per butterfly
    if c["kind"] == "rotate":
        n, e = c["n"], L + 1
        return {"bytes": 4 * n * L * poly + 2 * L * e * poly, "flops": n * (L * e + 2 * e) * ntt + 4.0 * n * L * e * N}
    if c["kind"] == "client":
        n = c["n"]  # encrypt: messages, a, errors in, ciphertexts out; decrypt: ciphertexts in, messages out
        return {"bytes": n * poly * (2 + 3 * L) + n * poly * (2 * L + 1), "flops": 4.0 * n * L * ntt}
    if c["kind"] == "zp":
        D, n, e = 1 << (c["rows"] - 1).bit_length(), c["n"], L + 1
        folds = ((c["cols"] - 1).bit_length() - (c["rows"] - 1).bit_length())
        per = n * (L * e + 2 * e) * ntt + n * (4.0 * L * e + 4.0 * L) * N
        return {"bytes": D * L * poly + 4 * n * L * poly + (2 + folds) * 2 * L * e * poly, "flops": (D + folds) * per}
    byt = flo = 0.0
    for shape in _shapes(c):
        d, CB, S = _planned(c, shape)
        B, M = c["B"], d.M
        cts = B * (CB + M) * S
        byt += M * CB * L * poly + cts * 2 * L * poly
        flo += cts * 2 * L * ntt + 2.0 * B * M * S * CB * 2 * L * N
        if c["kind"] == "server":
            ho, wo = heconv.Context.out_hw(d)
            byt += 8.0 * B * (d.C * d.H * d.W + (L + 1) * M * ho * wo)
    return {"bytes": byt, "flops": flo}


class _Rand:
    """Seeded int64 device tensors, drawn in blocks of bounded size."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda").manual_seed(1 + int(seed))

    def ints(self, shape, lo, hi):
        return torch.randint(lo, hi, shape, generator=self.g, dtype=torch.int64, device="cuda")

    def residues(self, shape, q):
        """Words uniform below q[l] on the second last axis."""
        out = torch.empty(shape, dtype=torch.int64, device="cuda")
        for l, v in enumerate(q):
            out[..., l, :].random_(0, v, generator=self.g)
        return out


def _words(*shape):
    return torch.empty(shape, dtype=torch.int64, device="cuda")


def prepare(case, seed):
    c = dict(case)
    rnd = _Rand(seed)
    N, L, kind = c["N"], c["L"], c["kind"]
    s = {"kind": kind, "case": c}
    if kind in ("rotate", "zp"):
        primes = heconv.gen_primes(N, c["bits"], L + 1)
        ext = heconv.Context(N, primes)
        q = primes[:L]
        sk = rnd.ints((N,), -1, 2)

        def key(g):
            k = _words(L, 2, L + 1, N)
            ext.galois_key(g, sk, rnd.residues((L, L + 1, N), primes), rnd.ints((L, N), -21, 22), k,
                           _words(ext.galois_key_work_words()))
            return k

        n = c["n"]
        s.update(ext=ext, n=n, out=_words(n, 2, L, N))
        if kind == "rotate":
            s.update(g=c["g"], ct=rnd.residues((n, 2, L, N), q), key=key(c["g"]), work=_words(ext.keyswitch_work_words(n)))
            return s
        n_out, n_in = 1 << (c["rows"] - 1).bit_length(), 1 << (c["cols"] - 1).bit_length()
        t = heconv.gen_primes(N, 37, 1)[0]
        tctx = heconv.Context(N, [t], t)
        slots, coeffs, w = _words(n_out, N), _words(n_out, N), _words(n_out, L, N)
        tctx.zp_diagonals_rect(rnd.ints((c["rows"], c["cols"]), 0, t), c["rows"], c["cols"], n_out, n_in, slots)
        tctx.simd_encode(n_out, slots, coeffs)
        ext.zp_encode_plain(n_out, coeffs, w)
        x = rnd.residues((n, 2, L, N), q)
        base = heconv.Context(N, q)
        base.ntt_fwd(x)
        per = n_out // c["groups"]
        folds = []
        step = n_out
        while step < n_in:
            g = pow(5, step, 2 * N)
            folds.append((g, key(g)))
            step *= 2
        g2 = pow(5, per, 2 * N)
        s.update(x=x, w=w, D=n_out, groups=c["groups"], key=key(5), g2=g2, key2=key(g2), folds=folds,
                 out2=_words(n, 2, L, N), work=_words(ext.zp_grouped_work_words(n, c["groups"])))
        return s
    q = heconv.gen_primes(N, c["bits"], L)
    ctx = heconv.Context(N, q, T37)
    s["ctx"] = ctx
    if kind == "client":
        n = c["n"]
        sk_ntt = _words(L, N)
        ctx.key_encode(rnd.ints((N,), -1, 2), sk_ntt)
        s.update(n=n, sk=sk_ntt, msgs=rnd.ints((n, N), 0, T37), a=rnd.residues((n, L, N), q),
                 err=rnd.ints((n, N), -21, 22), ct=_words(n, 2, L, N), dec=_words(n, N), work=_words(n, L, N))
        return s
    layers = []
    for shape in _shapes(c):
        C, H, W, M, kh, kw, stride, pad = shape
        d = ctx.plan(shape, batch=c["B"])
        z = ctx.sizes(d)
        wntt = _words(z.w_words)
        ctx.encode_weights(d, rnd.ints((M, C, kh, kw), -2 ** 12, 2 ** 12), wntt)
        ct = rnd.residues((c["B"] * z.in_cts, 2, L, N), q)
        layers.append((d, ct, torch.empty_like(ct), wntt, _words(c["B"] * z.out_cts, 2, L, N)))
    s.update(B=c["B"], layers=layers)
    if kind == "batch":
        s["batch"] = heconv.Batch(ctx, [(d, c["B"], buf, w, out) for d, _, buf, w, out in layers])
    if kind == "server":
        d = layers[0][0]
        ho, wo = ctx.out_hw(d)
        s.update(share=rnd.ints((c["B"], d.C, d.H, d.W), 0, T37), mask=rnd.ints((c["B"], d.M, ho, wo), 0, T37),
                 y=_words(c["B"], d.M, L, ho, wo))
    return s


def run(state):
    s = state
    kind = s["kind"]
    if kind == "rotate":
        s["ext"].rotate(s["g"], s["n"], s["ct"], s["key"], s["out"], s["work"])
        return s["out"]
    if kind == "zp":
        ext, out, other = s["ext"], s["out"], s["out2"]
        ext.zp_matvec_grouped(5, s["n"], s["x"], s["w"], s["D"], s["groups"], s["key"], s["g2"], s["key2"], out, s["work"])
        for g, key in s["folds"]:
            ext.zp_fold(g, s["n"], out, key, other, s["work"])
            out, other = other, out
        return out
    ctx = s["ctx"]
    if kind == "client":
        ctx.encrypt(s["n"], s["msgs"], s["a"], s["err"], s["sk"], s["ct"], s["work"])
        ctx.decrypt(s["n"], s["ct"], s["sk"], s["dec"], s["work"])
        return {"ct": s["ct"], "dec": s["dec"]}
    for d, ct, buf, w, out in s["layers"]:
        buf.copy_(ct)
    if kind == "batch":
        s["batch"].launch()
        return [layer[4] for layer in s["layers"]]
    d, ct, buf, w, out = s["layers"][0]
    if kind == "server":
        ctx.add_share(d, s["B"], buf, s["share"])
        ctx.conv_layer(d, s["B"], buf, w, out)
        ctx.mask_extract(d, s["B"], out, s["mask"], None, s["y"])
        return {"out": out, "y": s["y"]}
    ctx.conv_layer(d, s["B"], buf, w, out)
    return out


def _packed(v, bits):
    """Nonnegative integers as one big integer of `bits`-bit slots."""
    b = bits // 8
    return int.from_bytes(b"".join(int(x).to_bytes(b, "little") for x in v), "little")


def exact(case, seed):
    """A small layer by its definition: negacyclic products of the packed
    polynomials over the integers, reduced mod q.  None where that takes too
    long (every output is a whole number)."""
    c = case
    if c["kind"] != "layer":
        return None
    shape = _shapes(c)[0]
    d, CB, S = _planned(c, shape)
    N, L, B, M = c["N"], c["L"], c["B"], d.M
    if B * S * 2 * L * M * CB * N > 200000:
        return None
    rnd = _Rand(seed)
    q = heconv.gen_primes(N, c["bits"], L)
    K = rnd.ints((M, d.C, d.kh, d.kw), -2 ** 12, 2 ** 12).cpu().numpy()
    ct = rnd.residues((B * CB * S, 2, L, N), q).cpu().numpy().reshape(B, CB, S, 2, L, N)
    hw, O = d.Hw * d.Ww, (d.Cw - 1) * d.Hw * d.Ww + (d.kh - 1) * d.Ww + (d.kw - 1)
    out = np.zeros((B * M * S, 2, L, N), dtype=np.int64)
    slot = 144  # bits of one coefficient of a product: above 2 * 60 + log2(N * CB)
    for l in range(L):
        ker = np.zeros((M, CB, N), dtype=object)
        for m in range(M):
            for ch in range(d.C):
                cb, cc = divmod(ch, d.Cw)
                for i in range(d.kh):
                    for j in range(d.kw):
                        ker[m, cb, O - cc * hw - i * d.Ww - j] = int(K[m, ch, i, j]) % q[l]
        kp = [[_packed(ker[m, cb], slot) for cb in range(CB)] for m in range(M)]
        for b in range(B):
            for s in range(S):
                for comp in range(2):
                    xp = [_packed(ct[b, cb, s, comp, l], slot) for cb in range(CB)]
                    for m in range(M):
                        p = sum(x * k for x, k in zip(xp, kp[m])).to_bytes(2 * N * slot // 8, "little")
                        v = [int.from_bytes(p[i * slot // 8:(i + 1) * slot // 8], "little") for i in range(2 * N)]
                        out[(b * M + m) * S + s, comp, l] = [(v[i] - v[i + N]) % q[l] for i in range(N)]
    return torch.from_numpy(out)
