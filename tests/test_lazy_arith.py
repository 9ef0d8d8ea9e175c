"""The lazily reduced butterflies (csrc/lazymod.hpp): their bounds on the CPU,
and every transform and product path at the moduli lengths where the
arithmetic changes, against the oracle.

Bounds: the device formulas in Python integers, for moduli at both ends of a
length and words at the ends of their ranges. The results are compared exactly
(whole numbers): no tolerance."""
import random

import numpy as np
import pytest

import oracle

from gpu_helpers import device_tables, first_mismatch


def _hi(x):
    return x >> 32


def _lo(x):
    return x & 0xffffffff


def _mulhi_low3(a, b):
    return _hi(a) * _hi(b) + _hi(_lo(a) * _hi(b)) + _hi(_hi(a) * _lo(b))


def _edge(rnd, n):
    """Words below n: its ends, full low or high words, uniform."""
    return rnd.choice([n - 1, 0, 1, n >> 1, rnd.randrange(n), (n - 1) & ~0xffffffff, min(n - 1, 0xffffffff),
                       max(0, (n & ~0xffffffff) - 1)])


@pytest.mark.parametrize("m", [34, 35, 47, 59, 60])
def test_bounds_64(m):
    rnd = random.Random(m)
    ends = [(1 << m) - 1 - 2 * i for i in range(3)] + [(1 << (m - 1)) + 1 + 2 * i for i in range(3)]
    for q in ends + [rnd.randrange(1 << (m - 1), 1 << m) | 1 for _ in range(6)]:
        ml = ((1 << (m + 64)) // q) - (1 << 64)
        assert 0 <= ml < 1 << 64
        c = (1 << (64 - m)) | (ml >> m)
        assert c == (1 << 64) // q < 1 << 32
        mu = (1 << 62) | (ml >> 2)
        assert mu == (1 << (m + 62)) // q
        for _ in range(200):
            w = _edge(rnd, q)
            ws = w << (64 - m)
            for p, d in ((ws + ((ws * ml) >> 64), 2), (ws + _mulhi_low3(ws, ml), 4)):
                assert p < 1 << 64 and 0 <= (w << 64) - p * q < d * q
                v = min(_edge(rnd, 16 * q), (1 << 64) - 1)
                r = v * w - _mulhi_low3(v, p) * q
                bound = 16 * (v + 1) // q + 1                      # v < bound/16 q
                assert 0 <= 16 * r < (48 + (d * min(bound, 256) + 15) // 16) * q
            x = min(_edge(rnd, 16 * q), (1 << 64) - 1)
            assert 0 <= x - _hi(_hi(x) * c) * q < 2 * q
            a, b = _edge(rnd, 2 * q), _edge(rnd, 2 * q)
            cc = (a * b) >> (m - 2)
            assert cc < 1 << 64
            assert 0 <= 2 * (a * b - _mulhi_low3(cc, mu) * q) < 9 * q


@pytest.mark.parametrize("m", [34, 35, 47, 59, 60])
def test_block_product_64(m):
    """Sums of four products of words below 2q: the limb sums fit 64 bits and the
    reduction leaves a word below 6q."""
    rnd = random.Random(m)
    M31 = (1 << 31) - 1
    for q in {(1 << m) - 1, (1 << (m - 1)) + 1, rnd.randrange(1 << (m - 1), 1 << m) | 1}:
        ml = ((1 << (m + 64)) // q) - (1 << 64)
        for _ in range(100):
            a = [_edge(rnd, 2 * q) for _ in range(4)]
            b = [_edge(rnd, 2 * q) for _ in range(4)]
            c0 = sum((x & M31) * (y & M31) for x, y in zip(a, b))
            c1 = sum((x & M31) * (y >> 31) + (x >> 31) * (y & M31) for x, y in zip(a, b))
            c2 = sum((x >> 31) * (y >> 31) for x, y in zip(a, b))
            assert max(c0, c1, c2) < 1 << 64
            u = c1 + (c0 >> 31)
            h = c2 + (u >> 31)
            S = sum(x * y for x, y in zip(a, b))
            assert u < 1 << 64 and h == S >> 62 and h < 1 << 64
            c = S >> m
            assert c < 1 << 64
            k = c + _mulhi_low3(c, ml)
            assert k < 1 << 64 and 0 <= S - k * q < 6 * q


@pytest.mark.parametrize("m", [4, 17, 29, 30])
def test_block_product_32(m):
    rnd = random.Random(m)
    for q in {(1 << m) - 1, (1 << (m - 1)) + 1, rnd.randrange(1 << (m - 1), 1 << m) | 1}:
        ml = ((1 << (m + 32)) // q) - (1 << 32)
        R = (-(((1 << 32) + ml) >> m) * q) % (1 << 32)
        assert R == (1 << 32) % q
        for i in range(200):
            a = [_edge(rnd, 2 * q) if i else 2 * q - 1 for _ in range(4)]
            b = [_edge(rnd, 2 * q + 1) if i else 2 * q for _ in range(4)]     # 2q: a negated zero
            S = sum(x * y for x, y in zip(a, b))
            assert S < 1 << 64
            s = _hi(S) * R + _lo(S)
            c = s >> m
            assert s % q == S % q and s < 1 << 64 and c < 1 << 32
            k = c + _hi(c * ml)
            assert k < 1 << 32 and 0 <= s - k * q < 4 * q < 1 << 32


@pytest.mark.parametrize("bits,m", [(64, 2), (64, 33), (64, 61), (64, 62), (32, 3), (32, 29), (32, 30)])
def test_bounds_four_q(bits, m):
    """Harvey's rule: exact companions (32-bit words up to 29 bits: short by
    less than two), products of words below 4q stay below 2q."""
    rnd = random.Random(m)
    for q in {(1 << m) - 1, (1 << m) - 3, (1 << (m - 1)) + 1, rnd.randrange(1 << (m - 1), 1 << m) | 1}:
        if q < 3:
            continue
        ml = ((1 << (m + bits)) // q) - (1 << bits)
        for _ in range(200):
            w = _edge(rnd, q)
            ws = w << (bits - m)
            p = ws + ((ws * ml) >> bits)
            rem = (-p * q) % (1 << bits)
            assert rem == (w << bits) - p * q < 2 * q
            if not (bits == 32 and m <= 29):
                p += rem >= q
                assert p == (w << bits) // q
            v = _edge(rnd, 4 * q)
            assert 0 <= v * w - ((v * p) >> bits) * q < 2 * q


def _words(q, N, kind, rng):
    if kind == "max":
        return np.full(N, q - 1, dtype=np.uint64)
    x = rng.integers(0, q, N, dtype=np.uint64)
    x[:: 3] = q - 1                     # long runs of the largest word among random and zero ones
    x[1:: 5] = 0
    return x


# one size per form: a wave's rows, single rows at both ends of a row kernel, two passes of each column radix
@pytest.mark.gpu
@pytest.mark.parametrize("small", [False, True])
@pytest.mark.parametrize("log2n", [1, 2, 3, 5, 8, 10, 11, 12, 13, 14, 15, 16, 17])
@pytest.mark.parametrize("bits", [33, 34, 47, 60, 61, 62])
def test_paths_at_modulus_lengths(bits, log2n, small):
    import torch
    from paper_2209_01290_amd import lib as L
    N = 1 << log2n
    if bits < log2n + 2:
        pytest.skip("no such modulus")
    if small and not 8 <= log2n:
        pytest.skip("no small-batch split")
    rng = np.random.default_rng(bits * 100 + log2n)
    # the largest modulus of this length, and (in one batch) one of 60 bits
    qs = L.pm_ntt_primes(N, 1, bits) + L.pm_ntt_primes(N, 1, 60)[: 1 if bits in (34, 61) else 0]
    fw, iv, dfw, div = device_tables(qs, N)
    o = oracle.default()
    a = np.array([[_words(q, N, k, rng) for k in ("max", "mix")] for q in qs])
    b = np.array([[_words(q, N, k, rng) for k in ("max", "mix")] for q in qs])
    da, db = L.to_device(a), L.to_device(b)
    limbs, polys = len(qs), 2
    ws = torch.empty(limbs * polys * N, dtype=torch.int64, device="cuda")

    def check(got, want, what):
        msg = first_mismatch(L.to_host(got).reshape(want.shape), want)
        assert msg is None, "%s bits %d N 2^%d: %s" % (what, bits, log2n, msg)

    if small:
        for op in (L.OP_NTT_FWD, L.OP_NTT_INV, L.OP_POLYMUL):
            L.pm_tune_set_small(op, log2n, max(5, log2n - 7) if log2n != 10 else 10, 4)
        L.pm_tune_set_small_batch(1 << 40)
    try:
        want = np.array([[o.polymul_ntt(a[l, p], b[l, p], q, fw[l], iv[l]) for p in range(polys)]
                         for l, q in enumerate(qs)])
        c = torch.empty_like(da)
        L.pm_polymul(da, db, c, N, limbs, polys, qs, dfw, div, ws)
        check(c, want, "polymul")
        L.pm_polymul_fused(da, db, c, N, limbs, polys, qs, dfw, div, ws)
        check(c, want, "fused")
        ntt = np.array([[o.ntt_fwd(a[l, p], q, fw[l]) for p in range(polys)] for l, q in enumerate(qs)])
        x = da.clone()
        L.pm_ntt_fwd(x, N, limbs, polys, qs, dfw)
        check(x, ntt, "ntt_fwd")
        L.pm_ntt_inv(x, N, limbs, polys, qs, div)
        check(x, a, "ntt_inv of ntt_fwd")
        y = da.clone()
        L.pm_ntt_inv(y, N, limbs, polys, qs, div)
        check(y, np.array([[o.ntt_inv(a[l, p], q, iv[l]) for p in range(polys)] for l, q in enumerate(qs)]),
              "ntt_inv")
        if not small:
            il = da.transpose(1, 2).contiguous()
            cl = torch.empty_like(il)
            L.pm_polymul_il(il, db.transpose(1, 2).contiguous(), cl, N, limbs, polys, qs, dfw, div, ws)
            check(cl.transpose(1, 2).contiguous(), want, "polymul_il")
            L.pm_ntt_fwd_il(il, N, limbs, polys, qs, dfw)
            check(il.transpose(1, 2).contiguous(), ntt, "ntt_fwd_il")
            L.pm_ntt_inv_il(il, N, limbs, polys, qs, div)
            check(il.transpose(1, 2).contiguous(), a, "ntt_inv_il")
    finally:
        for op in (L.OP_NTT_FWD, L.OP_NTT_INV, L.OP_POLYMUL):
            L.pm_tune_set_small(op, log2n, 0, 0)
        L.pm_tune_set_small_batch(0)
