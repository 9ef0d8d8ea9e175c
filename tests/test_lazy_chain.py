"""Column passes and the rows behind them as one chain of lazily reduced words
(csrc/lazymod.hpp): the rows reduce only as far as the bound they are compiled for
needs, so a column form must not leave more than that.

On the CPU: the bounds of the library's own headers, compiled for the host, over
both word types, kinds and every column radix; and the device formulas of k_colq
and of a row's first stages in 64-bit words, on columns chosen for large outputs.
On the GPU: a product of those columns under every small-batch plan that puts rows
of 2^12 words behind k_colq. Whole numbers: no tolerance."""
import functools
import os
import subprocess

import numpy as np
import pytest

from gpu_helpers import first_mismatch, operands, oracle_polymul, oracle_tables

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
U = np.uint64
M32 = U(0xffffffff)


# ------------------------------------------------- bounds, from the headers --

PROGRAM = r"""
#include <cstdio>
#include "ntt_device.hpp"
using namespace pm;
template <typename W, int KIND, int LOGR> void one() {
  printf("%d %d %d %d %d %d\n", (int)sizeof(W) * 8, KIND, LOGR, col_bound<LOGR, KIND, W>(),
         colq_bound<LOGR, KIND, W>(), LazyRule<W, KIND>::H);
  if constexpr (LOGR < 7) one<W, KIND, LOGR + 1>();
}
int main() { one<uint64_t, 0, 0>(); one<uint64_t, 1, 0>(); one<uint32_t, 0, 0>(); one<uint32_t, 1, 0>(); }
"""


@functools.lru_cache(maxsize=None)
def _bounds():
    """{(bits, kind, logr): (col_bound, colq_bound, H)} in sixteenths of q."""
    import tempfile
    from paper_2209_01290_amd import build
    with tempfile.TemporaryDirectory() as d:
        src, exe = os.path.join(d, "bounds.hip"), os.path.join(d, "bounds")
        with open(src, "w") as f:
            f.write(PROGRAM)
        subprocess.run([build.HIPCC] + build.CFLAGS + ["-O0", "-I", build.CSRC, src, "-o", exe], check=True,
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
        out = subprocess.run([exe], check=True, stdout=subprocess.PIPE, text=True).stdout
    rows = [tuple(int(v) for v in line.split()) for line in out.splitlines()]
    return {r[:3]: r[3:] for r in rows}


def _ct(b, deficit, wide):
    """One stage on words below b: (reduced first, k, bound left), worked out here."""
    r = 48 + -(-deficit * b // 16) if wide else 32
    k, H = -(-r // 16), 256 if wide else 64
    red = b + 16 * k > H
    return red, k, (32 if red else b) + 16 * k


def _chain(b, deficits, wide):
    for d in deficits:
        b = _ct(b, d, wide)[2]
    return b


@pytest.mark.parametrize("bits,kind", [(64, 0), (64, 1), (32, 0), (32, 1)])
def test_column_bounds(bits, kind):
    """col_bound and colq_bound are what the stages of each form leave, and fit."""
    wide = bits == 64 and kind == 0
    for logr in range(8):
        col, colq, H = _bounds()[(bits, kind, logr)]
        one = _chain(16, [2] * logr, wide)                       # k_col, the pipelined kernels' columns
        pair = _chain(16, [2] + [4] * 4, wide) if logr == 5 else one   # a column on two lanes
        assert col == max(one, pair) <= H
        assert colq == _chain(16, [4] * logr, wide) <= H
    if wide:
        # the fixed-radix rows' bound does not cover k_colq's words at these radices
        assert [_bounds()[(64, 0, r)][:2] for r in (2, 3, 4, 5)] == [(144, 160), (224, 256), (112, 144), (240, 240)]


# --------------------------------------------------- the formulas on words --

def _mulhi32(a, b):
    return (a * b) >> U(32)


def _mulhi_low3(a, b):
    ah, al, bh, bl = a >> U(32), a & M32, b >> U(32), b & M32
    return ah * bh + _mulhi32(al, bh) + _mulhi32(ah, bl)


class Model:
    """ct_lazy on 64-bit words with both companions, for one 60-bit modulus."""

    def __init__(self, q):
        self.q, self.m = q, q.bit_length()
        self.ml = ((1 << (self.m + 64)) // q) - (1 << 64)
        self.c = (1 << 64) // q

    def companion(self, w, uni):
        ws = int(w) << (64 - self.m)
        if uni:
            return ws + ((ws * self.ml) >> 64)
        h, l = ws >> 32, ws & 0xffffffff
        mh, ml = self.ml >> 32, self.ml & 0xffffffff
        return ws + h * mh + ((l * mh) >> 32) + ((h * ml) >> 32)

    def ct(self, u, v, w, b, uni):
        """(u, v) after a stage on words below b, as the bound's reductions make it."""
        red, k, out = _ct(b, 2 if uni else 4, True)
        q = U(self.q)
        if red:
            u = u - _mulhi32(u >> U(32), U(self.c)) * q
        s = u + v * U(int(w)) - _mulhi_low3(v, U(self.companion(w, uni))) * q
        return s, u * U(2) + U(k * self.q) - s, out

    def exact_ct(self, u, v, w):
        """The residues of the same outputs (object arrays of whole numbers)."""
        p = v * int(w) % self.q
        return (u + p) % self.q, (u - p) % self.q


def _stages(x, ct, tw, logr, rb):
    """Stages of a radix-2^logr block on x (a list of 2^logr words), ct(u, v, w, stage)."""
    for s in range(logr):
        k = 1 << (logr - 1 - s)
        for g in range(1 << s):
            for j in range(k):
                a = 2 * g * k + j
                x[a], x[a + k] = ct(x[a], x[a + k], tw[(rb << s) + g], s)
    return x


LOGN, LOGR, ROW = 16, 4, 1


@functools.lru_cache(maxsize=None)
def _columns():
    """(q, psi_br, columns): four columns of 16 canonical words at the offsets 0, 1024,
    2048, 3072 of N = 2^16 whose words of row 1, as k_colq leaves them, are the largest
    (first) and make the smallest twiddle products (the others) of 2^18 random columns."""
    from paper_2209_01290_amd import lib
    q = lib.pm_ntt_primes(1 << LOGN, 1, 60)[0]
    tw = [int(w) for w in lib.pm_make_tables(q, 1 << LOGN)[0][:128]]
    M = Model(q)
    with np.errstate(over="ignore"):
        x = list(np.random.default_rng(2209).integers(0, q, (1 << LOGR, 1 << 18), dtype=np.uint64))
        keep = np.stack(x)
        b = 16
        bs = []
        for s in range(LOGR):
            bs.append(b)
            b = _ct(b, 4, True)[2]
        last = _stages(x, lambda u, v, w, s: M.ct(u, v, w, bs[s], False)[:2], tw, LOGR, 1)[ROW]
        # the twiddles of the row's first stage, and of the second's upper half
        w0, w1 = tw[16 + ROW], tw[2 * (16 + ROW) + 1]
        p0 = last * U(w0) - _mulhi_low3(last, U(M.companion(w0, True))) * U(q)
        big, small = int(np.argmax(last)), int(np.argmin(p0))
        # the word at 3072 of the pair (1024, 3072): its product with w1 small after the first stage
        i1, i3 = np.arange(0, 1 << 17), np.arange(1 << 17, 1 << 18)
        v = last[i1] + U(4 * q) - p0[i3]
        p1 = v * U(w1) - _mulhi_low3(v, U(M.companion(w1, True))) * U(q)
        j = int(np.argmin(p1))
    return q, tw, [keep[:, c] for c in (big, int(i1[j]), small, int(i3[j]))]


def _row_word(bound):
    """The word at 3072 of row 1 after two stages of a row compiled for words below
    `bound`: (the 64-bit word, its true residue)."""
    q, tw, cols = _columns()
    M = Model(q)
    words, exact = [], []
    with np.errstate(over="ignore"):
        for c in cols:
            b, bs = 16, []
            for s in range(LOGR):
                bs.append(b)
                b = _ct(b, 4, True)[2]
            words.append(_stages([np.array([w]) for w in c], lambda u, v, w, s: M.ct(u, v, w, bs[s], False)[:2],
                                 tw, LOGR, 1)[ROW])
            exact.append(_stages([int(w) for w in c], lambda u, v, w, s: M.exact_ct(u, v, w), tw, LOGR, 1)[ROW])
        assert [int(w[0]) % q for w in words] == exact           # the columns themselves are right
        b1 = _ct(bound, 2, True)[2]
        row = _stages(words, lambda u, v, w, s: M.ct(u, v, w, (bound, b1)[s], True)[:2], tw, 2, 16 + ROW)
    want = _stages(exact, lambda u, v, w, s: M.exact_ct(u, v, w), tw, 2, 16 + ROW)
    return int(row[3][0]), want[3]


def test_rows_behind_colq_words():
    """A row told k_colq's bound, or H, keeps the residue of these columns; one told
    col_bound wraps 2^64, which is why it does not get them."""
    q = _columns()[0]
    col, colq, H = _bounds()[(64, 0, LOGR)]
    for bound in (colq, H):
        word, want = _row_word(bound)
        assert word % q == want
    word, want = _row_word(col)
    assert word % q != want


@pytest.mark.gpu
@pytest.mark.parametrize("log2n", [14, 15, 16, 17])
def test_fused_small_plan_rows_of_4096(log2n):
    """The fused product under a 4-word plan with rows of 2^12 words (columns by k_colq)."""
    import torch
    from paper_2209_01290_amd import lib as L
    N = 1 << log2n
    q = L.pm_ntt_primes(N, 1, 60)[0]
    a, b = operands(N, [q], 1, request=4200 + log2n)
    if log2n == LOGN:
        q2, _, cols = _columns()
        assert q2 == q
        for o, c in zip((0, 1024, 2048, 3072), cols):
            a[0, 0].reshape(16, 4096)[:, o] = c
    fw, iv = oracle_tables([q], N)
    want = oracle_polymul(a, b, [q], N, fw, iv)
    prm = L.Params(N, 1, primes=[q])
    da, db = L.to_device(a), L.to_device(b)
    dc = torch.empty_like(da)
    ws = torch.empty(N, dtype=torch.int64, device="cuda")
    L.pm_tune_set_small(L.OP_POLYMUL, log2n, 12, 4)
    L.pm_tune_set_small_batch(N)
    try:
        for x, y in ((da, db), (db, da)):
            L.pm_polymul_fused(x, y, dc, N, 1, 1, [q], prm.psi_br, prm.psi_inv_br, ws)
            msg = first_mismatch(L.to_host(dc).reshape(want.shape), want)
            assert msg is None, "N 2^%d: %s" % (log2n, msg)
    finally:
        L.pm_tune_set_small(L.OP_POLYMUL, log2n, 0, 0)
        L.pm_tune_set_small_batch(0)
