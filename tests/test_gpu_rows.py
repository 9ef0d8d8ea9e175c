"""Row kernels where their lanes, rows and launches end: the coefficient-major
layout's LDS rows (16 polynomials to a workgroup) around 16 polynomials, and job
tables whose tuned rows are of 2^13 or 2^14 words, on both sides of the row
counts from which those are used. Whole numbers against the oracle: no tolerance."""
import numpy as np
import pytest

from gpu_helpers import first_mismatch, operands, oracle_ntt_fwd, oracle_ntt_inv, oracle_polymul, oracle_tables
from paper_2209_01290_amd import synth

pytestmark = pytest.mark.gpu


# one pass (2^6..2^10: every row length), rows of 2^8 at both ends, of 2^9, of 2^10 below one and two blocks
@pytest.mark.parametrize("bits", [60, 62])
@pytest.mark.parametrize("log2n", [6, 7, 8, 9, 10, 11, 14, 15, 16, 17])
@pytest.mark.parametrize("polys", [15, 16, 17, 33])
def test_il_rows(log2n, polys, bits):
    import torch
    from paper_2209_01290_amd import lib as L
    if log2n > 14 and polys > 17:
        pytest.skip("the oracle's time")
    N = 1 << log2n
    qs = L.pm_ntt_primes(N, 2, bits)
    prm = L.Params(N, 2, primes=qs)
    fw, iv = oracle_tables(qs, N)
    a, b = operands(N, qs, polys, request=1500 + log2n)
    il = lambda x: np.ascontiguousarray(np.transpose(x, (0, 2, 1)))
    da, db = L.to_device(il(a)), L.to_device(il(b))
    # the words behind the result belong to somebody else
    c = torch.full((2 * N * polys + 64,), -1, dtype=torch.int64, device="cuda")
    ws = torch.empty(L.pm_polymul_il_workspace_bytes(N, 2, polys) // 8, dtype=torch.int64, device="cuda")
    L.pm_polymul_il(da, db, c, N, 2, polys, qs, prm.psi_br, prm.psi_inv_br, ws)
    got = L.to_host(c)
    assert (got[2 * N * polys:] == np.uint64(2**64 - 1)).all()
    got = np.transpose(got[: 2 * N * polys].reshape(2, N, polys), (0, 2, 1))
    msg = first_mismatch(np.ascontiguousarray(got), oracle_polymul(a, b, qs, N, fw, iv))
    assert msg is None, "N 2^%d x %d, %d bits: %s" % (log2n, polys, bits, msg)
    x, y = da.clone(), da.clone()
    L.pm_ntt_fwd_il(x, N, 2, polys, qs, prm.psi_br)
    L.pm_ntt_inv_il(y, N, 2, polys, qs, prm.psi_inv_br)
    for what, t, want in (("fwd", x, oracle_ntt_fwd(a, qs, fw)), ("inv", y, oracle_ntt_inv(a, qs, iv))):
        got = np.transpose(L.to_host(t).reshape(2, N, polys), (0, 2, 1))
        msg = first_mismatch(np.ascontiguousarray(got), want)
        assert msg is None, "%s N 2^%d x %d, %d bits: %s" % (what, log2n, polys, bits, msg)


# one tuned row length for all long sizes (2^13: 512 rows and more, 2^14: 256 and more), several, none
@pytest.mark.parametrize("rows, mix", [
    ({13: 13}, [(13, 511), (10, 3)]), ({13: 13}, [(13, 512), (10, 3)]),
    ({14: 14}, [(14, 255)]), ({14: 14}, [(14, 256)]),
    ({13: 13, 15: 13}, [(13, 500), (15, 3)]), ({13: 13, 14: 14}, [(13, 512), (14, 256)]),
    ({13: 13}, [(13, 512), (12, 1)]), ({13: 10, 14: 11}, [(13, 5), (14, 4), (12, 1)]), ({13: 10}, [(13, 5)])],
    ids=lambda v: "_".join("%dx%d" % t for t in v) if isinstance(v, list) else "")
def test_job_rows(rows, mix):
    import torch
    from paper_2209_01290_amd import lib as L
    before = {n: L.pm_tune_get(L.OP_POLYMUL, n) for n in rows}
    jobs, keep = [], []
    try:
        for n, c in rows.items():
            L.pm_tune_set(L.OP_POLYMUL, n, c)
        L.pm_tune_set_jobs_pipeline(0)
        for i, (log2n, count) in enumerate(mix):
            N, q = 1 << log2n, L.pm_ntt_primes(1 << log2n, 1, 60)[0]
            a, b = synth.operands(synth.SEED_BASE + 6, [q], count, N, request=i)
            dfw, div = (L.to_device(x) for x in L.pm_make_tables(q, N))
            da, db = L.to_device(a[0]), L.to_device(b[0])
            jobs.append(L.make_job(log2n, count, q, dfw, div, da, db, da))
            keep.append((log2n, q, a, b, dfw, div, da, db))
        ws = torch.empty((L.pm_polymul_jobs_workspace_bytes(jobs) + 7) // 8, dtype=torch.int64, device="cuda")
        L.pm_polymul_jobs(jobs, ws)
        for log2n, q, a, b, _, _, da, _ in keep:
            N, got = 1 << log2n, L.to_host(da).reshape(a[0].shape)
            fw, iv = oracle_tables([q], N)
            for p in (0, 1, len(got) // 2, len(got) - 2, len(got) - 1):
                p = min(max(p, 0), len(got) - 1)
                msg = first_mismatch(got[p][None, None],
                                     oracle_polymul(a[:, p:p + 1], b[:, p:p + 1], [q], N, fw, iv))
                assert msg is None, "N 2^%d product %d: %s" % (log2n, p, msg)
    finally:
        L.pm_tune_set_jobs_pipeline(-1)
        for n, c in before.items():
            L.pm_tune_set(L.OP_POLYMUL, n, c)


# rows of up to 16 words are one thread's: 256 products to a work item, whatever N
@pytest.mark.parametrize("count", [255, 256, 257, 700])
@pytest.mark.parametrize("log2n", [1, 2, 3, 4, 5])
def test_job_short_rows(log2n, count):
    import torch
    from paper_2209_01290_amd import lib as L
    N, q = 1 << log2n, L.pm_ntt_primes(1 << log2n, 1, 60)[0]
    a, b = synth.operands(synth.SEED_BASE + 7, [q], count, N)
    fw, iv = oracle_tables([q], N)
    want = oracle_polymul(a, b, [q], N, fw, iv)
    dfw, div = (L.to_device(x) for x in L.pm_make_tables(q, N))
    da, db = L.to_device(a[0]), L.to_device(b[0])
    c = torch.full((count * N + 64,), -1, dtype=torch.int64, device="cuda")
    jobs = [L.make_job(log2n, count, q, dfw, div, da, db, c)]
    ws = torch.empty((L.pm_polymul_jobs_workspace_bytes(jobs) + 7) // 8, dtype=torch.int64, device="cuda")

    def check(what):
        got = L.to_host(c)
        assert (got[count * N:] == np.uint64(2**64 - 1)).all()
        msg = first_mismatch(got[: count * N], want)
        assert msg is None, "%s N 2^%d x %d: %s" % (what, log2n, count, msg)

    L.pm_polymul_jobs(jobs, ws)
    check("jobs")
    c.fill_(-1)
    plan = L.pm_plan_create(jobs)
    try:
        L.pm_plan_launch(plan)
        check("plan")
    finally:
        L.pm_plan_destroy(plan)


# where the passes of a coefficient-major transform change: by size alone, by odd counts of
# polynomials (None: register blocks alone), by the words of the batch
@pytest.mark.parametrize("bits", [60, 62])
@pytest.mark.parametrize("log2n, limbs, polys, row", [
    (6, 1, 100, None), (7, 1, 4095, 7), (7, 1, 4097, None), (7, 1, 4096, 7), (7, 3, 1367, None), (7, 1, 32769, 7),
    (8, 1, 4099, None), (9, 1, 4101, None), (9, 1, 8193, 9), (10, 1, 4095, 10), (10, 1, 4097, None),
    (10, 1, 512, 8), (10, 1, 513, 10), (11, 1, 2047, 7), (11, 1, 2049, None), (12, 1, 2047, 8), (12, 3, 683, None),
    (14, 1, 64, 7), (14, 1, 65, 8), (15, 1, 127, 8), (15, 1, 128, 9),
    (16, 1, 64, 8), (16, 1, 65, 10), (16, 5, 13, 10), (17, 1, 1023, 8), (17, 1, 1024, None), (17, 3, 342, None)])
def test_il_transform_passes(log2n, limbs, polys, row, bits):
    import torch
    from paper_2209_01290_amd import lib as L
    if bits == 62 and log2n == 17 and limbs > 1:
        pytest.skip("time")
    N = 1 << log2n
    qs = L.pm_ntt_primes(N, limbs, bits)
    prm = L.Params(N, limbs, primes=qs)
    fw, iv = oracle_tables(qs, N)
    x = torch.empty((limbs, polys, N), dtype=torch.int64, device="cuda")
    for l, q in enumerate(qs):
        x[l].random_(0, q, generator=torch.Generator(device="cuda").manual_seed(17 + l))
    ends = [x[:, p].cpu().numpy().astype(np.uint64) for p in (0, polys - 1)]
    for what, il, rows, one, want in (("fwd", L.pm_ntt_fwd_il, L.pm_ntt_fwd, prm.psi_br, oracle_ntt_fwd),
                                      ("inv", L.pm_ntt_inv_il, L.pm_ntt_inv, prm.psi_inv_br, oracle_ntt_inv)):
        L.pm_prof_read(reset=True)
        L.pm_prof_enable(True)
        try:
            y = x.transpose(1, 2).contiguous()
            il(y, N, limbs, polys, qs, one)
            torch.cuda.synchronize()
        finally:
            L.pm_prof_enable(False)
        names = L.pm_prof_read(reset=True)
        assert [n for n in names if "_c" in n] == ([] if row is None else ["il_%s_c%d" % (what, row)]), sorted(names)
        z = x.clone()
        rows(z, N, limbs, polys, qs, one)
        assert torch.equal(y.transpose(1, 2), z)              # every word, against the other layout
        for p, e in zip((0, polys - 1), ends):
            got = y[:, :, p].cpu().numpy().astype(np.uint64)
            msg = first_mismatch(got, want(e[:, None], qs, fw if one is prm.psi_br else iv)[:, 0])
            assert msg is None, msg
