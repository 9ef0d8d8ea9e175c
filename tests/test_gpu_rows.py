"""Job tables whose tuned rows are of 2^13 or 2^14 words, on both sides of the row
counts from which those are used. Whole numbers against the oracle: no tolerance."""
import pytest

from gpu_helpers import first_mismatch, oracle_polymul, oracle_tables
from paper_2209_01290_amd import synth

pytestmark = pytest.mark.gpu


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
