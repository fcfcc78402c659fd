"""The extension's batches and rankings against the oracle, where they can go
wrong: steps that repeat hashes (tandem arrays), long copies whose estimate
stays near the threshold, sorts of every size, keys of 32 and 64 bits.  All
outputs are whole numbers: equality."""
import numpy as np
import pytest

from paper_1807_00205_amd import synth

pytestmark = pytest.mark.gpu


# (w = 128 crowds the minimizers into the lowest hashes: large buckets)
@pytest.mark.parametrize("k,w,length,batch_min", [
    (12, 16, 60_000, None), (12, 16, 60_000, 0), (12, 4, 30_000, None), (14, 10, 40_000, None),
    (16, 16, 60_000, None), (9, 5, 20_000, None), (12, 128, 200_000, None)])
def test_extend_steps(oracle_lib, k, w, length, batch_min):
    from paper_1807_00205_amd import sdf
    g = synth.tandem_case(500 + k + w, length=length, n_arrays=30, copies_hi=40, n_seqs=2, n_sd=6)
    rng = synth.rng_for(k * w)
    src = g.seqs[0][1_000:length // 3]
    cp = synth.mutate(rng, src, 0.08)[:length // 2]
    g.seqs[1][length // 4:length // 4 + len(cp)] = cp
    b, off = g.concat()
    ix = sdf.Index(g.seqs, k, w)
    orc = oracle_lib.OracleIndex(b, off, k, w)
    tau, _, _ = oracle_lib.params(0.25, 1000, k)
    rows = [(o, qs, qb, qb + ln, ts, tb, tb + ln)
            for o in (0, 1) for qs, ts in ((0, 1), (1, 1), (0, 0))
            for qb, tb, ln in ((1_500, length // 4 + 500, 900), (length // 2, 200, 1_500),
                               (length // 3, 2 * length // 3, 400), (3_000, length // 4 + 2_000, 5_000))
            if qs != ts or abs(qb - tb) >= ln]
    got = ix.extend(rows, 0.25) if batch_min is None else None
    if got is None:
        with sdf.tuning(ext_batch_min=batch_min):
            got = ix.extend(rows, 0.25)
    want = orc.extend(np.array([[off[qs] + qb, off[qs] + qe, off[ts] + tb, off[ts] + te, o]
                                for o, qs, qb, qe, ts, tb, te in rows], np.uint64), tau)
    qo = off[got["q_seq"]].astype(np.uint64)
    to = off[got["t_seq"]].astype(np.uint64)
    for f, x in (("q_begin", want["q_begin"] - qo), ("q_end", want["q_end"] - qo),
                 ("t_begin", want["t_begin"] - to), ("t_end", want["t_end"] - to),
                 ("m", want["m"]), ("s", want["s"]), ("stop", want["stop"])):
        assert np.array_equal(got[f].astype(np.uint64), x.astype(np.uint64)), f
    ix.close()
