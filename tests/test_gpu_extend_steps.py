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


@pytest.mark.parametrize("strand", [0, 1])
def test_crowded_bucket_shortens_the_horizon(strand):
    """Sides of 1 Mbp under a wide winnowing window: the minimizers that both
    phases can reach crowd the lowest of 2,048 buckets of hashes (some 2,190 of
    them, most distinct, where 2,048 are held), so the horizon is shortened, as it
    is for too many minimizers, instead of the region being refused.  The result
    does not depend on the horizon: with 1/64 of the side never more than 1,970
    are gathered."""
    from paper_1807_00205_amd import sdf
    rng = np.random.default_rng(77)
    n, side, at = 2_500_000, 1_050_000, 350_000
    a, b = synth.random_bases(rng, n), synth.random_bases(rng, n)
    copy = a[at:at + side + 30_000].copy()
    hit = rng.random(len(copy)) < 0.02
    copy[hit] = synth.random_bases(rng, int(hit.sum()))
    t0 = n - at - len(copy) if strand else at
    b[t0:t0 + len(copy)] = synth.revcomp(copy) if strand else copy
    ix = sdf.Index([a, b], 12, 64)
    reg = np.zeros(1, sdf.REGION_DTYPE)
    reg["strand"], reg["t_seq"] = strand, 1
    reg["q_begin"], reg["q_end"] = at + 100, at + 100 + side
    reg["t_begin"] = t0 + (len(copy) - 100 - side if strand else 100)
    reg["t_end"] = reg["t_begin"] + side
    got = ix.extend(reg, 0.25, max_len=1_980_000)
    with sdf.tuning(ext_hdiv=64):
        want = ix.extend(reg, 0.25, max_len=1_980_000)
    for f in ("q_begin", "q_end", "t_begin", "t_end", "m", "s", "stop"):
        assert np.array_equal(got[f], want[f]), f
    assert got["q_end"][0] - got["q_begin"][0] > side + 20_000
    ix.close()
