"""The tile kernel's branches against the oracle, where they can go wrong:
blocks of windows at the edges of the mask words and past them, counters that
overflow, tiles in partitions.  All outputs are whole numbers: equality."""
import numpy as np
import pytest

from paper_1807_00205_amd import synth

pytestmark = pytest.mark.gpu

SEED_F = ["query_id", "i", "j", "strand", "shared", "sketch"]
CAND_F = ["query_id", "strand", "q_seq", "t_seq", "q_begin", "q_end", "t_begin", "t_end",
          "n_seeds", "max_shared"]


def _same(a, b, fields, what):
    assert len(a) == len(b), "%s: %d vs %d records" % (what, len(a), len(b))
    for f in fields:
        assert np.array_equal(np.asarray(a[f]).astype(np.uint64),
                              np.asarray(b[f]).astype(np.uint64)), (what, f)


# 64 windows reach 64 + 2 n / (w + 1) minimizers: three words of masks, four,
# and more (hits followed one by one); with k = 5 and 6 a tile has so many hits
# per target bin that counters of 4 and 8 bits overflow
@pytest.mark.parametrize("k,w,min_len,hits_per_part,threads", [
    (12, 16, 300, None, 512), (12, 16, 1400, None, 512), (12, 16, 1500, None, 1024),
    (12, 16, 3000, None, 1024), (12, 3, 1000, None, 512), (12, 1, 400, None, 1024),
    (12, 16, 1000, 1024, 1024), (12, 3, 1000, 1024, 512),
    (6, 8, 600, None, 512), (6, 8, 600, None, 1024), (6, 5, 500, 4000, 512),
    (5, 8, 600, None, 512), (5, 6, 600, None, 1024)])
def test_tile_kernel_branches(oracle_lib, k, w, min_len, hits_per_part, threads):
    from paper_1807_00205_amd import sdf
    g = synth.tandem_case(1000 + 31 * k + w + min_len, length=24_000, n_arrays=24, copies_hi=50,
                          n_seqs=2, n_sd=4)
    src = g.seqs[0][2_000:2_000 + 2 * min_len]
    g.seqs[1][9_000:9_000 + len(src)] = src          # an exact copy longer than the windows,
    g.seqs[0][15_000:15_000 + len(src)] = synth.revcomp(src)  # and one in reverse
    b, off = g.concat()
    spans = list(g.spans) + [(0, 1_111, 1_111 + min_len + 3), (1, 5, len(g.seqs[1]) - 7)]
    ix = sdf.Index(g.seqs, k, w)
    orc = oracle_lib.OracleIndex(b, off, k, w)
    os_, oc = orc.search(spans, 0.25, min_len)
    with sdf.tuning(tile_threads=threads, hits_per_part=hits_per_part):
        r = ix.search_batch(spans, 0.25, min_len)
    _same(r.seeds(), os_, SEED_F, "seeds")
    _same(r.candidates(), oc, CAND_F, "candidates")
    assert len(oc) > 0
    ix.close()


# windows of up to 128, 256 and more minimizers (sorts of two and four keys per
# lane, the second launch), keys of 32 and 64 bits (k <= 12, above), and runs
# that repeat hashes
@pytest.mark.parametrize("k,w,min_len", [(12, 16, 900), (12, 16, 1400), (12, 16, 2000),
                                         (12, 10, 1400), (13, 16, 900), (14, 9, 1200),
                                         (12, 16, 3100), (11, 4, 700)])
def test_estimate_windows(oracle_lib, k, w, min_len):
    from paper_1807_00205_amd import sdf
    g = synth.tandem_case(2000 + 31 * k + w + min_len, length=26_000, n_arrays=10, copies_hi=12,
                          n_seqs=2, n_sd=4)
    src = g.seqs[0][2_000:2_000 + 2 * min_len]
    g.seqs[1][9_000:9_000 + len(src)] = src
    g.seqs[0][15_000:15_000 + len(src)] = synth.revcomp(src)
    b, off = g.concat()
    ix = sdf.Index(g.seqs, k, w)
    orc = oracle_lib.OracleIndex(b, off, k, w)
    os_, oc = orc.search(g.spans, 0.25, min_len, estimate=True)
    r = ix.search_batch(g.spans, 0.25, min_len, estimate=True)
    _same(r.seeds(), os_, SEED_F, "seeds")
    _same(r.candidates(), oc, CAND_F, "candidates")
    assert len(oc) > 0
    ix.close()


@pytest.mark.parametrize("min_len", [1000, 1200, 2000])
def test_autotune_times_the_schedule_in_use(min_len):
    """The schedule that a search takes by itself is among the timed ones, after
    the listed ones where it is none of these, and the fastest of all is returned
    (windows of 1,035 bases are the longest that the 512-thread layout holds)."""
    import ctypes
    from paper_1807_00205_amd import sdf
    g = synth.config1()
    ix = sdf.Index(g.seqs, 12, 16)
    listed = [(1024, c) for c in range(512, 1025, 64)] + [(512, 512)] * (min_len * 0.75 <= 1035)
    for core in (192, 512):
        with sdf.tuning(tile_threads=1024, tile_core=core):
            ms = (ctypes.c_float * 16)(*[-1.0] * 16)
            out, p = sdf._Tuning(), sdf._SearchParams(0.25, min_len, 0)
            arr, n = sdf._span_array([(0, 0, 300_000)])
            sdf._check(sdf.lib().sdf_autotune(ix._h, arr.ctypes.data_as(ctypes.c_void_p), n,
                                              ctypes.byref(p), None, ctypes.byref(out), ms, 16))
            all_ = listed + ([(1024, core)] if core == 192 else [])
            assert sum(m > 0 for m in ms) == len(all_)
            assert (out.tile_threads, out.tile_core) == all_[int(np.argmin(ms[:len(all_)]))]
            best_core, best_threads, times = ix.autotune([(0, 0, 300_000)], 0.25, min_len)
            assert times[best_threads, best_core] == min(times.values())
            assert set(listed) <= set(times)
    ix.close()


# windows of 750 and 1,050 bases over diverged copies of a unit in a row: a block's
# minimizers repeat hashes one to four units back, through copies that lost them
@pytest.mark.parametrize("unit,min_len,w", [(171, 1000, 16), (350, 1000, 16), (600, 1000, 16),
                                            (350, 1400, 16), (350, 1400, 12)])
def test_rows_of_copies(oracle_lib, unit, min_len, w):
    from paper_1807_00205_amd import sdf
    rng = synth.rng_for(unit + min_len + w)
    seqs = [synth.random_bases(rng, 9_000) for _ in range(2)]
    one = synth.random_bases(rng, unit)
    row = np.concatenate([synth.mutate(rng, one, 0.06) for _ in range(5_000 // unit)])
    seqs[0][1_000:1_000 + len(row)] = row
    half = np.concatenate([synth.mutate(rng, one, 0.06) for _ in range(2_500 // unit)])
    seqs[1][3_000:3_000 + len(half)] = synth.revcomp(half)
    g = synth.Genome(seqs, [], [(0, 0, 9_000), (1, 0, 9_000)], "rows")
    b, off = g.concat()
    ix = sdf.Index(g.seqs, 12, w)
    os_, oc = oracle_lib.OracleIndex(b, off, 12, w).search(g.spans, 0.25, min_len)
    for threads in (512, 1024):
        with sdf.tuning(tile_threads=threads):
            r = ix.search_batch(g.spans, 0.25, min_len)
        _same(r.seeds(), os_, SEED_F, "seeds")
        _same(r.candidates(), oc, CAND_F, "candidates")
        r.close()
    assert len(oc) > 0
    ix.close()
