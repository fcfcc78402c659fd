"""Final SDs where the split of the work can go wrong (aligner, seeds, chaining,
records), against the oracle.  Whole numbers and CIGARs: equality."""
import numpy as np
import pytest

from paper_1807_00205_amd import synth
from test_gpu_final_sd import _regions, _same

pytestmark = pytest.mark.gpu

GAPS = [(0, 3000), (3000, 0), (1, 2100), (62, 63), (63, 63), (64, 63), (63, 64), (127, 128),
        (128, 127), (255, 256), (256, 255), (300, 511), (520, 512), (513, 700), (1022, 1023),
        (1023, 1022), (1023, 1023), (1024, 1024), (20, 4500), (4500, 20), (600, 900)]


@pytest.mark.parametrize("cells", [None, 1, 4096])
def test_wave_aligner_sides(oracle_lib, cells):
    """Two copies flank unlike stretches of dx and dy bases: one stretch of
    that size in each region (every third one on the other strand)."""
    from paper_1807_00205_amd import sdf
    rng = synth.rng_for(77)
    q, t, rows, qp, tp = [], [], [], 0, 0
    for u, (dx, dy) in enumerate(GAPS):
        a, b = synth.random_bases(rng, 2500), synth.random_bases(rng, 2500)
        x = np.concatenate([a, synth.random_bases(rng, dx), b])
        y = np.concatenate([a, synth.random_bases(rng, dy), b])
        o = int(u % 3 == 2)
        if o:
            y = synth.revcomp(y)
        rows.append([qp, qp + len(x), tp, tp + len(y), o])
        q.append(x)
        t.append(y)
        qp += len(x)
        tp += len(y)
    for r in rows:
        r[2] += qp
        r[3] += qp
    seqs = [np.concatenate(q), np.concatenate(t)]
    b = np.concatenate(seqs)
    off = np.array([0, qp, len(b)], np.uint64)
    ix = sdf.Index(seqs, 12, 16)
    kw = {} if cells is None else dict(align_wave_cells=cells)
    with sdf.tuning(**kw):
        got = ix.align_regions(_regions(sdf, rows, off), 11, 1000, 0.25, pad_frac=0.0)
    want = oracle_lib.sd_align(b, off, [tuple(r) for r in rows], 11, 1000, 0.25, pad_frac=0.0)
    assert len(want[0]) >= len(GAPS)
    _same(got, want, "sides, cells %s" % cells)


@pytest.mark.parametrize("nt", [10, 11, 12, 15_369, 15_370, 15_371, 33_000])
@pytest.mark.parametrize("strand", [0, 1])
def test_seed_tiles(oracle_lib, nt, strand):
    """Target sides around the edges of the seeds' rounds (15,360 starts of 11
    bases) and query sides around the 16,384 positions of a workgroup: copies
    across the edge, gap bases, and a k-mer that occurs 32, 33 or far more
    times, within a round and over two."""
    from paper_1807_00205_amd import sdf
    rng = synth.rng_for(nt)
    t = synth.random_bases(rng, max(nt, 40))
    q = synth.random_bases(rng, 33_100)
    unit = synth.random_bases(rng, 11)
    if nt > 1_000:
        for u in range(33):                          # 33 in all, the last in a later round
            at = (u * 211) if u < 32 else nt - 400
            t[at + 50:at + 61] = unit
        t[7_000:8_500] = t[7_000]                    # one base: above the limit at once
        t[9_000:10_200] = np.tile(t[9_000:9_002], 600)
        t[12_000:12_003] = 4                         # gap bases
        src = t[nt - 6_000:nt] if nt < 20_000 else t[14_000:20_000]
        cp = synth.mutate(rng, src, 0.05)
        q[14_500:14_500 + len(cp)] = cp              # across the query's edge too
        q[2_000:3_500] = t[6_800:8_300]
        q[4_000:5_500] = t[8_900:10_400]
        q[20_500:20_700:100] = 4
        q[25_000:25_011] = unit
        q[26_000:28_000] = t[:2_000]
    t = t[:nt]
    if strand:
        t = synth.revcomp(t)
    seqs = [q, np.concatenate([t, synth.random_bases(rng, 64)])]
    b = np.concatenate(seqs)
    off = np.array([0, len(q), len(b)], np.uint64)
    rows = [(0, nq, len(q), len(q) + nt, strand) for nq in (10, 11, 16_384, 16_385, 16_400, 33_100)]
    ix = sdf.Index(seqs, 12, 16)
    got = ix.align_regions(_regions(sdf, rows, off), 11, 200, 0.25, pad_frac=0.0)
    want = oracle_lib.sd_align(b, off, rows, 11, 200, 0.25, pad_frac=0.0)
    assert len(want[0]) > 0 or nt < 1_000
    _same(got, want, "target side %d" % nt)


@pytest.mark.parametrize("unit,copies", [(300, 28), (97, 31), (1_500, 12)])
@pytest.mark.parametrize("strand", [0, 1])
def test_crowded_region(oracle_lib, unit, copies, strand):
    """Diverged copies of a unit in a row on both sides: most pairs of chains
    are in reach of each other, many with equal values."""
    from paper_1807_00205_amd import sdf
    rng = synth.rng_for(unit)
    one = synth.random_bases(rng, unit)
    q = np.concatenate([synth.mutate(rng, one, 0.04) for _ in range(copies)])
    t = np.concatenate([synth.mutate(rng, one, 0.04) for _ in range(copies)])
    if strand:
        t = synth.revcomp(t)
    b = np.concatenate([q, t])
    off = np.array([0, len(q), len(b)], np.uint64)
    rows = [(0, len(q), len(q), len(b), strand), (0, len(q) // 2, len(q), len(b), strand)]
    ix = sdf.Index([q, t], 12, 16)
    got = ix.align_regions(_regions(sdf, rows, off), 11, 300, 0.25, pad_frac=0.0)
    want = oracle_lib.sd_align(b, off, rows, 11, 300, 0.25, pad_frac=0.0)
    assert len(want[0]) > 0
    _same(got, want, "unit %d" % unit)


@pytest.mark.parametrize("seed", [919, 923, 962, 965, 966, 992, 996])
def test_equal_values_far_apart(oracle_lib, seed):
    """Copies apart by 8,000 unlike bases: the best chain goes over chance matches
    in between, and at some of them two predecessors that different waves meet
    give the same value.  The one that starts later is taken."""
    from paper_1807_00205_amd import sdf
    rng = synth.rng_for(seed)
    q, t = [], []
    for _ in range(8):
        cp = synth.random_bases(rng, 9_000)
        q += [cp, synth.random_bases(rng, 8_000)]
        t += [cp, synth.random_bases(rng, 8_000)]
    q, t = np.concatenate(q), np.concatenate(t + [synth.random_bases(rng, 100_000)])
    b = np.concatenate([q, t])
    off = np.array([0, len(q), len(b)], np.uint64)
    rows = [(0, len(q), len(q), len(b), 0)]
    ix = sdf.Index([q, t], 12, 16)
    got = ix.align_regions(_regions(sdf, rows, off), 11, 1000, 0.25, pad_frac=0.0)
    want = oracle_lib.sd_align(b, off, rows, 11, 1000, 0.25, pad_frac=0.0)
    assert len(want[0]) > 0
    _same(got, want, "equal values")


def _sides_with_copies(seed, length, strand):
    """Random sides with three copies of 8 to 20 kbp at 4, 10 and 16%."""
    rng = synth.rng_for(seed)
    q, t = synth.random_bases(rng, length), synth.random_bases(rng, length)
    for u, (ln, rate) in enumerate(((20_000, 0.10), (8_000, 0.16), (12_000, 0.04))):
        at, to = (2 * u + 1) * length // 7, (2 * u + 2) * length // 8
        cp = synth.mutate(rng, q[at:at + ln], rate)
        t[to:to + len(cp)] = cp
    return q, synth.revcomp(t) if strand else t


@pytest.mark.parametrize("length,strand", [(600_000, 0), (450_000, 1)])
def test_large_region(oracle_lib, length, strand):
    """A region of some 86,000 and 48,000 chance anchors: more than a thousand
    blocks per tier, and chains taken out over 17 doublings."""
    from paper_1807_00205_amd import sdf
    q, t = _sides_with_copies(length, length, strand)
    b = np.concatenate([q, t])
    off = np.array([0, length, 2 * length], np.uint64)
    ix = sdf.Index([q, t], 12, 16)
    reg = np.zeros(1, sdf.REGION_DTYPE)
    reg[0] = (strand, 0, 1, 0, 0, length, 0, length, 0, 0)
    rows = np.array([[0, length, length, 2 * length, strand]], np.uint64)
    _same(ix.align_regions(reg, pad_frac=0.0),
          oracle_lib.sd_align(b, off, rows, 11, 1000, 0.25, pad_frac=0.0), "large region")
    ix.close()


@pytest.mark.parametrize("strand", [0, 1])
def test_largest_side_records(oracle_lib, strand):
    """The largest sides (2^20 - 1 bases, some 260,000 chance anchors), which no
    plain restatement chains in seconds: every record's counts follow from its
    CIGAR and the bases, and the records are those that the oracle finds in
    pieces of 40 kbp around each copy (chains reach over 10 kbp at most)."""
    from paper_1807_00205_amd import sdf
    length = (1 << 20) - 1
    q, t = _sides_with_copies(5, length, strand)
    ix = sdf.Index([q, t], 12, 16)
    reg = np.zeros(1, sdf.REGION_DTYPE)
    reg[0] = (strand, 0, 1, 0, 0, length, 0, length, 0, 0)
    sd, ops = ix.align_regions(reg, pad_frac=0.0)
    ts = synth.revcomp(t) if strand else t
    code = np.zeros(256, np.uint8)
    code[list(b"ACGT")] = np.arange(4)
    for d in sd:
        x = int(d["q_begin"])
        y = int(length - d["t_end"] if strand else d["t_begin"])
        n = dict.fromkeys(("matches", "mismatches", "ins", "dels", "gap_opens", "transitions",
                           "transversions"), 0)
        last = None
        for v in ops[int(d["cigar_off"]):int(d["cigar_off"]) + int(d["cigar_len"])]:
            op, ln = int(v) & 15, int(v) >> 4
            assert ln > 0 and op != last
            a, c = code[q[x:x + ln]], code[ts[y:y + ln]]
            if op == 7:
                assert np.array_equal(a, c)
                n["matches"] += ln
            elif op == 8:
                assert np.all(a != c)
                n["mismatches"] += ln
                n["transitions"] += int(np.sum((a ^ c) == 2))
                n["transversions"] += int(np.sum((a ^ c) != 2))
            else:
                n["ins" if op == 1 else "dels"] += ln
                n["gap_opens"] += 1
            x += ln if op != 2 else 0
            y += ln if op != 1 else 0
            last = op
        assert x == d["q_end"] and y == (length - d["t_begin"] if strand else d["t_end"])
        assert all(int(d[f]) == n[f] for f in n), (n, d)
        assert d["aln_len"] == sum(n[f] for f in ("matches", "mismatches", "ins", "dels")) >= 1000
    # around each copy: what the oracle finds in the two pieces
    whole = ("aln_len", "matches", "mismatches", "ins", "dels", "gap_opens", "transitions",
             "transversions", "cigar_len")
    found = 0
    for u, ln in ((0, 20_000), (1, 8_000), (2, 12_000)):
        at, to = (2 * u + 1) * length // 7, (2 * u + 2) * length // 8
        a, e = at - 40_000, at + ln + 40_000
        c, f = to - 40_000, to + ln + 40_000
        if strand:
            c, f = length - f, length - c
        want, wops = oracle_lib.sd_align(
            np.concatenate([q[a:e], t[c:f]]), np.array([0, e - a, e - a + f - c], np.uint64),
            np.array([[0, e - a, e - a, e - a + f - c, strand]], np.uint64), 11, 1000, 0.25,
            pad_frac=0.0)
        for w in want:
            d = sd[sd["q_begin"] == w["q_begin"] + a]
            assert len(d) == 1
            for v, base in (("q_end", a), ("t_begin", c), ("t_end", c)):
                assert int(d[v][0]) == int(w[v]) + base, v
            assert all(int(d[v][0]) == int(w[v]) for v in whole)
            at_ = int(d["cigar_off"][0])
            assert np.array_equal(ops[at_:at_ + int(d["cigar_len"][0])],
                                  wops[int(w["cigar_off"]):int(w["cigar_off"]) + int(w["cigar_len"])])
            found += 1
    assert found == len(sd) == 3
    ix.close()


def test_regions_alone_and_together(oracle_lib):
    """Regions of a few to a few thousand anchors one at a time (their chains
    taken out by one workgroup), in pairs, and all in one call: the same records
    each time, the oracle's."""
    from paper_1807_00205_amd import sdf
    rng = synth.rng_for(31)
    sizes = (40, 400, 1_200, 4_000, 12_000, 30_000, 60_000, 90_000, 110_000, 130_000, 131_000, 132_000)
    q, t, rows, at = [], [], [], 0
    for u, ln in enumerate(sizes):
        a = synth.random_bases(rng, ln)
        b = synth.random_bases(rng, ln)
        cp = synth.mutate(rng, a[ln // 4:ln // 4 + min(ln // 2, 3_000)], 0.03 * (u % 4))[:ln // 2]
        b[ln // 3:ln // 3 + len(cp)] = cp
        q.append(a)
        t.append(synth.revcomp(b) if u % 2 else b)
        rows.append((at, at + ln, at, at + ln, u % 2))
        at += ln
    q, t = np.concatenate(q), np.concatenate(t)
    b = np.concatenate([q, t])
    off = np.array([0, at, 2 * at], np.uint64)
    rows = [(qb, qe, tb + at, te + at, o) for qb, qe, tb, te, o in rows]
    ix = sdf.Index([q, t], 12, 16)
    for part in [[r] for r in rows] + [rows[i:i + 2] for i in range(6, 12, 2)] + [rows]:
        got = ix.align_regions(_regions(sdf, part, off), 11, 300, 0.25, pad_frac=0.0)
        _same(got, oracle_lib.sd_align(b, off, part, 11, 300, 0.25, pad_frac=0.0), "%d regions" % len(part))
    ix.close()
