"""Final SDs where the aligner's and the seeds' split can go wrong, against the
oracle: stretches with the edges of 64, 128, 256 and 512 lines per lane group
on either side, and long thin ones.  Whole numbers and CIGARs: equality."""
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
