"""Fragments longer than any target (insert sizes up to the largest value) with
windows of one k-mer: the range of windows a fragment can touch ends with its
target on every path (short list, sorted list, large-list pass), with no wrap of
the range's end.

All arithmetic is integer: results must be equal.
"""
import numpy as np
import pytest

import oracle as orc
import paper_2106_08150_amd as mc
from paper_2106_08150_amd import synth

pytestmark = pytest.mark.gpu

# copies of the genome and mate length: lists of about 30, 170 and 3,400 locations
PATHS = {"short": (1, 30), "sorted": (1, 100), "large": (20, 100)}


@pytest.mark.parametrize("condense", [False, True])
@pytest.mark.parametrize("path", list(PATHS))
def test_insert_size_past_every_target(path, condense):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    copies, mate = PATHS[path]
    g = synth.repeated_genome(copies, 1_500, seed=21)
    rng = np.random.default_rng(22)
    g0, n = g.genome(0), 40
    at = rng.integers(0, g0.size - 400, n)
    text = np.concatenate([np.concatenate([g0[a:a + mate], g0[a + 300:a + 300 + mate]]) for a in at])
    off = np.arange(0, (2 * n + 1) * mate, mate, dtype=np.uint64)
    gdb, odb = mc.Database(16, 16, 1, 254), orc.OracleDB(16, 16, 1, 254)
    gdb.add_targets(torch.from_numpy(g.text.copy()).cuda(), g.lengths, g.taxa)
    odb.add_targets(g.text, g.lengths, g.taxa, threads=8)
    for db in (gdb, odb):
        db.set_taxonomy(g.parents)
    if condense:
        gdb.condense()
    # any insert size past the longest target gives the whole target
    want, want_top = odb.classify(text, off, paired=True, insert_size=3_000, threads=8)
    r = torch.from_numpy(text.copy()).cuda()
    o = torch.from_numpy(off.view(np.int64).copy()).cuda()
    for insert in (3_000, (1 << 18) + 16, (1 << 31) + 5, 0xFFFFFDFF, 0xFFFFFE01, 0xFFFFFFFF):
        lab, top = gdb.classify(r, o, n, with_top=True, paired=True, insert_size=insert)
        torch.cuda.synchronize()
        assert np.array_equal(lab.cpu().numpy().view(np.uint32), want), insert
        assert np.array_equal(top.cpu().numpy().view(np.uint32), want_top), insert
