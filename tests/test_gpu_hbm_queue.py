"""The queue of records whose candidate list outgrows the large-list pass: its
workgroups share it at the end of that pass, with four regions of scratch (one
in the allocation-free call). Few and many queued records, none, and calls,
graph replays and the allocation-free call in turn on the same database: every
call finds the queue's counts as it expects them.

All arithmetic is integer: results must be equal.
"""
import numpy as np
import pytest

import oracle as orc
import paper_2106_08150_amd as mc
from paper_2106_08150_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def setup():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = synth.repeated_genome(1100, 600, seed=3)          # a window's 16 features: 17,600 locations
    gdb, odb = mc.Database(16, 128, 16, 65535), orc.OracleDB(16, 128, 16, 65535)
    gdb.add_targets(torch.from_numpy(g.text.copy()).cuda(), g.lengths, g.taxa)
    odb.add_targets(g.text, g.lengths, g.taxa, threads=8)
    for db in (gdb, odb):
        db.set_taxonomy(g.parents)
    return torch, g, gdb, odb


def batch(torch, g, odb, n, huge):
    """n records, the first `huge` of them with more than 16,384 locations."""
    g0, rng = g.genome(0), np.random.default_rng(n + huge)
    pieces = []
    for i in range(n):
        at = int(rng.integers(0, 400))
        pieces.append(g0[at:at + 128 + i % 60] if i < huge else synth.random_text(rng, 100))
    off = np.zeros(n + 1, np.uint64)
    off[1:] = np.cumsum([p.size for p in pieces])
    text = np.concatenate(pieces)
    want = odb.classify(text, off, threads=8)
    return (torch.from_numpy(text.copy()).cuda(),
            torch.from_numpy(off.view(np.int64).copy()).cuda(), want)


# queued records: none, one, fewer and more than the regions, one more than the
# workgroups of the pass
@pytest.mark.parametrize("condense", [False, True])
def test_shared_queue(setup, condense):
    torch, g, gdb, odb = setup
    if condense:
        gdb.condense(release_table=True)
    opts = mc.QueryOpts(4, 4, 0, 0, 0)
    before = gdb.stats()["q_hbm_records"]
    for n, huge in ((40, 0), (40, 1), (40, 3), (40, 5), (600, 513), (20, 0), (9, 9)):
        r, o, (want, want_top) = batch(torch, g, odb, n, huge)
        lab = torch.empty(n, dtype=torch.int32, device="cuda")
        top = torch.empty((n, 4, 3), dtype=torch.int32, device="cuda")
        graph = mc.ClassifyGraph(gdb.h, r, o, n, opts, lab, top)

        def eager():
            a, b = gdb.classify(r, o, n, with_top=True)
            lab.copy_(a)
            top.copy_(b)
        calls = (eager, graph.launch, graph.launch,
                 lambda: mc.mc_classify_noalloc(gdb.h, r, o, n, opts, lab, top), eager)
        for i, call in enumerate(calls):
            lab.fill_(-7)
            top.fill_(-7)
            torch.cuda.synchronize()
            call()
            torch.cuda.synchronize()
            assert np.array_equal(lab.cpu().numpy().view(np.uint32), want), (n, huge, i)
            assert np.array_equal(top.cpu().numpy().view(np.uint32), want_top), (n, huge, i)
    assert gdb.stats()["q_hbm_records"] > before
    assert mc.mc_db_query_status(gdb.h) == 0
