"""Records with more sketch elements than the fast pass's list holds: those of
unknown organisms have short lists and stay in the fast pass, those of stored
genomes go on to the large-list pass after a few windows, and records that
start as the one and end as the other are right on either path.

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
    g = synth.clustered_genomes(4, 3, 2e6, seed=31, median_bp=1.5e5, clip=(3e4, 4e5))
    gdb, odb = mc.Database(), orc.OracleDB()
    gdb.add_targets(torch.from_numpy(g.text.copy()).cuda(), g.lengths, g.taxa)
    odb.add_targets(g.text, g.lengths, g.taxa, threads=8)
    for db in (gdb, odb):
        db.set_taxonomy(g.parents)
    return torch, g, gdb, odb


def pieces(g, kind, rng, length):
    own = g.genome(int(rng.integers(0, g.lengths.size)))
    at = int(rng.integers(0, own.size - length))
    stored, foreign = own[at:at + length].copy(), synth.random_text(rng, length)
    half = length // 2
    return {"foreign": foreign, "stored": stored,
            "stored_first": np.concatenate([stored[:half], foreign[half:]]),
            "stored_last": np.concatenate([foreign[:half], stored[half:]])}[kind]


# list capacity and record lengths: 16 elements a window of 113 bases, so that
# the first records lie just past the capacity; from 8,192 bases on a record
# with more elements than that is handed on unseen
@pytest.mark.parametrize("condense", [False, True])
@pytest.mark.parametrize("cap", [256, 512, 1024])
def test_long_records(setup, cap, condense):
    torch, g, gdb, odb = setup
    if condense:
        gdb.condense()
    mc.mc_db_set_launch_config(gdb.h, cap, 4, 16384)
    rng = np.random.default_rng(cap + condense)
    edge = 113 * cap // 16 + 15
    looked_at = [edge - 113, edge, edge + 1, edge + 113, edge + 250, 5_000, 8_191]
    unseen = [8_192, 2 * edge + 7_000, 20_000]
    for kind in ("foreign", "stored", "stored_first", "stored_last"):
        for lengths in (looked_at, unseen):
            recs = [pieces(g, kind, rng, n) for n in lengths]
            off = np.zeros(len(recs) + 1, np.uint64)
            off[1:] = np.cumsum([r.size for r in recs])
            text = np.concatenate(recs)
            want, want_top = odb.classify(text, off, threads=8)
            before = gdb.stats()["q_large_records"]
            lab, top = gdb.classify(torch.from_numpy(text).cuda(),
                                    torch.from_numpy(off.view(np.int64).copy()).cuda(), len(recs),
                                    with_top=True)
            torch.cuda.synchronize()
            assert np.array_equal(lab.cpu().numpy().view(np.uint32), want), kind
            assert np.array_equal(top.cpu().numpy().view(np.uint32), want_top), kind
            passed_on = gdb.stats()["q_large_records"] - before
            if lengths is unseen:
                assert passed_on == len(unseen)
            elif kind == "foreign":
                assert passed_on == 0, "a short list needs no large-list pass"
            elif kind == "stored":
                assert passed_on > 0


def test_pairs_and_malformed(setup):
    """Pairs whose lengths together reach 8,192 bases, and offsets that descend
    by as much."""
    torch, g, gdb, odb = setup
    mc.mc_db_set_launch_config(gdb.h, 512, 4, 16384)
    rng = np.random.default_rng(5)
    sizes = [(4_095, 4_096), (4_096, 4_096), (8_191, 0), (0, 8_192), (100, 8_091), (100, 8_092),
             (3_000, 3_000)]
    recs = [pieces(g, k, rng, n + m) for n, m in sizes for k in ("foreign", "stored")]
    lens = np.repeat(np.array(sizes, np.uint64), 2, axis=0).reshape(-1)
    off = np.zeros(lens.size + 1, np.uint64)
    off[1:] = np.cumsum(lens)
    text = np.concatenate(recs)
    n = len(recs)
    want, want_top = odb.classify(text, off, paired=True, threads=8)
    r = torch.from_numpy(text).cuda()
    lab, top = gdb.classify(r, torch.from_numpy(off.view(np.int64).copy()).cuda(), n,
                            with_top=True, paired=True)
    torch.cuda.synchronize()
    assert np.array_equal(lab.cpu().numpy().view(np.uint32), want)
    assert np.array_equal(top.cpu().numpy().view(np.uint32), want_top)
    # a record whose offsets descend is unclassified and not counted as too long
    bad = np.array([9_000, 300, 600, 20_000, 11_000, 11_500], np.uint64)
    lab, _ = gdb.classify(r, torch.from_numpy(bad.view(np.int64).copy()).cuda(), 5)
    torch.cuda.synchronize()
    got = lab.cpu().numpy().view(np.uint32)
    for i, (a, b) in enumerate(zip(bad[:-1], bad[1:])):
        if b < a:
            assert got[i] == 0xFFFFFFFF
        else:
            one = odb.classify(text[int(a):int(b)], np.array([0, b - a], np.uint64))[0]
            assert got[i] == one[0]
    assert mc.mc_db_query_status(gdb.h) == 0
