"""The fast query pass against the oracle at the sizes where its lookups and
its record headers branch: whole, partial and one-step batches of bucket lines
(1 to 130 features a record), buckets that are just full and chains over
several buckets, lists at both capacities, mates of which one is empty, and
offsets that do not ascend.

All arithmetic is integer: results must be equal.
"""
import numpy as np
import pytest

import oracle as orc
import paper_2106_08150_amd as mc
from paper_2106_08150_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as T
    if not T.cuda.is_available():
        pytest.skip("no GPU")
    return T


def both(torch, g, k, w, s):
    gdb, odb = mc.Database(k, w, s, 254), orc.OracleDB(k, w, s, 254)
    gdb.add_targets(torch.from_numpy(g.text.copy()).cuda(), g.lengths, g.taxa)
    odb.add_targets(g.text, g.lengths, g.taxa, threads=8)
    for db in (gdb, odb):
        db.set_taxonomy(g.parents)
    return gdb, odb


# copies: locations a feature (1 and 2: inline in the condensed layout; 7, 8,
# 15, 16, 17: around a full bucket's 16 slots with neighbours; 40: long chains)
@pytest.mark.parametrize("condense", [False, True])
@pytest.mark.parametrize("paired", [False, True])
@pytest.mark.parametrize("copies", [1, 2, 3, 7, 8, 15, 16, 17, 40])
def test_batches(torch, copies, paired, condense):
    k, w, s = 16, 64, 8                       # stride 49: up to 130 features in 820 bases
    g = synth.repeated_genome(copies, 4000, seed=copies)
    gdb, odb = both(torch, g, k, w, s)
    if condense:
        gdb.condense(release_table=True)
    g0, rng = g.genome(0), np.random.default_rng(copies)
    lens = list(range(15, 30)) + list(range(30, 830, 7))
    pieces = []
    for n in lens:
        at = int(rng.integers(0, 4000 - n))
        pieces.append(g0[at:at + n])
        if paired:                            # a second mate, every third one empty
            pieces.append(g0[at // 2:at // 2 + (0 if n % 3 == 0 else n // 2)])
    off = np.zeros(len(pieces) + 1, np.uint64)
    off[1:] = np.cumsum([p.size for p in pieces])
    text = np.concatenate(pieces)
    ol, ot = odb.classify(text, off, paired=paired, threads=8, min_hits=1)
    r, o = torch.from_numpy(text.copy()).cuda(), torch.from_numpy(off.view(np.int64).copy()).cuda()
    for lcap, wpb in ((256, 2), (256, 4), (512, 4), (1024, 2)):
        mc.mc_db_set_launch_config(gdb.h, lcap, wpb, 16384)
        lab, top = gdb.classify(r, o, len(lens), paired=paired, with_top=True, min_hits=1)
        torch.cuda.synchronize()
        assert np.array_equal(lab.cpu().numpy().view(np.uint32), ol)
        assert np.array_equal(top.cpu().numpy().view(np.uint32), ot)
    assert mc.mc_db_query_status(gdb.h) == 0


# a record whose offsets descend, also around 2^64, is left unclassified and
# its bytes are not read; its neighbours are classified as ever
@pytest.mark.parametrize("bad", [[500, 400], [(1 << 64) - 50, 100], [(1 << 63) + 7, 3]])
def test_offsets_that_do_not_ascend(torch, bad):
    g = synth.repeated_genome(2, 4000, seed=9)
    gdb, odb = both(torch, g, 16, 64, 8)
    text = g.genome(0)[:1200]
    off = np.array(bad + [550, 700, 850], np.uint64)
    good = [(1, bad[1], 550), (2, 550, 700), (3, 700, 850)]
    lab, _ = gdb.classify(torch.from_numpy(text.copy()).cuda(),
                          torch.from_numpy(off.view(np.int64).copy()).cuda(), 4, min_hits=1)
    torch.cuda.synchronize()
    lab = lab.cpu().numpy().view(np.uint32)
    assert lab[0] == 0xFFFFFFFF
    for n, a, b in good:
        want, _ = odb.classify(text[a:b], np.array([0, b - a], np.uint64), threads=1, min_hits=1)
        assert lab[n] == want[0]
    assert mc.mc_db_query_status(gdb.h) == 0
