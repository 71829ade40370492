"""Large-list pass (one workgroup a record) against the oracle, at the sizes
where its sort, its feature buffer and its list end.

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


def dev(torch, a, dtype=np.uint8):
    a = np.ascontiguousarray(a, dtype=dtype)
    if dtype == np.uint64:
        a = a.view(np.int64)
    return torch.from_numpy(a.copy()).cuda()


def both(torch, g, k=16, w=128, s=16, cap=65535):
    gdb = mc.Database(k, w, s, cap)
    gdb.add_targets(dev(torch, g.text), g.lengths, g.taxa)
    gdb.set_taxonomy(g.parents)
    odb = orc.OracleDB(k, w, s, cap)
    odb.add_targets(g.text, g.lengths, g.taxa, threads=8)
    odb.set_taxonomy(g.parents)
    return gdb, odb


def check(torch, gdb, odb, pieces, paired=False, **opts):
    off = np.zeros(len(pieces) + 1, np.uint64)
    off[1:] = np.cumsum([p.size for p in pieces])
    text = np.concatenate(pieces)
    n = len(pieces) // (2 if paired else 1)
    ol, ot = odb.classify(text, off, paired=paired, threads=8, **opts)
    r, o = dev(torch, text), dev(torch, off, np.uint64)
    for shape in ((256, 4, 16384), (1024, 2, 16384)):
        mc.mc_db_set_launch_config(gdb.h, *shape)
        lab, top = gdb.classify(r, o, n, paired=paired, with_top=True, **opts)
        labels_only, _ = gdb.classify(r, o, n, paired=paired, **opts)
        torch.cuda.synchronize()
        assert np.array_equal(lab.cpu().numpy().view(np.uint32), ol)
        assert np.array_equal(top.cpu().numpy().view(np.uint32), ot)
        assert np.array_equal(labels_only.cpu().numpy().view(np.uint32), ol)
    assert mc.mc_db_query_status(gdb.h) == 0


# a one-window read of c identical genomes gathers 16 c locations: just over
# the fast paths' capacities, the sort's sizes and one past them, the largest
# list and the first one that the HBM-list pass takes
@pytest.mark.parametrize("condense", [False, True])
@pytest.mark.parametrize("copies", [17, 33, 64, 65, 128, 129, 257, 512, 513, 1023, 1024, 1025])
def test_list_sizes(torch, copies, condense):
    g = synth.repeated_genome(copies, 700, seed=copies)
    gdb, odb = both(torch, g)
    if condense:
        gdb.condense(release_table=True)
    g0 = g.genome(0)
    pieces = [g0[:128], g0[113:241], g0[60:170], g0[100:128], g0[:700], g0[5:300],
              synth.reverse_complement_text(g0[200:330])]
    check(torch, gdb, odb, pieces, top_m=8, min_hits=1, hit_diff=2)
    check(torch, gdb, odb, [g0[:128], g0[300:450], g0[226:354], g0[:0]], paired=True,
          insert_size=500)


# long records: many windows (several rounds of the feature buffer for large
# sketches), ragged lengths, unknown bases, foreign records without a location;
# strides of one, two and four k-mers a lane
@pytest.mark.parametrize("condense", [False, True])
@pytest.mark.parametrize("k,w,s", [(16, 128, 16), (16, 48, 16), (16, 200, 64), (12, 260, 3)])
def test_long_records(torch, k, w, s, condense):
    g = synth.clustered_genomes(3, 8, 6e5, seed=k + w, median_bp=25_000, clip=(14_000, 60_000))
    gdb, odb = both(torch, g, k, w, s, 254)
    if condense:
        gdb.condense()
    rng = np.random.default_rng(s)
    pieces = []
    for i, L in enumerate([900, 1501, 3000, 4999, 7000, 9001, 12_000, 13_777, 1200, 2500]):
        t = g.genome(i % 24)[i:i + L].copy()
        t = synth.substitute(rng, t, 0.01)
        if i % 3 == 0:
            t[L // 2:L // 2 + 37] = ord("N")
        pieces.append(synth.reverse_complement_text(t) if i % 2 else t)
    pieces.append(synth.random_text(rng, 8000))
    pieces.append(np.concatenate([g.genome(0)[:6000], g.genome(9)[:6000]]))
    check(torch, gdb, odb, pieces, top_m=4, min_hits=4)
    check(torch, gdb, odb, pieces, paired=True, top_m=3, min_hits=2, hit_diff=5,
          insert_size=15_000)
