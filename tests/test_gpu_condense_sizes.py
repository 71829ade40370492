"""Conversion to the condensed layout at the sizes where its slices, bins and
index buckets end, against the oracle: dense tables (slices past the usual
form's entries), features with thousands of locations (bins that are sorted,
chains past a slice's held slots, whole index buckets per slice), features
carried past their slice's index buckets (a list that is first too short).

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


def clustered(seed=71):
    return synth.clustered_genomes(5, 6, 6e6, seed=seed, median_bp=2e5, clip=(3e3, 8e5))


CASES = {
    # name: (genomes, k, w, s, cap, load factor, first deferred-list size)
    "default": (clustered, 16, 128, 16, 254, 0.0, 0),
    "dense": (clustered, 16, 128, 16, 254, 0.9, 0),
    "dense_short_list": (clustered, 16, 128, 16, 254, 0.9, 1),
    "sparse": (clustered, 16, 128, 16, 254, 0.01, 1),
    "large_sketch": (clustered, 16, 200, 64, 254, 0.7, 1),
    "copies_40": (lambda: synth.repeated_genome(40, 30_000, seed=5), 16, 128, 16, 254, 0.8, 1),
    "copies_300": (lambda: synth.repeated_genome(300, 20_000, seed=6), 16, 128, 16, 254, 0.5, 1),
    "copies_1500": (lambda: synth.repeated_genome(1500, 1_500, seed=7), 16, 128, 16, 65535, 0.1, 1),
    "one_window": (lambda: synth.repeated_genome(3, 130, seed=8), 16, 128, 16, 254, 0.0, 0),
}


@pytest.mark.parametrize("name", list(CASES))
def test_condense_sizes(torch, name):
    make, k, w, s, cap, load, defer = CASES[name]
    g = make()
    gdb = mc.Database(k, w, s, cap)
    odb = orc.OracleDB(k, w, s, cap)
    odb.add_targets(g.text, g.lengths, g.taxa, threads=8)
    odb.set_taxonomy(g.parents)
    of, ol = odb.dump()
    if load:
        gdb.reserve(of.size, load)
    if defer:
        mc.mc_db_set_insert_path(gdb.h, defer_entries=defer)
    gdb.add_targets(dev(torch, g.text), g.lengths, g.taxa)
    gdb.set_taxonomy(g.parents)
    reads = synth.sample_reads(g, 1500, 100 if g.lengths.min() > 100 else 60, seed=9, foreign=0.1)
    want, want_top = odb.classify(reads.text, reads.offsets, threads=8, min_hits=1)
    r, o = dev(torch, reads.text), dev(torch, reads.offsets, np.uint64)
    for release in (False, True):
        gdb.condense(release_table=release)
        lab, top = gdb.classify(r, o, reads.n_records, min_hits=1, with_top=True)
        torch.cuda.synchronize()
        assert np.array_equal(lab.cpu().numpy().view(np.uint32), want)
        assert np.array_equal(top.cpu().numpy().view(np.uint32), want_top)
    # the layout holds exactly the oracle's pairs
    cf, cl = gdb.dump()
    assert np.array_equal(cf, of) and np.array_equal(cl, ol)
    st = gdb.stats()
    assert st["n_pairs_stored"] == of.size and st["n_features"] == odb.num_features
