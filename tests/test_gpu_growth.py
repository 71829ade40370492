"""Table growth by additions against the oracle: many small steps and one large
one, dense tables, tombstones of capped features, features whose chains run
over slices (more entries in a slice than its workgroup holds, a deferred list
that is too short so that the growth starts over).

All arithmetic is integer: the stored pairs must be equal.
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


def clustered():
    return synth.clustered_genomes(6, 4, 4e6, seed=91, median_bp=1.5e5, clip=(3e3, 5e5))


def copies(n, length, seed):
    return lambda: synth.repeated_genome(n, length, seed=seed)


CASES = {
    # name: (genomes, cap, load factor, first targets of each addition, list size)
    "small_steps": (clustered, 254, 0.0, [0, 1, 2, 4, 6, 9, 13, 17, 21], 0),
    "small_steps_short_list": (clustered, 254, 0.0, [0, 1, 2, 4, 6, 9, 13, 17, 21], 1),
    "large_step": (lambda: synth.Genomes(*_tiny_first()), 254, 0.0, [0, 1], 0),
    "dense": (clustered, 254, 0.9, [0, 3, 8, 15], 0),
    "tombstones": (copies(40, 20_000, 3), 3, 0.0, [0, 10, 20, 30], 0),
    "copies": (copies(260, 12_000, 4), 254, 0.0, [0, 60, 130, 200], 0),
    "copies_short_list": (copies(260, 12_000, 4), 254, 0.0, [0, 60, 130, 200], 1),
    "copies_dense": (copies(260, 12_000, 5), 254, 0.9, [0, 100, 250], 0),
}


def _tiny_first():
    g = clustered()
    text = np.concatenate([g.text[:200], g.text])
    lengths = np.concatenate([np.array([200], np.uint64), g.lengths])
    taxa = np.concatenate([g.taxa[:1], g.taxa])
    return text, lengths, taxa, g.parents


@pytest.mark.parametrize("name", list(CASES))
def test_growth(torch, name):
    make, cap, load, starts, short = CASES[name]
    g = make()
    gdb, odb = mc.Database(16, 128, 16, cap), orc.OracleDB(16, 128, 16, cap)
    if load:
        gdb.reserve(1, load)
    if short:
        mc.mc_db_set_insert_path(gdb.h, defer_entries=short)
    off = g.offsets
    grown = []
    for a, b in zip(starts, starts[1:] + [g.lengths.size]):
        text = np.ascontiguousarray(g.text[int(off[a]):int(off[b])])
        gdb.add_targets(torch.from_numpy(text.copy()).cuda(), g.lengths[a:b], g.taxa[a:b])
        odb.add_targets(text, g.lengths[a:b], g.taxa[a:b], threads=8)
        grown.append(gdb.stats()["n_buckets"])
        gf, gl = gdb.dump()
        of, ol = odb.dump()
        assert np.array_equal(gf, of) and np.array_equal(gl, ol), f"after targets [{a}, {b})"
    assert len(set(grown)) > 1, "the table never grew"
    gdb.set_taxonomy(g.parents)
    odb.set_taxonomy(g.parents)
    reads = synth.sample_reads(g, 800, 100, seed=12)
    want, want_top = odb.classify(reads.text, reads.offsets, threads=8)
    r = torch.from_numpy(reads.text.copy()).cuda()
    o = torch.from_numpy(reads.offsets.view(np.int64).copy()).cuda()
    lab, top = gdb.classify(r, o, reads.n_records, with_top=True)
    torch.cuda.synchronize()
    assert np.array_equal(lab.cpu().numpy().view(np.uint32), want)
    assert np.array_equal(top.cpu().numpy().view(np.uint32), want_top)
