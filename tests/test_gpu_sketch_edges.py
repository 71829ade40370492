"""Window sketches and tables against the oracle at the sizes where the sketch
code branches: strides of one, two and four k-mers a lane and their
neighbours, sketches of 1 to 64 elements (up to 32 of them take the two-window
path, whose threshold is moved when it passes too few or too many hashes),
partial last windows of every length, repeated motifs (fewer distinct hashes
than candidates), unknown bases.

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


def sequences(k, w, s):
    S = w - k + 1
    rng = np.random.default_rng(k * 7 + w * 3 + s)
    out = []
    for tail in [0, 1, 2, s - 1, s, s + 1, 31, 32, 33, 63, 64, 65, S - 1]:   # k-mers of the last window
        out.append(synth.random_text(rng, 4 * S + k - 1 + max(tail, 0)))
    out.append(np.tile(synth.random_text(rng, 23), 40))           # few distinct k-mers
    out.append(np.tile(synth.random_text(rng, 60), 12))
    out.append(np.concatenate([np.tile(synth.random_text(rng, 9), 30), synth.random_text(rng, 500)]))
    t = synth.random_text(rng, 3000)
    t[rng.random(t.size) < 0.01] = ord("N")
    t[1200:1200 + w] = ord("N")
    out.append(t)
    out.append(synth.random_text(rng, 40 * S))                    # several whole tiles
    return out


@pytest.mark.parametrize("k,w,s", [(16, 47, 32), (16, 48, 33), (16, 79, 32), (16, 79, 16),
                                   (16, 80, 16), (16, 143, 32), (16, 143, 31), (16, 144, 16),
                                   (16, 271, 64), (11, 128, 1), (16, 128, 24), (3, 90, 20)])
def test_sketches_and_tables(torch, k, w, s):
    seqs = sequences(k, w, s)
    lengths = np.array([x.size for x in seqs], np.uint64)
    text = np.concatenate(seqs)
    d_text = torch.from_numpy(text.copy()).cuda()
    db = mc.Database(k, w, s, 254)
    nw = [orc.num_windows(int(L), k, w) for L in lengths]
    counts = torch.zeros(sum(nw), dtype=torch.int32, device="cuda")
    feats = torch.zeros(sum(nw) * s, dtype=torch.int32, device="cuda")
    mc.mc_db_sketch(db.h, d_text, lengths, counts, feats)
    torch.cuda.synchronize()
    counts = counts.cpu().numpy().view(np.uint32)
    feats = feats.cpu().numpy().view(np.uint32)
    g = 0
    for n, x in enumerate(seqs):
        for j, want in enumerate(orc.sketch_windows(x, k, w, s)):
            got = feats[g * s:g * s + counts[g]].tolist()
            assert got == want, (n, j)
            g += 1
    # the build's own emission and the query's sketches of the same text
    taxa = np.arange(1, len(seqs) + 1, dtype=np.uint32)
    parents = np.zeros(len(seqs) + 1, np.uint32)
    odb = orc.OracleDB(k, w, s, 254)
    odb.add_targets(text, lengths, taxa, threads=8)
    odb.set_taxonomy(parents)
    db.add_targets(d_text, lengths, taxa)
    db.set_taxonomy(parents)
    gf, gl = db.dump()
    of, ol = odb.dump()
    assert np.array_equal(gf, of) and np.array_equal(gl, ol)
    off = np.zeros(lengths.size + 1, np.uint64)
    off[1:] = np.cumsum(lengths)
    want, want_top = odb.classify(text, off, threads=8, min_hits=1)
    lab, top = db.classify(d_text, torch.from_numpy(off.view(np.int64).copy()).cuda(), len(seqs),
                           min_hits=1, with_top=True)
    torch.cuda.synchronize()
    assert np.array_equal(lab.cpu().numpy().view(np.uint32), want)
    assert np.array_equal(top.cpu().numpy().view(np.uint32), want_top)
