"""The inputs of the growth and conversion tests reach the paths they are meant
for: entries carried past their slice (more than the short lists hold, so that
a growth starts over and a conversion is repeated), slices with more entries
than a growth's workgroup holds, slices past the conversion's usual form.

The table's and the index's sizes come from the device; which entries leave
their slice follows from them and the stored pairs, computed here.
"""
import numpy as np
import pytest

import paper_2106_08150_amd as mc
import test_gpu_condense_sizes as sizes
import test_gpu_growth as growth

pytestmark = pytest.mark.gpu

SLICE = 256          # buckets of a slice
GROW_CAP = 3072      # entries a growth's workgroup holds
COND_MID = 2944      # entries of the conversion's usual form


@pytest.fixture(scope="module")
def torch():
    import torch as T
    if not T.cuda.is_available():
        pytest.skip("no GPU")
    return T


def h2(f):
    f = f.astype(np.uint32)
    f ^= f >> np.uint32(16)
    f *= np.uint32(0x7FEB352D)
    f ^= f >> np.uint32(15)
    f *= np.uint32(0x846CA68B)
    f ^= f >> np.uint32(16)
    return f


def home(f, n):
    return ((h2(f).astype(np.uint64) * np.uint64(n)) >> np.uint64(32)).astype(np.int64)


def carried(homes, n, per_slice, room):
    """Items carried past the end of their slice of per_slice buckets of `room`
    places, slice by slice (an item goes to its home or the next free place)."""
    count = np.bincount(homes, minlength=n).reshape(-1, per_slice)
    carry = np.zeros(count.shape[0], np.int64)
    for r in range(per_slice):
        carry = np.maximum(0, carry + count[:, r] - room)
    return carry, count.sum(axis=1)


# growth cases that put entries off (with a list of one: more than it holds) and
# have a slice over the workgroup's entries (clusters without repeats, as in
# small_steps, fill their slices evenly and put nothing off)
@pytest.mark.parametrize("name", ["copies", "copies_short_list", "copies_dense"])
def test_growth_inputs(torch, name):
    make, cap, load, starts, short = growth.CASES[name]
    g = make()
    db = mc.Database(16, 128, 16, cap)
    if load:
        db.reserve(1, load)
    off, most_off, most_in = g.offsets, 0, 0
    for a, b in zip(starts, starts[1:] + [g.lengths.size]):
        before = db.dump()[0]
        old_nb = db.stats()["n_buckets"]
        text = np.ascontiguousarray(g.text[int(off[a]):int(off[b])])
        db.add_targets(torch.from_numpy(text.copy()).cuda(), g.lengths[a:b], g.taxa[a:b])
        nb = db.stats()["n_buckets"]
        assert nb % SLICE == 0
        if nb == old_nb or before.size == 0:
            continue
        carry, held = carried(home(before, nb), nb, SLICE, 16)
        over = held > GROW_CAP
        most_off = max(most_off, int(carry[~over].sum() + held[over].sum()))
        most_in = max(most_in, int(held.max()))
    assert most_off > max(short, 1), "no growth puts off more entries than the list holds"
    assert most_in > GROW_CAP, "no slice with more entries than a workgroup holds"


def conversion(torch, name):
    make, k, w, s, cap, load, defer = sizes.CASES[name]
    g = make()
    db = mc.Database(k, w, s, cap)
    if load:
        import oracle as orc
        odb = orc.OracleDB(k, w, s, cap)
        odb.add_targets(g.text, g.lengths, g.taxa, threads=8)
        db.reserve(odb.dump()[0].size, load)
    db.add_targets(torch.from_numpy(np.ascontiguousarray(g.text).copy()).cuda(), g.lengths, g.taxa)
    f = db.dump()[0]
    nb = db.stats()["n_buckets"]
    n_slices = nb // SLICE
    feats = np.unique(f)
    per = max(1, -(-max(64, (feats.size + 3) // 4) // n_slices))
    deferred, _ = carried(home(feats, n_slices * per), n_slices * per, per, 8)
    return int(deferred.sum()), int(np.bincount(home(f, nb) // SLICE, minlength=n_slices).max())


def test_conversion_inputs(torch):
    short = [n for n, c in sizes.CASES.items() if c[6]]
    seen = {n: conversion(torch, n) for n in short + ["dense"]}
    assert any(seen[n][0] > sizes.CASES[n][6] for n in short), seen   # list made anew
    assert any(0 < v[0] for v in seen.values()), seen
    assert any(v[1] > COND_MID for v in seen.values()), seen          # large form
    assert any(v[1] <= COND_MID for v in seen.values()), seen         # usual form
