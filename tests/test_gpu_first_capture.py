"""The first classification on a stream captured by the caller (relaxed mode),
then plain calls and replays in turn: the workspace that the capture made is
ready for each of them.

All arithmetic is integer: results must be equal.
"""
import numpy as np
import pytest

import oracle as orc
import paper_2106_08150_amd as mc
from paper_2106_08150_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("replay_first", [False, True])
def test_first_call_captured(replay_first):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = synth.repeated_genome(300, 2_000, seed=11)      # lists past the fast pass's capacity
    reads = synth.sample_reads(g, 400, 150, seed=12, foreign=0.2)
    gdb, odb = mc.Database(), orc.OracleDB()
    gdb.add_targets(torch.from_numpy(g.text.copy()).cuda(), g.lengths, g.taxa)
    odb.add_targets(g.text, g.lengths, g.taxa, threads=8)
    for db in (gdb, odb):
        db.set_taxonomy(g.parents)
    want, want_top = odb.classify(reads.text, reads.offsets, threads=8)
    r = torch.from_numpy(reads.text.copy()).cuda()
    o = torch.from_numpy(reads.offsets.view(np.int64).copy()).cuda()
    n = reads.n_records
    lab = torch.empty(n, dtype=torch.int32, device="cuda")
    top = torch.empty((n, 4, 3), dtype=torch.int32, device="cuda")
    opts = mc.QueryOpts(4, 4, 0, 0, 0)
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()

    def plain():
        mc.mc_classify_ex(gdb.h, r, o, n, opts, lab, top, stream)

    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(stream):
        graph.capture_begin(capture_error_mode="relaxed")
        try:
            plain()
        finally:
            graph.capture_end()

    def replay():
        with torch.cuda.stream(stream):
            graph.replay()

    calls = [replay, plain] if replay_first else [plain, replay]
    for i, call in enumerate(calls + [plain, replay, replay, plain]):
        with torch.cuda.stream(stream):
            lab.fill_(-7)
            top.fill_(-7)
        torch.cuda.synchronize()
        call()
        torch.cuda.synchronize()
        assert np.array_equal(lab.cpu().numpy().view(np.uint32), want), i
        assert np.array_equal(top.cpu().numpy().view(np.uint32), want_top), i
    assert gdb.stats()["q_large_records"] > 0
