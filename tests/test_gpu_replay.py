"""vf_verify captured into a graph and replayed, for each of its ways through the library: the persistent kernel of the
whole pass, the one of the layers alone, and a launch per operation.  Eager calls of another size run between the
replays; every replay gives the eager call's logits bit for bit, and so does an eager call behind them.  A sequence that
has changed its length on the device is read at that length."""
import numpy as np
import pytest
import torch

import workloads as wl
import paper_2510_15312_amd as vf
from util_gpu import DEV, i32
from util_oracle import rel_inf
from test_gpu_persistent_rows import _model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,rows", [("narrow", 1), ("narrow", 48), ("two_passes_128", 17), ("two_passes_128", 33), ("two_passes_128", 66)])
def test_replay_equals_eager(name, rows):
    cfg, model, _, _, seqs, _, ctx = _model(name)
    off = [0, rows] if rows <= 33 else [0, rows // 2, rows]
    seqs = seqs[:len(off) - 1]
    rng = np.random.default_rng(rows)
    ids, other = i32(wl.make_context(cfg.vocab, rows, rng)), i32(wl.make_context(cfg.vocab, 5, rng))
    eager, out = (torch.empty((rows, cfg.vocab), dtype=torch.float32, device=DEV) for _ in range(2))
    small = torch.empty((5, cfg.vocab), dtype=torch.float32, device=DEV)

    def at(n):
        for s in seqs:
            vf.vf_seq_set_len(s, n)

    at(ctx)
    vf.vf_verify(model, seqs, ids, off, eager)   # also what a first call sets up
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        vf.vf_verify(model, seqs, ids, off, out)
    for i in range(4):
        out.zero_()
        if i % 2:
            vf.vf_verify(model, seqs[:1], other, [0, 5], small)
        graph.replay()
        if i > 1:
            graph.replay()   # two in a row
        torch.cuda.synchronize()
        assert torch.equal(out, eager), f"replay {i}"
    out.zero_()
    vf.vf_verify(model, seqs, ids, off, out)
    assert torch.equal(out, eager)

    at(ctx - 37)
    vf.vf_verify(model, seqs, ids, off, eager)
    graph.replay()
    assert rel_inf(out.cpu().numpy(), eager.cpu().numpy()).max() < 2e-2
    at(ctx)
    vf.vf_seq_get_state(seqs[0])   # raises if a barrier gave up
