"""Calls of vf_verify where others share the GPU or the launch: captured and replayed, and two models at once.

vf_verify captured into a graph and replayed, for each of its ways through the library: the persistent kernel of the
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
from util_plan import persistent_plan
from test_gpu_persistent_rows import _model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,rows", [("narrow", 1), ("narrow", 48), ("two_passes_128", 17), ("two_passes_128", 33), ("two_passes_128", 56), ("two_passes_128", 66)])
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


def test_two_models_on_two_streams():
    """Calls that a launch per operation serves may overlap: neither needs the whole GPU."""
    name, rows = "two_passes_128", 56
    cfg, first, _, _, seqs, _, ctx = _model(name)
    assert persistent_plan(first.cfg, rows)[0] is None
    w = vf.upload_weights(wl.make_weights(cfg, wl.streams(cfg).weights), cfg.dtype, DEV)
    models = [first, vf.vf_model_create(first.cfg, w, DEV)]
    seqs = [seqs, [vf.vf_seq_create(models[1], 1024) for _ in range(2)]]
    for a, b in zip(*seqs):
        b.kv.copy_(a.kv)
    ids = i32(wl.make_context(cfg.vocab, rows, np.random.default_rng(3)))
    want = torch.empty((rows, cfg.vocab), dtype=torch.float32, device=DEV)
    for pair in seqs:
        for s in pair:
            vf.vf_seq_set_len(s, ctx)
    vf.vf_verify(models[0], seqs[0], ids, [0, rows // 2, rows], want)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in models]
    outs = [torch.zeros_like(want) for _ in models]
    torch.cuda.synchronize()
    for _ in range(20):
        for m, q, st, out in zip(models, seqs, streams, outs):
            with torch.cuda.stream(st):
                vf.vf_verify(m, q, ids, [0, rows // 2, rows], out)
    torch.cuda.synchronize()
    assert torch.equal(outs[0], want) and torch.equal(outs[1], want)
