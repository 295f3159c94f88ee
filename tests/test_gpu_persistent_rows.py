"""The persistent kernels at the edges of their tiles: rows that fill or just exceed a block, a staging round or a row group,
rows of the residual stream that take several passes or end within one, K splits of unequal length, one key part or
several.  Logits of every row against the oracle: two layers of bfloat16 arithmetic differ by the rounding of the
products' inputs, the stated 2e-2 of the largest logit; a wrong tile is off by the size of the logits."""
import numpy as np
import pytest
import torch

import workloads as wl
import oracle
import paper_2510_15312_amd as vf
from oracle.transformer import forward
from util_gpu import DEV, i32
from util_oracle import rel_inf, spec_of, weights_of

pytestmark = pytest.mark.gpu
_cache = {}

# name: dimensions, context (keys before the rows of the call)
MODELS = {
    "narrow": (dict(d_model=320, n_q_heads=5, n_kv_heads=1, head_dim=64, d_ffn=992, vocab=1040), 600),
    "two_passes_64": (dict(d_model=1600, n_q_heads=10, n_kv_heads=2, head_dim=64, d_ffn=2080, vocab=1040), 70),
    "two_passes_128": (dict(d_model=2048, n_q_heads=12, n_kv_heads=4, head_dim=128, d_ffn=4128, vocab=2064), 300),
    # rows of the residual stream of more than two passes of the norm: up to 8 of them fit LDS
    "widest": (dict(d_model=8256, n_q_heads=6, n_kv_heads=2, head_dim=64, d_ffn=992, vocab=1040), 70),
}
VERIFY = (1, 7, 8, 9, 16, 17, 24, 25, 32, 33)   # two_passes_128: 32 rows are the most that LDS takes
BATCH = (34, 47, 48, 49, 63, 64, 65, 66)        # two sequences; from 65 rows on a launch per operation


def _model(name):
    if name not in _cache:
        _cache.clear()
        dims, ctx = MODELS[name]
        cfg = wl.scaled(wl.CONFIGS["1.5b_k16"], n_layers=2, **dims)
        wd = wl.make_weights(cfg, wl.streams(cfg).weights)
        model = vf.vf_model_create(vf.config_from(cfg, 128, 1024), vf.upload_weights(wd, cfg.dtype, DEV), DEV)
        spec, w32 = spec_of(cfg), weights_of(wd, np.float32)
        seqs = [vf.vf_seq_create(model, 1024) for _ in range(2)]
        ids = wl.make_context(cfg.vocab, ctx, np.random.default_rng(7))
        cache = oracle.KVCache(spec, 1024, np.float32)
        forward(spec, w32, cache, ids, np.float32)
        # the same keys and values on both sides
        for layer in range(cfg.n_layers):
            k, v = (np.ascontiguousarray(c[layer, :, :ctx].transpose(1, 0, 2)) for c in (cache.k, cache.v))
            for seq in seqs:
                vf.vf_kv_write(model, seq, layer, 0, torch.as_tensor(k, device=DEV), torch.as_tensor(v, device=DEV))
        _cache[name] = cfg, model, spec, w32, seqs, cache, ctx
    return _cache[name]


def _want(name, rows, seed=0):
    cfg, _, spec, w32, _, cache, ctx = _model(name)
    ids = wl.make_context(cfg.vocab, rows, np.random.default_rng((rows, seed)))
    cache.len = ctx
    z = forward(spec, w32, cache, ids, np.float32)
    cache.len = ctx
    return ids, z


@pytest.mark.parametrize("name,rows", [(n, r) for n in MODELS for r in VERIFY])
def test_verify_logits_against_oracle(name, rows):
    cfg, model, _, _, (seq, _), _, ctx = _model(name)
    ids, z = _want(name, rows)
    out = torch.empty((rows, cfg.vocab), dtype=torch.float32, device=DEV)
    again = torch.empty_like(out)
    vf.vf_seq_set_len(seq, ctx)
    vf.vf_verify(model, [seq], i32(ids), [0, rows], out)
    vf.vf_verify(model, [seq], i32(ids[:1]), [0, 1], torch.empty((1, cfg.vocab), dtype=torch.float32, device=DEV))
    vf.vf_verify(model, [seq], i32(ids), [0, rows], again)
    err = rel_inf(out.cpu().numpy(), z).max()
    print(f"{name}, {rows} rows: {err:.2e}", flush=True)
    assert err < 2e-2
    assert torch.equal(out, again)   # nothing of a launch is left for the next


@pytest.mark.parametrize("persistent", [1, 0])
@pytest.mark.parametrize("name,rows", [(n, r) for n in MODELS for r in BATCH])
def test_batch_logits_against_oracle(name, rows, persistent):
    cfg, model, _, _, seqs, _, ctx = _model(name)
    first = rows // 2
    (ids_a, z_a), (ids_b, z_b) = _want(name, first, 1), _want(name, rows - first, 2)
    out = torch.empty((rows, cfg.vocab), dtype=torch.float32, device=DEV)
    for seq in seqs:
        vf.vf_seq_set_len(seq, ctx)
    vf.vf_set_option(model, vf.VF_OPT_PERSISTENT, persistent)
    try:
        vf.vf_verify(model, seqs, i32(np.concatenate([ids_a, ids_b])), [0, first, rows], out)
    finally:
        vf.vf_set_option(model, vf.VF_OPT_PERSISTENT, 1)
    err = rel_inf(out.cpu().numpy(), np.concatenate([z_a, z_b])).max()
    print(f"{name}, {rows} rows: {err:.2e}", flush=True)
    assert err < 2e-2
