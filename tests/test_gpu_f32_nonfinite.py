"""The float32 attention where numbers are not ordinary ones.  A row takes nothing from a row it does not see: an
infinity or NaN in a later row of a chunk, or in a sibling of a token tree, leaves it as it is (compared with the
same call with an ordinary token in that place, to the 1e-5 of the float32 path).  And a row whose scores all lie
below -1e30 still has a softmax: against the float64 oracle, which is one-hot there."""
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
BAD = 7   # the token whose embedding is not finite


def _model(hd, value):
    cfg = wl.scaled(wl.CONFIGS["tiny_f32"], n_layers=2, d_model=128, n_q_heads=4, n_kv_heads=2, head_dim=hd, d_ffn=256, vocab=512)
    wd = wl.make_weights(cfg, wl.streams(cfg).weights, std=0.05)
    wd["embed"][BAD] = value
    return cfg, vf.vf_model_create(vf.config_from(cfg, 160, 2400), vf.upload_weights(wd, cfg.dtype, DEV), DEV)


def _start(model, ctx):
    seq = vf.vf_seq_create(model, 2400)
    if ctx:
        gen = torch.Generator(device=DEV).manual_seed(ctx)
        for layer in range(model.cfg.n_layers):
            kv = torch.randn((2, ctx, model.cfg.n_kv_heads, model.cfg.head_dim), device=DEV, generator=gen)
            vf.vf_kv_write(model, seq, layer, 0, kv[0], kv[1])
        vf.vf_seq_set_len(seq, ctx)
    return seq


# context 2100: 66 key tiles, two key parts
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("hd,ctx,rows,at", [(64, 0, 40, 21), (64, 100, 70, 3), (128, 45, 33, 32), (128, 2100, 20, 9)])
def test_later_rows_of_a_chunk(hd, ctx, rows, at, value):
    cfg, model = _model(hd, value)
    ids = wl.make_context(cfg.vocab, rows, np.random.default_rng(rows))
    ids[ids == BAD] = BAD + 1
    got = []
    for tok in (BAD, BAD + 1):
        ids[at] = tok
        out = torch.empty((rows, cfg.vocab), dtype=torch.float32, device=DEV)
        vf.vf_prefill_chunk(model, _start(model, ctx), i32(ids), logits_mode=2, logits_out=out)
        got.append(np.delete(out.cpu().numpy(), BAD, axis=1))   # the tied output head gives that token no finite logit
    assert np.isfinite(got[0][:at]).all() and np.isfinite(got[1]).all()
    assert rel_inf(got[0][:at], got[1][:at]).max() < 1e-5
    assert not np.isfinite(got[0][at:]).any()   # rows that do see it


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_siblings_of_a_tree(value):
    cfg, model = _model(64, value)
    parents = [-1, 0, 0, 2, 1, 2, 3]
    unseen = [0, 2, 3, 5, 6]   # rows 1 and 4 are the bad node and its child
    ids = wl.make_context(cfg.vocab, 7, np.random.default_rng(1))
    ids[ids == BAD] = BAD + 1
    got = []
    for tok in (BAD, BAD + 1):
        ids[1] = tok
        out = torch.empty((7, cfg.vocab), dtype=torch.float32, device=DEV)
        vf.vf_verify_tree(model, [_start(model, 61)], i32(ids), [0, 7], parents, out)
        got.append(np.delete(out.cpu().numpy(), BAD, axis=1))
    assert np.isfinite(got[0][unseen]).all()
    assert rel_inf(got[0][unseen], got[1][unseen]).max() < 1e-5
    assert not np.isfinite(got[0][[1, 4]]).any()


@pytest.mark.parametrize("hd", [64, 128])
def test_scores_far_below_zero(hd):
    cfg = wl.scaled(wl.CONFIGS["tiny_f32"], n_layers=1, d_model=128, n_q_heads=2, n_kv_heads=2, head_dim=hd, d_ffn=256, vocab=512)
    wd = wl.make_weights(cfg, wl.streams(cfg).weights, std=0.1)
    lw = wd["layers"][0]
    lw["wk"] = np.float32(-2.0 ** 103) * lw["wq"]   # a row's own score: -1e31 |q|^2 / sqrt(hd), with |q| > 1
    model = vf.vf_model_create(vf.config_from(cfg, 16, 64), vf.upload_weights(wd, cfg.dtype, DEV), DEV)
    ids = wl.make_context(cfg.vocab, 1, np.random.default_rng(hd))
    out = torch.empty((1, cfg.vocab), dtype=torch.float32, device=DEV)
    vf.vf_prefill_chunk(model, vf.vf_seq_create(model, 64), i32(ids), logits_mode=2, logits_out=out)
    spec = spec_of(cfg)
    z = forward(spec, weights_of(wd), oracle.KVCache(spec, 1), ids)
    assert rel_inf(out.cpu().numpy(), z).max() < 1e-5
