"""The many-row GEMM kernels against the oracle: one layer, all logits of one chunk, at sizes that take each kernel
with each of its epilogues that some call takes (test_plans.py has the list and checks that none is left out), with
ragged row blocks, column tiles that do not divide the matrix and K splits of unequal length; the deep model has a
bias of the size of the projections.  One layer of bfloat16 arithmetic differs from the oracle's by the rounding
of its products' inputs: the stated 2e-2 of the largest logit (measured 4e-3); a wrong tile is off by the size of
the logits."""
from types import SimpleNamespace

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


# name: dimensions, bias, rows of the chunks
MODELS = {
    "wide": (dict(d_model=512, n_q_heads=4, n_kv_heads=2, head_dim=128, d_ffn=8960, vocab=16400), False,
             (1, 17, 49, 128, 144, 272, 384, 512, 777, 1030, 1500)),
    "narrow": (dict(d_model=288, n_q_heads=3, n_kv_heads=1, head_dim=64, d_ffn=4128, vocab=4112), False, (33, 65, 448, 1499, 200)),
    "deep": (dict(d_model=3072, n_q_heads=48, n_kv_heads=16, head_dim=128, d_ffn=2048, vocab=40000), True,
             (33, 65, 129, 300, 511, 777, 1000, 1030, 1281, 100, 600)),
}
MAX_ROWS = 1500


def config_of(name):
    dims, bias, _ = MODELS[name]
    cfg = wl.scaled(wl.CONFIGS["1.5b_k16"], n_layers=1, **dims)
    return cfg, vf.config_from(cfg, MAX_ROWS, 1600, bias)


def candidates(rows):
    """Candidates of the top-k call: the most with which it takes the epilogue (28 to 40 rows a candidate, from 65 rows on)."""
    return max(1, min(vf.VF_TOPK_MAX, rows // 40))


def _pair(name):
    if name not in _cache:
        _cache.clear()
        (cfg, vcfg), bias = config_of(name), MODELS[name][1]
        wd = wl.make_weights(cfg, wl.streams(cfg).weights, qkv_bias=bias)
        for b in ("bq", "bk", "bv") if bias else ():
            wd["layers"][0][b] *= 50
        model = vf.vf_model_create(vcfg, vf.upload_weights(wd, cfg.dtype, DEV), DEV)
        _cache[name] = SimpleNamespace(cfg=cfg, spec=spec_of(cfg, bias), model=model), weights_of(wd, np.float32)
    return _cache[name]


@pytest.mark.parametrize("name,rows", [(n, r) for n, m in MODELS.items() for r in m[2]])
def test_chunk_logits_against_oracle(name, rows):
    pair, w32 = _pair(name)
    V = pair.cfg.vocab
    ids = wl.make_context(V, rows, np.random.default_rng(rows))
    seq = vf.vf_seq_create(pair.model, 1600)
    out = torch.empty((rows, V), dtype=torch.float32, device=DEV)
    vf.vf_prefill_chunk(pair.model, seq, i32(ids), logits_mode=2, logits_out=out)
    z = forward(pair.spec, w32, oracle.KVCache(pair.spec, rows, np.float32), ids, np.float32)
    err = rel_inf(out.cpu().numpy(), z).max()
    print(f"{name}, {rows} rows: {err:.2e}", flush=True)
    assert err < 2e-2
    # the same rows' top candidates out of the output head's epilogue
    k = candidates(rows)
    tv = torch.empty((rows, k), dtype=torch.float32, device=DEV)
    ti = torch.empty((rows, k), dtype=torch.int32, device=DEV)
    vf.vf_seq_set_len(seq, 0)
    vf.vf_prefill_chunk_topk(pair.model, seq, i32(ids), k, tv, ti)
    want, at = torch.sort(out, dim=-1, descending=True, stable=True)   # equal logits by rising id
    assert torch.equal(ti.long(), at[:, :k]) and torch.equal(tv, want[:, :k])
