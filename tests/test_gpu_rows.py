"""The many-row GEMM kernels against the oracle: one layer, all logits of one chunk, at row counts that
take each shape of tile (square tiles and the weight-stream tiles of 64 to 384 rows), with ragged row
blocks, column tiles that do not divide the matrix and K splits of unequal length.  One layer of bfloat16
arithmetic differs from the oracle's by the rounding of its products' inputs: the stated 2e-2 of the
largest logit (measured 4e-3); a wrong tile is off by the size of the logits."""
import numpy as np
import pytest
import torch

import workloads as wl
import oracle
import paper_2510_15312_amd as vf
from oracle.transformer import forward
from util_gpu import DEV, Pair, i32
from util_oracle import rel_inf, weights_of

pytestmark = pytest.mark.gpu
_cache = {}


def _pair(name):
    if name not in _cache:
        _cache.clear()
        dims = {"wide": dict(d_model=512, n_q_heads=4, n_kv_heads=2, head_dim=128, d_ffn=8960, vocab=16400),
                "narrow": dict(d_model=288, n_q_heads=3, n_kv_heads=1, head_dim=64, d_ffn=4128, vocab=4112)}[name]
        cfg = wl.scaled(wl.CONFIGS["1.5b_k16"], n_layers=1, **dims)
        pair = Pair(cfg, max_rows=1500, max_positions=1600)
        wd = wl.make_weights(cfg, wl.streams(cfg).weights)
        _cache[name] = pair, weights_of(wd, np.float32)
    return _cache[name]


@pytest.mark.parametrize("name,rows", [("wide", r) for r in (1, 17, 49, 128, 144, 272, 384, 512, 777, 1030, 1500)] +
                         [("narrow", r) for r in (33, 65, 448, 1499)])
def test_chunk_logits_against_oracle(name, rows):
    pair, w32 = _pair(name)
    V = pair.cfg.vocab
    ids = wl.make_context(V, rows, np.random.default_rng(rows))
    seq = pair.new_seq(1600)
    out = torch.empty((rows, V), dtype=torch.float32, device=DEV)
    vf.vf_prefill_chunk(pair.model, seq, i32(ids), logits_mode=2, logits_out=out)
    z = forward(pair.spec, w32, oracle.KVCache(pair.spec, rows, np.float32), ids, np.float32)
    err = rel_inf(out.cpu().numpy(), z).max()
    print(f"{name}, {rows} rows: {err:.2e}", flush=True)
    assert err < 2e-2
    # the same rows' top candidates out of the output head's epilogue
    k = 5
    tv = torch.empty((rows, k), dtype=torch.float32, device=DEV)
    ti = torch.empty((rows, k), dtype=torch.int32, device=DEV)
    vf.vf_seq_set_len(seq, 0)
    vf.vf_prefill_chunk_topk(pair.model, seq, i32(ids), k, tv, ti)
    want, at = torch.sort(out, dim=-1, descending=True, stable=True)   # equal logits by rising id
    assert torch.equal(ti.long(), at[:, :k]) and torch.equal(tv, want[:, :k])
