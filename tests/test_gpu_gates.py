"""SwiGLU with gates far from zero, in the gate/up GEMM's epilogue of every many-row pass: e^-g overflows float32
below a gate of -88.7, and silu(g) * u is then -0 * u.  One layer whose gate rows are scaled so that the gates run
from -1e4 to 1e4 and lie densely around the overflow, as a prefill chunk and as a verify of more rows than the
few-row kernels take, against the oracle, the general kernels and the few-row kernels.  The bound is the stated
2e-2 of the largest logit; a gate that comes out as NaN makes its whole row NaN."""
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
ROWS_MAX = 1030
_cache = {}


def _model():
    if not _cache:
        cfg = wl.scaled(wl.CONFIGS["1.5b_k16"], n_layers=1, d_model=512, n_q_heads=4, n_kv_heads=2, head_dim=128,
                        d_ffn=8960, vocab=4096)
        wd = wl.make_weights(cfg, wl.streams(cfg).weights)
        gate = wd["layers"][0]["w_gate"]   # a row's gates have a spread of 0.45; scaled: 0.45 to 3200
        gate *= np.logspace(0, np.log10(7000), cfg.d_ffn, dtype=np.float32)[:, None]
        wd["layers"][0]["w_gate"] = wl.generate.to_bf16_values(gate)
        model = vf.vf_model_create(vf.config_from(cfg, ROWS_MAX, 1100), vf.upload_weights(wd, cfg.dtype, DEV), DEV)
        _cache["m"] = cfg, spec_of(cfg), weights_of(wd, np.float32), model
    return _cache["m"]


def _oracle(spec, w, ids):
    with np.errstate(over="ignore"):
        return forward(spec, w, oracle.KVCache(spec, len(ids), np.float32), ids, np.float32)


def test_gates_cover_the_overflow():
    cfg, spec, w, _ = _model()
    x = w.embed[wl.make_context(cfg.vocab, 49, np.random.default_rng(0))]
    x = x / np.sqrt((x * x).mean(-1, keepdims=True))
    g = x @ w.layers[0].w_gate.T
    assert g.min() < -9e3 and g.max() > 9e3
    assert ((g > -92) & (g < -86)).sum() > 100 and ((g > -104) & (g < -88.8)).sum() > 100


# the row counts take weight-stream and square tiles, of one and of several row tiles
@pytest.mark.parametrize("rows", [1, 40, 130, 300, 600, ROWS_MAX])
def test_chunk(rows):
    cfg, spec, w, model = _model()
    ids = wl.make_context(cfg.vocab, rows, np.random.default_rng(rows))
    seq = vf.vf_seq_create(model, 1100)
    out = torch.empty((rows, cfg.vocab), dtype=torch.float32, device=DEV)
    got = []
    for fast in (1, 0):
        vf.vf_set_option(model, vf.VF_OPT_FAST_PATH, fast)
        vf.vf_seq_set_len(seq, 0)
        vf.vf_prefill_chunk(model, seq, i32(ids), logits_mode=2, logits_out=out)
        got.append(out.cpu().numpy())
    vf.vf_set_option(model, vf.VF_OPT_FAST_PATH, 1)
    assert np.isfinite(got[0]).all() and np.isfinite(got[1]).all()
    errs = rel_inf(got[0], _oracle(spec, w, ids)).max(), rel_inf(got[0], got[1]).max()
    print(f"{rows} rows: oracle {errs[0]:.2e}, general kernels {errs[1]:.2e}", flush=True)
    assert max(errs) < 2e-2


def test_verify_of_49_rows():
    cfg, spec, w, model = _model()
    ids = wl.make_context(cfg.vocab, 49, np.random.default_rng(49))
    seqs = [vf.vf_seq_create(model, 128) for _ in range(2)]
    logits = torch.empty((49, cfg.vocab), dtype=torch.float32, device=DEV)
    vf.vf_verify(model, seqs, i32(ids), [0, 33, 49], logits)
    got = logits.cpu().numpy()
    assert np.isfinite(got).all()
    few = torch.empty((33, cfg.vocab), dtype=torch.float32, device=DEV)   # the first sequence alone: few-row kernels
    vf.vf_verify(model, seqs[:1], i32(ids[:33]), [0, 33], few)
    assert rel_inf(got[:33], few.cpu().numpy()).max() < 2e-2
    assert rel_inf(got[:33], _oracle(spec, w, ids[:33])).max() < 2e-2
    assert rel_inf(got[33:], _oracle(spec, w, ids[33:])).max() < 2e-2
