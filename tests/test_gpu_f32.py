"""The float32 decoder stack against the float64 oracle at the sizes where its kernels change shape:
row counts around a tile (16, 32, 64 rows), widths whose K chunks do not fill the eight wavefronts of a
workgroup, both head dimensions, grouped heads and bias, the wide tile, and keys shared out over
several workgroups.  The bound is 1e-5: K of at most 512 float32 products a sum, 24 bits each."""
import numpy as np
import pytest
import torch

import oracle
from oracle.transformer import forward
import workloads as wl
import paper_2510_15312_amd as vf
from util_gpu import DEV, Pair, i32
from util_oracle import rel_inf

pytestmark = pytest.mark.gpu
BASE = wl.CONFIGS["tiny_f32"]


# (d, q heads, kv heads, head_dim, ffn, vocab, prompt, chunk, rows of the verify, bias)
SHAPES = [
    (96, 2, 2, 64, 160, 272, 70, 33, 1, False),
    (256, 4, 4, 64, 512, 1024, 129, 64, 16, True),
    (160, 4, 2, 128, 224, 320, 65, 65, 17, True),
    (256, 4, 1, 64, 288, 8208, 160, 160, 33, False),   # 160 rows of 513 column blocks: the 64 x 32 tile
    (64, 2, 1, 64, 64, 64, 2240, 560, 9, False),       # 70 key tiles: two key parts
]


@pytest.mark.parametrize("d,hq,hkv,hd,ffn,vocab,n,chunk,rows,bias", SHAPES)
def test_f32_prefill_and_verify_against_oracle(d, hq, hkv, hd, ffn, vocab, n, chunk, rows, bias):
    cfg = wl.scaled(BASE, d_model=d, n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, d_ffn=ffn, vocab=vocab)
    pair = Pair(cfg, max_rows=max(chunk, rows), max_positions=n + 64, qkv_bias=bias, std=0.05)
    seq, cache = pair.new_seq(n + 64), oracle.KVCache(pair.spec, n + 64)
    ids = wl.make_context(vocab, n, pair.s.context)
    toks = i32(ids)
    for a in range(0, n, chunk):
        b = min(a + chunk, n)
        out = torch.empty((b - a, vocab), dtype=torch.float32, device=DEV)
        vf.vf_prefill_chunk(pair.model, seq, toks[a:b], logits_mode=2, logits_out=out)
        z = forward(pair.spec, pair.ow, cache, ids[a:b])
        assert rel_inf(out.cpu().numpy(), z).max() < 1e-5
    for layer in range(cfg.n_layers):
        (k, v), (ko, vo) = pair.kv_both(seq, cache, layer, 0, n)
        for got, want in ((k, ko), (v, vo)):
            assert np.abs(got - want).max() < 1e-5 * np.abs(want).max()
    drafts = wl.make_context(vocab, rows, pair.s.drafts)
    logits = torch.empty((rows, vocab), dtype=torch.float32, device=DEV)
    vf.vf_verify(pair.model, [seq], i32(drafts), [0, rows], logits)
    z = oracle.verify(pair.spec, pair.ow, cache, int(drafts[0]), drafts[1:])
    assert rel_inf(logits.cpu().numpy(), z).max() < 1e-5


# Precision: the 2-norm of the logits' error against float64, at a row count of every tile.  A plain kernel whose
# lanes each sum K / 64 products has 4.37e-7 and 7.58e-7 here, sums of K / 8 products 5.62e-7 and 9.79e-7; the bounds lie
# 5 % above the first (the same seeds: what varies is the order within a chain).
@pytest.mark.parametrize("d,ffn,vocab,bound", [(256, 1024, 4096, 4.6e-7), (512, 2048, 8192, 8.0e-7)])
def test_f32_error_of_the_sums(d, ffn, vocab, bound):
    cfg = wl.scaled(BASE, d_model=d, d_ffn=ffn, vocab=vocab)
    pair = Pair(cfg, max_rows=320, max_positions=320, std=0.05)
    ids = wl.make_context(vocab, 320, pair.s.context)
    z = forward(pair.spec, pair.ow, oracle.KVCache(pair.spec, 320), ids)
    for chunk in (16, 64, 320):
        seq, got = pair.new_seq(320), []
        for a in range(0, 320, chunk):
            out = torch.empty((chunk, vocab), dtype=torch.float32, device=DEV)
            vf.vf_prefill_chunk(pair.model, seq, i32(ids[a:a + chunk]), logits_mode=2, logits_out=out)
            got.append(out.cpu().numpy().astype(np.float64))
        err = np.linalg.norm(np.concatenate(got) - z) / np.linalg.norm(z)
        print(f"d {d}, chunks of {chunk}: {err:.3e}", flush=True)
        assert err < bound
