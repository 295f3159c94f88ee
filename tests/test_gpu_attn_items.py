"""The attention kernel for many items over long contexts against the scalar one, through a model of one
layer: random keys and values are written to it, a chunk or a batch of paged sequences runs over them, and the
logits are compared with the general kernels' (VF_OPT_FAST_PATH 0: scalar attention, plain GEMMs).  Sizes sit
where the kernel's shapes turn: contexts at, below and above a page of 64 and a part of pages, items that do
not fill a wavefront or a workgroup, one part and several, both head sizes, pages in random order; each case
asserts that the cost model gives it to this kernel (test_plans.py, that some have one part and some several).  The two
paths round the same values to bfloat16, so they differ by the order of float32 sums and the roundings that
tips over: under 1e-2 of the largest logit (the tolerance of either against the oracle is 2e-2); a key left
out, or one too many, moves a row whose weight is spread over few keys by far more, and the softmax here is
peaked (keys with a spread of 3)."""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

import workloads as wl
import paper_2510_15312_amd as vf
from util_gpu import DEV, Pair, i32
from util_plan import attention_plan
from util_oracle import rel_inf

pytestmark = pytest.mark.gpu
_cache = {}


CHUNKS = [(1, 1056), (63, 1000), (64, 1055), (1900, 777), (4095, 512), (7900, 1051)]   # (context, rows)
BATCHES = [(32, 30, 8200), (16, 1000, 3000), (9, 3968, 4224), (16, 400, 700)]          # (sequences, contexts from .. to)


def config_of(hd):
    # heads enough that the model gives short contexts to this kernel for either head size
    heads = dict(n_q_heads=24, n_kv_heads=8) if hd == 128 else dict(n_q_heads=48, n_kv_heads=16)
    return wl.scaled(wl.CONFIGS["1.5b_k16"], n_layers=1, d_model=512, head_dim=hd, d_ffn=1024, vocab=2048, **heads)


def batch_of(n_seqs, lo, hi):
    rng = np.random.default_rng(n_seqs + lo)
    return rng.integers(lo, hi, n_seqs), rng.integers(6, 34, n_seqs), rng


def _pair(hd):
    if hd not in _cache:
        _cache.clear()
        _cache[hd] = Pair(config_of(hd), max_rows=1056, max_positions=9000)
    return _cache[hd]


def _fill(pair, seq, n, gen):
    kv = torch.empty((2, n, pair.cfg.n_kv_heads, pair.cfg.head_dim), dtype=torch.float32, device=DEV)
    kv.normal_(0.0, 3.0, generator=gen)
    vf.vf_kv_write(pair.model, seq, 0, 0, kv[0], kv[1])
    vf.vf_seq_set_len(seq, n)


def _both(pair, run):
    out = []
    for fast in (1, 0):
        vf.vf_set_option(pair.model, vf.VF_OPT_FAST_PATH, fast)
        out.append(run().cpu().numpy())
    vf.vf_set_option(pair.model, vf.VF_OPT_FAST_PATH, 1)
    return rel_inf(out[0], out[1]).max()


# 1056 rows of one page and less, contexts around a page, several parts
@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("ctx,rows", CHUNKS)
def test_chunk(hd, ctx, rows):
    pair = _pair(hd)
    assert attention_plan(pair.vcfg, [ctx], [rows])[0]
    gen = torch.Generator(device=DEV).manual_seed(ctx + rows)
    seq = pair.new_seq(9000)
    _fill(pair, seq, ctx, gen)
    ids = i32(wl.make_context(pair.cfg.vocab, rows, np.random.default_rng(rows)))
    logits = torch.empty((rows, pair.cfg.vocab), dtype=torch.float32, device=DEV)

    def run():
        vf.vf_seq_set_len(seq, ctx)
        vf.vf_prefill_chunk(pair.model, seq, ids, logits_mode=2, logits_out=logits)
        return logits
    err = _both(pair, run)
    print(f"hd {hd}, {ctx} + {rows}: {err:.2e}", flush=True)
    assert err < 1e-2


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("n_seqs,lo,hi", BATCHES)
def test_paged_batch(hd, n_seqs, lo, hi):
    pair = _pair(hd)
    ctx, rows, rng = batch_of(n_seqs, lo, hi)
    assert attention_plan(pair.vcfg, ctx, rows)[0]
    need = [int(-(-(c + r) // 64)) for c, r in zip(ctx, rows)]
    perm = rng.permutation(sum(need))
    pool = torch.full((vf.vf_kv_bytes(pair.model, 64, sum(need)),), 255, dtype=torch.uint8, device=DEV)   # NaN where nothing is written
    gen = torch.Generator(device=DEV).manual_seed(n_seqs)
    seqs, at = [], 0
    for c, n in zip(ctx, need):
        seqs.append(pair.new_seq(n * 64, pool=pool, block_table=i32(perm[at:at + n])))
        at += n
        _fill(pair, seqs[-1], int(c), gen)
    off = [0] + [int(x) for x in np.cumsum(rows)]
    ids = i32(rng.integers(0, pair.cfg.vocab, off[-1]))
    logits = torch.empty((off[-1], pair.cfg.vocab), dtype=torch.float32, device=DEV)

    def run():
        for s, c in zip(seqs, ctx):
            vf.vf_seq_set_len(s, int(c))
        vf.vf_verify(pair.model, seqs, ids, off, logits)
        return logits
    err = _both(pair, run)
    print(f"hd {hd}, {n_seqs} sequences: {err:.2e}", flush=True)
    assert err < 1e-2


# more parts than the merge requests together (eight), and rows that do not see the last one, whose records for them hold anything
@pytest.mark.parametrize("hd,ctx", [(64, 5720), (128, 5740)])
def test_merge_of_many_parts(hd, ctx):
    pair, rows = _pair(hd), 64
    pages, _ = attention_plan(pair.vcfg, [ctx], [rows])
    parts = -(-(-(-(ctx + rows) // 64)) // pages)
    assert parts > 8 and ctx < (parts - 1) * pages * 64 < ctx + rows
    seq = pair.new_seq(9000)
    _fill(pair, seq, ctx, torch.Generator(device=DEV).manual_seed(ctx))
    ids = i32(wl.make_context(pair.cfg.vocab, rows, np.random.default_rng(ctx)))
    logits = torch.empty((rows, pair.cfg.vocab), dtype=torch.float32, device=DEV)

    def run():
        vf.vf_seq_set_len(seq, ctx)
        vf.vf_prefill_chunk(pair.model, seq, ids, logits_mode=2, logits_out=logits)
        return logits
    err = _both(pair, run)
    print(f"hd {hd}, {parts} parts: {err:.2e}", flush=True)
    assert err < 1e-2


# The same with records that would show: a call before it, whose rows all see the last part, leaves there the records of
# keys and values far above all others, which outweigh a row's own by any number of orders if they are added to it.
@pytest.mark.parametrize("hd,ctx", [(64, 5720), (128, 5720)])
def test_merge_drops_the_parts_a_row_does_not_see(hd, ctx):
    pair, rows = _pair(hd), 64
    pages, merged = attention_plan(pair.vcfg, [ctx], [rows])
    parts = -(-(-(-(ctx + rows) // 64)) // pages)
    last = (parts - 1) * pages * 64
    # the first 64 items, 21 rows of three heads, see nothing of the last part
    assert merged and ctx + 22 < last < ctx + rows
    assert attention_plan(pair.vcfg, [last + 32], [rows]) == (pages, True) and -(-(-(-(last + 32 + rows) // 64)) // pages) == parts
    seq, gen = pair.new_seq(9000), torch.Generator(device=DEV).manual_seed(ctx)
    _fill(pair, seq, last, gen)
    far = torch.empty((2, 32, pair.cfg.n_kv_heads, hd), dtype=torch.float32, device=DEV).normal_(0.0, 100.0, generator=gen)
    far[1] = 1e4
    vf.vf_kv_write(pair.model, seq, 0, last, far[0], far[1])
    ids = i32(wl.make_context(pair.cfg.vocab, rows, np.random.default_rng(ctx)))
    logits = torch.empty((rows, pair.cfg.vocab), dtype=torch.float32, device=DEV)

    def run_at(n):
        vf.vf_seq_set_len(seq, n)
        vf.vf_prefill_chunk(pair.model, seq, ids, logits_mode=2, logits_out=logits)
        return logits
    before = run_at(last + 32).cpu().numpy()
    err = _both(pair, lambda: run_at(ctx))   # the kernel for many items first
    own = logits.cpu().numpy()
    print(f"hd {hd}, {parts} parts: {err:.2e}", flush=True)
    assert np.isfinite(own).all() and rel_inf(before, own).min() > 0.1   # every row of the call before saw the far values
    assert err < 1e-2


# A value that is not finite may reach the rows of its own 32 keys and of the items (16 to a wavefront, 3 to a
# row here) that share them, as in the kernel for few items, and no row further up.
@pytest.mark.parametrize("at", [44, 70, 703])   # second half of the chunk's first page, first half, a later page
def test_value_that_is_not_finite(at):
    pair = _pair(128)
    rows, ctx, V, d = 777, 1920, pair.cfg.vocab, pair.cfg.d_model
    seq = pair.new_seq(9000)
    ids = wl.make_context(V, rows, np.random.default_rng(at))
    ids[at] = np.setdiff1d(np.arange(V), ids)[0]   # a token of its own
    assert attention_plan(pair.vcfg, [ctx], [rows])[0]
    _fill(pair, seq, ctx, torch.Generator(device=DEV).manual_seed(at))
    logits = torch.empty((rows, V), dtype=torch.float32, device=DEV)

    def run(value):
        w = {**pair.dw, "lm_head": pair.dw["embed"], "embed": pair.dw["embed"].clone()}
        w["embed"][int(ids[at])] = value
        cfg = vf.make_config(1, d, pair.cfg.n_q_heads, pair.cfg.n_kv_heads, 128, pair.cfg.d_ffn, V, "bf16", pair.cfg.rope_theta,
                             pair.cfg.rms_eps, rows, 9000, tie_embeddings=False)
        model = vf.vf_model_create(cfg, w, DEV)
        own = vf.vf_seq_create(model, 9000)
        own.kv.copy_(seq.kv)
        vf.vf_seq_set_len(own, ctx)
        vf.vf_prefill_chunk(model, own, i32(ids), logits_mode=2, logits_out=logits)
        return logits.cpu().numpy()
    want, got = run(0.02), run(float("inf"))
    clear = [r for r in range(at) if r + 6 < at - at % 32]
    assert len(clear) > 20 and np.isnan(got[at:]).any(axis=1).all()
    assert np.array_equal(got[clear], want[clear])


# One key that all rows see scores some 270 above every other (natural logarithm): its weight is 1, and a running maximum
# that is not the largest of all keys of a page lets its exponential overflow.  Every lane of an item holds eight keys of 32.
# The queries are a bias that the rotary embedding hardly turns (theta so large that only the first quarter of the
# frequencies counts, where the bias is zero).
@pytest.mark.parametrize("hd", [64, 128])
def test_one_key_far_above_the_others(hd):
    pair = _pair(hd)
    ctx, rows, half = 1900, 777, hd // 2
    assert attention_plan(pair.vcfg, [ctx], [rows])[0]
    turned = torch.arange(hd, device=DEV) % half < half // 4
    direction = torch.where(turned, 0.0, 1.0).to(DEV)
    nq, nkv = pair.cfg.n_q_heads, pair.cfg.n_kv_heads
    layer = {**pair.dw["layers"][0], "bq": 2.0 * direction.repeat(nq), "bk": torch.zeros(nkv * hd, device=DEV),
             "bv": torch.zeros(nkv * hd, device=DEV)}
    cfg = vf.make_config(1, pair.cfg.d_model, nq, nkv, hd, pair.cfg.d_ffn, pair.cfg.vocab, "bf16", 1e38, pair.cfg.rms_eps, rows, 9000,
                         qkv_bias=True)
    own = SimpleNamespace(cfg=pair.cfg, model=vf.vf_model_create(cfg, {**pair.dw, "layers": [layer]}, DEV))
    seq = vf.vf_seq_create(own.model, 9000, device=DEV)
    ids = i32(wl.make_context(pair.cfg.vocab, rows, np.random.default_rng(hd)))
    logits = torch.empty((rows, pair.cfg.vocab), dtype=torch.float32, device=DEV)
    scale = 270.0 / (2.0 * float(direction.sum()) / hd ** 0.5)

    def run():
        vf.vf_seq_set_len(seq, ctx)
        vf.vf_prefill_chunk(own.model, seq, ids, logits_mode=2, logits_out=logits)
        return logits
    for key in (192 + 3, 192 + 9, 192 + 20, 192 + 31, 192 + 36, 192 + 46, 192 + 55, 192 + 56, ctx - 1):
        gen = torch.Generator(device=DEV).manual_seed(key)
        kv = torch.empty((2, ctx, nkv, hd), dtype=torch.float32, device=DEV).normal_(0.0, 1.0, generator=gen)
        kv[0, key] = scale * direction
        vf.vf_kv_write(own.model, seq, 0, 0, kv[0], kv[1])
        err = _both(own, run)
        print(f"hd {hd}, key {key}: {err:.2e}", flush=True)
        assert err < 1e-2
