"""The persistent kernels at the edges of their tiles: rows that fill or just exceed a block, a staging round or a row group,
rows of the residual stream that take several passes or end within one, K splits of unequal length, one key part or
several.  Logits of every row against the oracle: two layers of bfloat16 arithmetic differ by the rounding of the
products' inputs, the stated 2e-2 of the largest logit; a wrong tile is off by the size of the logits.  Which kernel runs is
asserted from the launches that the library times: the whole pass, or the layers and then the head, or neither.  A call
is repeated behind one of another size, bit for bit: nothing of a launch is left for the next."""
import numpy as np
import pytest
import torch

import workloads as wl
import oracle
import paper_2510_15312_amd as vf
from oracle.transformer import forward
from util_gpu import DEV, i32
from util_oracle import rel_inf, spec_of, weights_of
from util_plan import persistent_plan

pytestmark = pytest.mark.gpu
_cache = {}

# name: dimensions, context (keys before the rows of the call)
MODELS = {
    "narrow": (dict(d_model=320, n_q_heads=5, n_kv_heads=1, head_dim=64, d_ffn=992, vocab=1040), 600),
    "two_passes_64": (dict(d_model=1600, n_q_heads=10, n_kv_heads=2, head_dim=64, d_ffn=2080, vocab=1040), 70),
    "two_passes_128": (dict(d_model=2048, n_q_heads=12, n_kv_heads=4, head_dim=128, d_ffn=4128, vocab=2064), 300),
    # with bias, rows of the residual stream of two passes
    "biased": (dict(d_model=2048, n_q_heads=4, n_kv_heads=2, head_dim=128, d_ffn=992, vocab=1040, qkv_bias=True), 70),
    # rows of the residual stream of more than two passes of the norm: up to 8 of them fit LDS
    "widest": (dict(d_model=8256, n_q_heads=6, n_kv_heads=2, head_dim=64, d_ffn=992, vocab=1040), 70),
}
VERIFY = (1, 7, 8, 9, 16, 17, 24, 25, 32, 33)   # two_passes_128: 32 rows are the most that LDS takes
BATCH = (34, 47, 48, 49, 63, 64, 65, 66)        # two sequences; from 65 rows on a launch per operation


def _model(name):
    if name not in _cache:
        _cache.clear()
        dims, ctx = MODELS[name]
        dims = dict(dims)
        bias = dims.pop("qkv_bias", False)
        cfg = wl.scaled(wl.CONFIGS["1.5b_k16"], n_layers=2, **dims)
        wd = wl.make_weights(cfg, wl.streams(cfg).weights, qkv_bias=bias)
        for lw in wd["layers"] if bias else []:   # as large as what it is added to
            for b in ("bq", "bk", "bv"):
                lw[b] *= np.float32(cfg.d_model ** 0.5)
        model = vf.vf_model_create(vf.config_from(cfg, 128, 1024, qkv_bias=bias), vf.upload_weights(wd, cfg.dtype, DEV), DEV)
        spec, w32 = spec_of(cfg, bias), weights_of(wd, np.float32)
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


def _kernel_that_runs(model, call):
    """None, "pass" or "layers": from the launches the library times in one call."""
    vf.vf_profile_read(model)
    vf.vf_profile(model, 1)
    try:
        call()
    finally:
        vf.vf_profile(model, 0)
    n = {site: count for site, (_, count) in vf.vf_profile_read(model).items()}
    assert n["step"] in (0, 1) and (n["step"] == 0) == (n["gateup"] > 0)
    return None if n["step"] == 0 else "layers" if n["head"] else "pass"


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
    assert torch.equal(out, again)
    ran = _kernel_that_runs(model, lambda: vf.vf_verify(model, [seq], i32(ids), [0, rows], again))
    assert ran == persistent_plan(model.cfg, rows)[0] and ran is not None


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
    again, small = torch.empty_like(out), torch.empty((5, cfg.vocab), dtype=torch.float32, device=DEV)
    ids = i32(np.concatenate([ids_a, ids_b]))
    try:
        vf.vf_verify(model, seqs, ids, [0, first, rows], out)
        vf.vf_verify(model, seqs[:1], ids[:5], [0, 5], small)
        ran = _kernel_that_runs(model, lambda: vf.vf_verify(model, seqs, ids, [0, first, rows], again))
    finally:
        vf.vf_set_option(model, vf.VF_OPT_PERSISTENT, 1)
    assert ran == (persistent_plan(model.cfg, rows)[0] if persistent else None)
    err = rel_inf(out.cpu().numpy(), np.concatenate([z_a, z_b])).max()
    print(f"{name}, {rows} rows: {err:.2e}", flush=True)
    assert err < 2e-2
    assert torch.equal(out, again)


def _random_tree(rng, n):
    return [-1] + [int(rng.integers(max(0, r - 4), r)) for r in range(1, n)]


# whole pass, layers alone, launches; over tiles with and without keys of the call
@pytest.mark.parametrize("name,rows", [("narrow", 44), ("two_passes_128", 41), ("two_passes_128", 56), ("widest", 20)])
def test_tree_batch_against_oracle(name, rows):
    cfg, model, spec, w32, seqs, cache, ctx = _model(name)
    rng = np.random.default_rng(rows)
    first = rows // 2
    sizes = [first, rows - first]
    ids = [wl.make_context(cfg.vocab, n, rng) for n in sizes]
    parents = [_random_tree(rng, n) for n in sizes]
    want = []
    for t, p in zip(ids, parents):
        cache.len = ctx
        want.append(forward(spec, w32, cache, t, np.float32, parents=p))
        cache.len = ctx
    out = torch.empty((rows, cfg.vocab), dtype=torch.float32, device=DEV)
    for seq in seqs:
        vf.vf_seq_set_len(seq, ctx)
    ran = _kernel_that_runs(model, lambda: vf.vf_verify_tree(model, seqs, i32(np.concatenate(ids)), [0, first, rows], sum(parents, []), out))
    assert ran == persistent_plan(model.cfg, rows)[0]
    err = rel_inf(out.cpu().numpy(), np.concatenate(want)).max()
    print(f"{name}, tree batch of {rows} rows: {err:.2e}", flush=True)
    assert err < 2e-2


def _two(model, seqs, ctx, ids, rows, vocab):
    out = torch.empty((rows, vocab), dtype=torch.float32, device=DEV)
    for seq in seqs:
        vf.vf_seq_set_len(seq, ctx)
    vf.vf_verify(model, seqs, ids, [0, rows // 2, rows], out)
    return out.cpu().numpy()


# What one workgroup sends another goes through memory that is marked where nothing has been sent.
@pytest.mark.parametrize("name,rows", [("narrow", 34), ("two_passes_64", 34), ("two_passes_128", 34)])
def test_value_that_is_not_finite_stays_with_its_sequence(name, rows):
    cfg, base, _, _, seqs, _, ctx = _model(name)
    dw = vf.upload_weights(wl.make_weights(cfg, wl.streams(cfg).weights), cfg.dtype, DEV)
    dw = {**dw, "lm_head": dw["embed"], "embed": dw["embed"].clone()}
    ids = wl.make_context(cfg.vocab, rows, np.random.default_rng(rows))
    ids[-1] = np.setdiff1d(np.arange(cfg.vocab), ids)[0]   # the last row of the second sequence: a token of its own
    vcfg = vf.make_config(cfg.n_layers, cfg.d_model, cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, cfg.d_ffn, cfg.vocab, cfg.dtype,
                          cfg.rope_theta, cfg.rms_eps, 128, 1024, tie_embeddings=False)

    def run(value):
        dw["embed"][int(ids[-1])] = value
        model = vf.vf_model_create(vcfg, dw, DEV)
        own = [vf.vf_seq_create(model, 1024) for _ in seqs]
        for a, b in zip(own, seqs):
            a.kv.copy_(b.kv)
        clean = ids.copy()
        clean[-1] = clean[0]
        out = _two(model, own, ctx, i32(ids), rows, cfg.vocab)
        return out, _two(model, own, ctx, i32(clean), rows, cfg.vocab)
    want, clean = run(0.02)
    for value in (float("inf"), float("nan")):
        got, behind = run(value)
        assert np.isnan(got[-1]).any()
        assert np.array_equal(got[:rows // 2], want[:rows // 2])
        assert np.array_equal(behind, clean)   # the next call finds the marks in place


# The counters, their start value and the marks, all of them wrong, and the flag of a barrier that gave up: as after a launch
# that did.  The next query of a state reports it and puts everything back.
@pytest.mark.parametrize("name,rows", [("narrow", 34), ("two_passes_128", 20), ("two_passes_128", 34)])
def test_calls_behind_a_wait_that_gave_up(name, rows):
    cfg, model, _, _, seqs, _, ctx = _model(name)
    ids = i32(wl.make_context(cfg.vocab, rows, np.random.default_rng(rows)))
    want = _two(model, seqs, ctx, ids, rows, cfg.vocab)
    n = vf.vf_model_packed_bytes(model.cfg)
    exchange = 256 * max(12, cfg.head_dim // 8) * 1024   # bytes, and 64 KB of counters: the end of the packed buffer
    torch.cuda.synchronize()
    assert bool((model.buf[n - 65536 - exchange:n - 65536] == 255).all())   # marks everywhere between calls
    model.buf[n - 65536 - exchange:n].fill_(1)
    torch.cuda.synchronize()
    with pytest.raises(vf.VfError):
        vf.vf_seq_get_state(seqs[0])
    vf.vf_seq_get_state(seqs[0])
    assert np.array_equal(_two(model, seqs, ctx, ids, rows, cfg.vocab), want)
    assert bool((model.buf[n - 65536 - exchange:n - 65536] == 255).all())
