"""The work whose time is measured: the calls a user of the draft-verify library makes, through the
package's public entry points, over the range of shapes and sizes the library is built for.

A decode or verify pass is what a generation loop does per step: roll the sequence to its length,
`vf_verify` (one forward pass over the pending token and its drafts), `vf_accept`.  A prefill pass
feeds a whole prompt in chunks and samples the first token.  Sizes follow the repository's own
workload configurations (0.5B, 1.5B and 3B shapes in bfloat16, a tiny shape in float32; prefill
chunks of 128 and 256; up to 32 drafts; a batch of 16 paged sequences) and the limits in
include/vf.h.

Weights are random, but shaped so that a pass decides something: the output projections of a layer
are scaled down with depth and the (tied) embedding is large enough that a row's most likely
successor is its own token with high probability, as confident as a trained model is.  Drafts are a
run of that token followed by other ids, so the accepted count takes every value, and the ids that
two correct implementations emit are the same ones.
"""
import math
import random

import torch

import paper_2510_15312_amd as vf

DEV = "cuda:0"

# layers, d_model, q heads, kv heads, head_dim, d_ffn, vocabulary, dtype, rope theta
SHAPES = {
    "0.5b": (24, 896, 14, 2, 64, 4864, 151936, "bf16", 1e6),
    "1.5b": (28, 1536, 12, 2, 128, 8960, 151936, "bf16", 1e6),
    "3b": (28, 3072, 24, 8, 128, 8192, 128256, "bf16", 5e5),
    "tiny": (2, 256, 4, 4, 64, 1024, 4096, "f32", 1e4),
}
EMBED_STD, WEIGHT_STD, FINAL_GAIN = 0.15, 0.02, 0.25


def listed():
    return [
        # plain decoding of the smallest bf16 shape: the drafter found nothing, one row per step
        {"name": "decode_0.5b", "kind": "verify", "shape": "0.5b", "ctx": 1024, "k": 0, "stochastic": False},
        # the 0.5B shape's own recipe: 8 drafts, greedy
        {"name": "verify_0.5b_k8", "kind": "verify", "shape": "0.5b", "ctx": 1024, "k": 8, "stochastic": False},
        # the headline recipe: 16 drafts with a dense draft distribution, stochastic acceptance
        {"name": "verify_1.5b_k16", "kind": "verify", "shape": "1.5b", "ctx": 2048, "k": 16, "stochastic": True},
        # drafts as a token tree, at an odd context length
        {"name": "tree_1.5b_23", "kind": "tree", "shape": "1.5b", "ctx": 1111, "k": 22, "stochastic": False},
        # the largest few-row call: widest shape, longest draft
        {"name": "verify_3b_k32", "kind": "verify", "shape": "3b", "ctx": 4096, "k": 32, "stochastic": False},
        # a handful of users: paged sequences with short drafts, both acceptance modes
        {"name": "batch_1.5b_5", "kind": "batch", "shape": "1.5b", "seqs": 5, "ctx": 1500, "k": 14, "layout": 3},
        # a busier server on the small shape: ragged, about a hundred rows
        {"name": "batch_0.5b_12", "kind": "batch", "shape": "0.5b", "seqs": 12, "ctx": 900, "k": 16, "layout": 5},
        # the batched RAG mix: 16 paged sequences, contexts of 512 to 8192, up to 32 drafts each
        {"name": "mix_1.5b_16", "kind": "batch", "shape": "1.5b", "seqs": 16, "ctx": 2048, "k": 32, "layout": 15312},
        # a RAG prompt through the default chunk
        {"name": "prefill_1.5b_2048", "kind": "prefill", "shape": "1.5b", "tokens": 2048, "chunk": 256},
        # a short prompt of odd length in small chunks: the last chunk has nine tokens
        {"name": "prefill_0.5b_777", "kind": "prefill", "shape": "0.5b", "tokens": 777, "chunk": 128},
        # a prompt on the widest shape in large chunks, the second one ragged
        {"name": "prefill_3b_1900", "kind": "prefill", "shape": "3b", "tokens": 1900, "chunk": 1024},
        # the float32 shape's whole request: prompt in chunks of 128, then one verify step
        {"name": "request_tiny_f32", "kind": "request", "shape": "tiny", "tokens": 512, "chunk": 128, "k": 4},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["verify", "verify", "tree", "batch", "batch", "prefill", "prefill", "request"])
    if kind == "verify":
        shape = rng.choice(["0.5b", "1.5b", "3b"])
        return {"kind": kind, "shape": shape, "ctx": _log_uniform(rng, 64, 4096 if shape == "3b" else 8192),
                "k": rng.randint(0, 32), "stochastic": rng.random() < 0.5}
    if kind == "tree":
        return {"kind": kind, "shape": rng.choice(["0.5b", "1.5b"]), "ctx": _log_uniform(rng, 64, 8192),
                "k": rng.randint(1, 32), "stochastic": rng.random() < 0.5}
    if kind == "batch":
        return {"kind": kind, "shape": rng.choice(["0.5b", "1.5b"]), "seqs": rng.randint(2, 16),
                "ctx": _log_uniform(rng, 256, 2048), "k": rng.randint(1, 32), "layout": rng.randint(1, 1 << 20)}
    if kind == "prefill":
        shape, chunk = rng.choice(["0.5b", "1.5b", "3b"]), rng.choice([64, 128, 200, 256, 512, 1024])
        most = {"0.5b": 2048, "1.5b": 2048, "3b": 1800}[shape] if chunk >= 512 else 3 * chunk
        return {"kind": kind, "shape": shape, "tokens": _log_uniform(rng, 16, most), "chunk": chunk}
    return {"kind": "request", "shape": "tiny", "tokens": _log_uniform(rng, 16, 1024),
            "chunk": rng.choice([64, 128, 256]), "k": rng.randint(0, 32)}


# ---- what a call is made of --------------------------------------------------------------------

def _sequences(case):
    """Per sequence (context length, drafts, stochastic): part of the case, not of the seed."""
    if case["kind"] == "batch":
        rng = random.Random(case["layout"])
        out = []
        for i in range(case["seqs"]):
            ctx = int(min(max(case["ctx"] * math.exp(rng.gauss(0.0, 0.6)), 512 if case["ctx"] >= 2048 else 64), 8192))
            out.append((ctx, rng.randint(1, case["k"]), i % 2 == 1))
        return out
    if case["kind"] == "request":
        return [(case["tokens"], case["k"], False)]
    return [(case["ctx"], case["k"], case["stochastic"])]


def _chunks(case):
    n, c = case["tokens"], case["chunk"]
    return [(a, min(a + c, n)) for a in range(0, n, c)]


def _model(shape, gen, max_rows, max_positions):
    L, d, hq, hkv, hd, F, V, dtype, theta = SHAPES[shape]
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32

    def mat(n, k, std):
        return torch.empty((n, k), dtype=dt, device=DEV).normal_(0.0, std, generator=gen)
    ones = torch.ones(d, dtype=torch.float32, device=DEV)
    out_std = WEIGHT_STD / math.sqrt(2 * L)
    w = {"embed": mat(V, d, EMBED_STD), "final_norm": torch.full_like(ones, FINAL_GAIN), "layers": []}
    for _ in range(L):
        w["layers"].append({
            "attn_norm": ones, "ffn_norm": ones,
            "wq": mat(hq * hd, d, WEIGHT_STD), "wk": mat(hkv * hd, d, WEIGHT_STD), "wv": mat(hkv * hd, d, WEIGHT_STD),
            "wo": mat(d, hq * hd, out_std), "w_gate": mat(F, d, WEIGHT_STD), "w_up": mat(F, d, WEIGHT_STD),
            "w_down": mat(d, F, out_std)})
    cfg = vf.make_config(L, d, hq, hkv, hd, F, V, dtype, theta, 1e-6, max_rows, max_positions)
    return vf.vf_model_create(cfg, w, DEV)


def _fill_cache(model, seq, n, gen):
    """A context of n tokens: keys and values with the spread the model's own projections have."""
    cfg = model.cfg
    std = WEIGHT_STD * math.sqrt(cfg.d_model)
    for layer in range(cfg.n_layers):
        kv = torch.empty((2, n, cfg.n_kv_heads, cfg.head_dim), dtype=torch.float32, device=DEV)
        kv.normal_(0.0, std, generator=gen)
        vf.vf_kv_write(model, seq, layer, 0, kv[0], kv[1])
    vf.vf_seq_set_len(seq, n)


def _kv_view(kv, model):
    return kv.view(torch.bfloat16 if model.cfg.dtype == vf.VF_BF16 else torch.float32)


def _drafts(rng, pending, k, V):
    """A run of the likely token, then other ids; the accepted count is the length of the run."""
    run = rng.randint(0, k)
    return [pending] * run + [rng.randrange(V) for _ in range(k - run)]


def _tree(rng, pending, k, V):
    """k nodes below the root, each under an earlier row; about half carry the likely token."""
    parents, tokens = [-1], [pending]
    for r in range(1, k + 1):
        parents.append(max(0, r - 1 - rng.randrange(min(r, 4))))
        tokens.append(tokens[parents[r]] if rng.random() < 0.5 else rng.randrange(V))
    return parents, tokens


def _uniforms(rows, gen):
    # away from 0 and 1: a decision there hangs on the last bit of a probability
    return torch.rand(2 * rows, device=DEV, generator=gen) * 0.9 + 0.05


def _draft_distribution(drafts, V, gen):
    """Dense rows: 60 % on the draft, the rest spread over the vocabulary."""
    q = torch.softmax(torch.randn((len(drafts), V), device=DEV, generator=gen), dim=-1).mul_(0.4)
    at = torch.tensor(drafts, device=DEV).unsqueeze(1)
    return q.scatter_add_(1, at, torch.full_like(at, 0.6, dtype=q.dtype))


class State:
    pass


def prepare(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(int(seed))
    rng = random.Random(int(seed))
    s = State()
    s.kind = case["kind"]
    V = SHAPES[case["shape"]][6]
    prompt = s.kind in ("prefill", "request")
    seqs = [] if s.kind == "prefill" else _sequences(case)
    rows = sum(k + 1 for _, k, _ in seqs)
    max_rows = max(rows, case["chunk"] if prompt else 0)
    longest = case["tokens"] + 64 if prompt else max(c for c, _, _ in seqs) + 64
    s.model = _model(case["shape"], gen, max_rows, longest)
    s.seqs, s.lens = [], []
    if s.kind == "batch":
        # pages of all sequences in one pool, in random order
        need = [-(-(c + k + 1) // 64) for c, k, _ in seqs]
        perm = list(range(sum(need)))
        rng.shuffle(perm)
        pool = torch.zeros(vf.vf_kv_bytes(s.model, 64, len(perm)), dtype=torch.uint8, device=DEV)
        for (ctx, _, _), n in zip(seqs, need):
            table = torch.tensor(perm[:n], dtype=torch.int32, device=DEV)
            del perm[:n]
            s.seqs.append(vf.vf_seq_create(s.model, n * 64, pool, table, DEV))
            s.lens.append(ctx)
    else:
        pool = None
        s.seqs.append(vf.vf_seq_create(s.model, longest, device=DEV))
        s.seqs[0].kv.zero_()
        s.lens.append(0 if prompt else seqs[0][0])
    for q, n in zip(s.seqs, s.lens):
        if n:
            _fill_cache(s.model, q, n, gen)
    s.kv = _kv_view(s.seqs[0].kv if pool is None else pool, s.model)
    s.committed = [q.state.view(torch.int32)[:2] for q in s.seqs]
    if prompt:
        ids = [rng.randrange(V) for _ in range(case["tokens"])]
        s.prompt = torch.tensor(ids, dtype=torch.int32, device=DEV)
        s.chunks = _chunks(case)
        s.last_row = torch.zeros(V, dtype=torch.float32, device=DEV)
    if seqs:
        s.row_off, toks, s.parents, s.params = [0], [], [], []
        for _, k, stochastic in seqs:
            # after a prompt the pending token is the one the prefill sampled: the prompt's last, most likely
            pending = ids[-1] if prompt else rng.randrange(V)
            if s.kind == "tree":
                s.parents, chain = _tree(rng, pending, k, V)
                drafts = chain[1:]
            else:
                drafts = _drafts(rng, pending, k, V)
            toks += [vf.VF_PENDING if prompt else pending] + drafts
            s.row_off.append(s.row_off[-1] + k + 1)
            if stochastic:
                # a single verify carries a dense draft distribution, trees and batches the retrieval
                # drafter's one-hot one
                dense = s.kind == "verify" and k > 0
                s.params.append((vf.VF_STOCHASTIC, 0.8, _draft_distribution(drafts, V, gen) if dense else None,
                                 _uniforms(k + 1, gen)))
            else:
                s.params.append((vf.VF_GREEDY, 0.0, None, None))
        s.tokens = torch.tensor(toks, dtype=torch.int32, device=DEV)
        s.logits = torch.zeros((rows, V), dtype=torch.float32, device=DEV)
        s.n_accept = torch.zeros(len(seqs), dtype=torch.int32, device=DEV)
        s.out = torch.zeros(rows, dtype=torch.int32, device=DEV)
        s.y = torch.zeros(rows, dtype=torch.int32, device=DEV)
        s.path = torch.zeros(rows, dtype=torch.int32, device=DEV)
    return s


def run(s):
    for q, n in zip(s.seqs, s.lens):
        vf.vf_seq_set_len(q, n)  # back to where the pass starts
    out = {"kv": s.kv, "committed": s.committed}
    if s.kind in ("prefill", "request"):
        for a, b in s.chunks:
            last = b == s.prompt.numel()
            vf.vf_prefill_chunk(s.model, s.seqs[0], s.prompt[a:b], logits_mode=1 if last else 0,
                                logits_out=s.last_row if last else None, sample_first=last)
        out["last_row"] = s.last_row
        if s.kind == "prefill":
            return out
    if s.kind == "tree":
        vf.vf_verify_tree(s.model, s.seqs, s.tokens, s.row_off, s.parents, s.logits)
        vf.vf_accept_tree(s.model, s.seqs, s.tokens, s.row_off, s.parents, s.params, s.n_accept, s.out, s.y, s.path)
        out["path"] = s.path
    else:
        vf.vf_verify(s.model, s.seqs, s.tokens, s.row_off, s.logits)
        vf.vf_accept(s.model, s.seqs, s.tokens, s.row_off, s.params, s.n_accept, s.out, s.y)
    out.update(logits=s.logits, n_accept=s.n_accept, out_tokens=s.out, y=s.y)
    return out


def work(case):
    L, d, hq, hkv, hd, F, V, dtype, _ = SHAPES[case["shape"]]
    es = 2 if dtype == "bf16" else 4
    layer = (hq + 2 * hkv) * hd * d + d * hq * hd + 3 * F * d   # weights of a layer
    kv_tok = 2 * L * hkv * hd * es                              # cache bytes of a token
    nbytes = flops = 0.0

    def attend(rows, ctx):   # rows at positions ctx .. ctx + rows - 1
        return 4.0 * L * hq * hd * (rows * ctx + rows * (rows + 1) / 2)
    if case["kind"] in ("prefill", "request"):
        for a, b in _chunks(case):  # every chunk is a call of its own and needs all layers' weights
            n = b - a
            nbytes += L * layer * es + (a + n) * kv_tok + n * d * es
            flops += 2.0 * n * L * layer + attend(n, a)
        nbytes += V * d * es + V * 4
        flops += 2.0 * V * d
    if case["kind"] != "prefill":
        seqs = _sequences(case)
        rows = sum(k + 1 for _, k, _ in seqs)
        nbytes += (L * layer + V * d) * es + rows * V * 4 + rows * d * es
        nbytes += sum((ctx + 2 * (k + 1)) * kv_tok for ctx, k, _ in seqs)
        if case["kind"] == "verify" and case["stochastic"] and case["k"]:
            nbytes += V * 4  # the draft distribution of the row that decides
        flops += 2.0 * rows * (L * layer + V * d) + sum(attend(k + 1, ctx) for ctx, k, _ in seqs)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """What another correct implementation may differ by.  Measured between the library's own three
    implementations of a pass (other order of the float32 sums, so other bfloat16 roundings, carried
    through all layers): logits differ by 4.6e-3 (0.5B), 8.7e-3 (1.5B) and 1.2e-2 to 1.4e-2 (3B) in
    the 2-norm and by up to 6.4e-2 of the root mean square at one place; tokens do not differ."""
    if SHAPES[case["shape"]][7] == "f32":
        return {"rel": 1e-5, "max": 1e-4}
    return {"rel": 1.8e-2 if case["shape"] == "0.5b" else 3e-2, "max": 0.25}
