"""Performance cases: the calls a user of this package makes, over the range of sizes and options they are made in.

Three paths, each through the package's public entry points:

  step     one verify step of a target model: forward over B x (k + 1) positions against the paged cache, rejection
           sampling, commit (``VerifySession.step``; k = 0 is plain autoregressive decoding).  The cache bookkeeping is put
           back first (``spec_kv_restore``), so that a pass can be repeated.
  draft    one pass of a draft model, what ``DraftLoop`` does k times per step: forward over one position per sequence (two,
           fed with the target's features, on a step's first pass of a feature-fed draft), the draft's own draw, commit.
  sample   rejection sampling alone on logits in hand (a caller with a forward pass of its own).

Models and widths are those of ``synth_inputs``; ``layers`` > 0 takes that many layers of a model instead of all (every layer
runs the same launches, and a state with fewer of them is prepared in a fraction of the time).  Weights, cached context, page
lists, tokens and draft distributions are drawn from the seed; contexts are uniform between ``ctx_lo`` and ``ctx_hi`` and the
pages of the pool are handed out shuffled.

A step returns its logits.  The tokens that are drawn from them are not compared there: an accept test or the race between two
tokens of nearly equal keys goes the other way for about one sequence in 150 when the logits move by as little as another order
of the sums moves them.  The sample path draws from given logits, and its tokens have to be the same.
"""
import math

import numpy as np
import torch

import synth_inputs as si
from paper_2604_26779_amd import binding as sv
from paper_2604_26779_amd.session import VerifySession
from paper_2604_26779_amd.workloads import fill_pool

PAGE = si.PAGE_SIZE


def _case(name, path, model, B, k, ctx_lo=0, ctx_hi=0, layers=0):
    c = dict(path=path, model=model, B=B, k=k, ctx_lo=ctx_lo, ctx_hi=ctx_hi, layers=layers)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest configuration: launches and host work
        _case("tiny_fp32_b4_k3", "step", "tiny_fp32", 4, 3, 128, 128),
        # a small bf16 model: ragged row, column and context tails, still launch-bound
        _case("small_bf16_b5_k3", "step", "small_bf16", 5, 3, 37, 700),
        # one user: the latency of a speculation step at batch size 1
        _case("8b_b1_k3_ctx2k", "step", "llama8b_bf16", 1, 3, 2000, 2100),
        # the tail of a rollout, when few sequences are left: 28 rows
        _case("8b_b7_k3_ctx1k-8k", "step", "llama8b_bf16", 7, 3, 1024, 8192),
        # the benchmark's default workload: 128 rows
        _case("8b_b32_k3_ctx1k-8k", "step", "llama8b_bf16", 32, 3, 1024, 8192),
        # the same batch with 8-bit matrices and an 8-bit cache
        _case("8b_w8kv8_b32_k3_ctx1k-8k", "step", "llama8b_bf16_w8kv8", 32, 3, 1024, 8192),
        # the verify step of the draft + verify pair: 384 rows
        _case("8b_b64_k5_ctx4k", "step", "llama8b_bf16", 64, 5, 4096, 4096),
        # a large rollout batch: 1024 rows, the GEMMs are compute-bound
        _case("8b_b256_k3_ctx1k-6k", "step", "llama8b_bf16", 256, 3, 1024, 6144, 8),
        # mixture of experts: all 128 experts touched by a few rows each
        _case("moe_b64_k3_ctx1k-8k", "step", "moe235b_slice_bf16", 64, 3, 1024, 8192),
        # one pass of the pair's draft model
        _case("draft_b64_ctx4k", "draft", "draft1l_8b_bf16", 64, 0, 4096, 4096),
        # the first pass of a feature-fed draft with the reduced head, an odd batch
        _case("draft_eagle3r_b37_ctx1k-6k", "draft", "draft1l_eagle3r_8b_bf16", 37, 1, 1024, 6144),
        # the pair's sampling call
        _case("sample_b64_k5", "sample", "llama8b_bf16", 64, 5),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    path = rng.choice(["step", "step", "step", "step", "draft", "sample"])
    if path == "sample":
        k = rng.randint(0, 7)
        return _case("", path, "llama8b_bf16", _log_int(rng, 1, 1024 // (k + 1)), k)
    lo = _log_int(rng, 64, 8000)
    hi = lo + rng.randint(0, 8192)
    if path == "draft":
        model = rng.choice(["draft1l_8b_bf16", "draft1l_eagle3_8b_bf16", "draft1l_eagle3r_8b_bf16"])
        k = 0 if model == "draft1l_8b_bf16" else 1
        return _case("", path, model, _log_int(rng, 1, 200), k, lo, hi)
    model = rng.choice(["small_bf16", "llama8b_bf16", "llama8b_bf16", "llama8b_bf16_kv8", "llama8b_bf16_w8kv8", "moe235b_slice_bf16"])
    k = rng.randint(0, 7)
    B = _log_int(rng, 1, 1024 // (k + 1) if model.startswith("llama") else 64)
    layers = {"small_bf16": 0, "moe235b_slice_bf16": 2}.get(model, 8)
    # no more cached context than the largest listed case streams
    hi = min(hi, max(256, 600000 // B))
    return _case("", path, model, B, k, min(lo, hi), hi, layers)


def _config(case):
    cfg = dict(si.MODELS[case["model"]])
    if case["layers"] > 0:
        cfg["n_layers"] = case["layers"]
    return cfg


def _contexts(case, seed):
    rng = np.random.Generator(np.random.Philox(int(seed) + 1))
    return rng.integers(case["ctx_lo"], case["ctx_hi"] + 1, size=case["B"]).astype(np.int64), rng


class _State:
    """Session and buffers of one case; the library's handles are released with it."""

    sess = None

    def __del__(self):
        if self.sess is not None:
            self.sess.close()


def _open_session(st, cfg, case, seed, g):
    """Model, cache and the contexts of the batch, as a serving program holds them."""
    B, k = case["B"], case["k"]
    ctx, rng = _contexts(case, seed)
    weights = si.make_weights(cfg, seed=seed, device="cuda")
    for name in weights:            # a trained router is more decided than a random one: its last choice weighs a few percent
        if name.endswith("router"):
            weights[name] *= 4
    need = [-(-int(c) // PAGE) for c in ctx]
    n_pages = sum(need) + 2 * B + 8
    st.sess = VerifySession(cfg, weights, max_seqs=B, max_ctx_len=int(ctx.max()) + 256, n_pages=n_pages, device="cuda")
    if cfg["dtype"] == "bf16":      # the library keeps its own tiled copy of the matrices
        st.sess.weights = [t for n, t in weights.items() if n == "embed" or n.endswith("norm")]
    del weights
    fill_pool(st.sess, cfg, g, seed)
    order, at = rng.permutation(n_pages), 0
    for b in range(B):
        st.sess.assign(b, int(ctx[b]), [int(p) for p in order[at:at + need[b]]])
        at += need[b]
    st.seq_ids = torch.arange(B, dtype=torch.int32, device="cuda")
    st.snapshot = torch.empty(sv.spec_kv_state_bytes(st.sess.kv), dtype=torch.uint8, device="cuda")
    sv.spec_kv_snapshot(st.sess.kv, st.snapshot)


def prepare(case, seed):
    st = _State()
    st.case, st.seed = dict(case), int(seed)
    cfg = _config(case)
    B, k, V = case["B"], case["k"], cfg["vocab"]
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) + 2)
    if case["path"] != "sample":
        _open_session(st, cfg, case, seed, g)
    st.tokens = torch.randint(0, V, (B, k + 1), generator=g, device="cuda", dtype=torch.int32)
    if case["path"] == "draft":
        st.width = cfg.get("head_vocab", 0) or V
        st.q = torch.zeros((B, 1, V), dtype=torch.float32, device="cuda")
        st.drafts = torch.zeros((B, 1), dtype=torch.int32, device="cuda")
        st.feed = torch.zeros(B, dtype=torch.int32, device="cuda")
        st.fed = torch.full((B,), k, dtype=torch.int32, device="cuda")        # positions kept by the commit: all k + 1
        st.workspace = torch.empty(sv.spec_draft_sample_workspace_bytes(B), dtype=torch.uint8, device="cuda")
        st.token_map = st.features = st.hidden = None
        if cfg.get("head_vocab", 0):
            st.token_map = torch.from_numpy(si.make_token_map(cfg, seed=int(seed) + 29)).cuda()
        if cfg.get("fuse_taps", 0):
            st.features = torch.randn((B, k + 1, cfg["fuse_taps"] * cfg["d_model"]), generator=g, device="cuda")
            st.hidden = torch.zeros((B, k + 1, cfg["d_model"]), dtype=torch.float32, device="cuda")
        return st
    # the target's logits (sample path) or a stand-in of their spread, and a draft that follows them loosely
    logits = torch.randn((B, k + 1, V), generator=g, device="cuda") * 1.3
    if k:
        q = torch.empty((B, k, V), dtype=torch.float32, device="cuda")
        for i in range(k):
            q[:, i], st.tokens[:, i + 1] = si.device_draft_step(logits[:, i], 1.0, 1.0, g)
    else:
        q = None
    st.q, st.draft = q, st.tokens[:, 1:].contiguous()
    if case["path"] == "sample":
        st.logits = logits
        st.accept_len = torch.empty(B, dtype=torch.int32, device="cuda")
        st.out_tokens = torch.empty((B, k + 1), dtype=torch.int32, device="cuda")
        st.workspace = torch.empty(sv.spec_sample_workspace_bytes(B, k), dtype=torch.uint8, device="cuda")
    return st


def run(st):
    c = st.case
    B, k = c["B"], c["k"]
    if c["path"] == "sample":
        sv.spec_reject_sample(B, k, st.logits.shape[2], st.logits, st.q, st.draft, 1.0, st.seed, 0, st.accept_len, st.out_tokens,
                              None, st.workspace)
        return {"accept_len": st.accept_len, "out_tokens": st.out_tokens}
    sess = st.sess
    sv.spec_kv_restore(sess.kv, st.snapshot)
    if c["path"] == "step":
        logits, _, _ = sess.step(st.seq_ids, st.tokens, st.q, st.draft, 1.0, st.seed, 0)
        return {"logits": logits}
    V, W = st.width, st.q.shape[2]
    if st.features is not None:
        logits = sess.forward(st.seq_ids, st.tokens, features_in=st.features, hidden_out=st.hidden)
    else:
        logits = sess.forward(st.seq_ids, st.tokens)
    last, stride = logits.data_ptr() + k * V * 4, (k + 1) * V
    if st.token_map is not None:
        sv.spec_draft_sample_mapped(B, V, last, stride, 1.0, st.seed, 0, 0, st.drafts, 1, st.feed, 1, st.q, W, st.token_map, W,
                                    workspace=st.workspace)
    else:
        sv.spec_draft_sample(B, V, last, stride, 1.0, st.seed, 0, 0, st.drafts, 1, st.feed, 1, st.q, W, workspace=st.workspace)
    sv.spec_commit_kv(sess.kv, B, k, st.seq_ids, st.fed, None, None)
    out = {"logits": logits, "q": st.q}
    if st.hidden is not None:
        out["hidden"] = st.hidden
    return out


def work(case):
    """Matrices once (of a mixture's experts those that the rows reach), every cached key and value once, logits written,
    what the sampler reads of logits and q; two operations per matrix entry and row, four per row, channel and cached position."""
    cfg = _config(case)
    B, k, V = case["B"], case["k"], cfg["vocab"]
    M, H = B * (k + 1), cfg.get("head_vocab", 0) or V
    if case["path"] == "sample":
        return {"bytes": 4.0 * B * V * (k + 1 + (1 if k else 0)), "flops": 0.0}
    eb = 4 if cfg["dtype"] == "f32" else 2
    web = 1 if cfg.get("w_dtype") else eb
    kvb = 1 if cfg.get("kv_dtype") else eb
    L, D = cfg["n_layers"], cfg["d_model"]
    nq, nkv = cfg["n_q_heads"] * cfg["head_dim"], cfg["n_kv_heads"] * cfg["head_dim"]
    layer = active = (nq + 2 * nkv) * D + D * nq
    E = cfg.get("n_experts", 0)
    if E:
        one = 3 * cfg["expert_ffn_dim"] * D
        layer += E * D + E * (1.0 - (1.0 - cfg["top_k"] / E) ** M) * one
        active += E * D + cfg["top_k"] * one
    else:
        layer += 3 * cfg["ffn_dim"] * D
        active += 3 * cfg["ffn_dim"] * D
    fuse = 0
    if cfg.get("fuse_hidden", 0):
        fuse = (2 + cfg.get("fuse_taps", 0)) * D * D
    tokens = B * ((case["ctx_lo"] + case["ctx_hi"]) / 2.0 + k + 1)
    out = (2 * B * H + B * V if case["path"] == "draft" else 2 * M * H + (B * V if k else 0)) * 4.0
    return {"bytes": (L * layer + fuse) * web + H * D * web + tokens * 2 * nkv * kvb * L + out + M * D * eb,
            "flops": 2.0 * M * (L * active + fuse + H * D) + 4.0 * tokens * (k + 1) * nq * L}


def tolerance(case):
    # Another order of the sums moves an fp32 logit by about 1e-6 of its size.  The bf16 models round their activations to 16 bits
    # at every projection (hi + lo bf16 pairs or one fp16), so that two correct orders differ by about one such rounding per
    # layer: with other K splits and attention chunks 2.2e-3 (largest 1.3e-2) after 32 layers, 3e-4 (2e-3) after a draft's one.
    # In a mixture a few rows per hundred then take another last expert as well.
    if case["path"] == "sample":
        return "exact"
    if si.MODELS[case["model"]]["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-4}
    if case["path"] == "draft":
        return {"rel": 3e-3, "max": 2e-2}
    if si.MODELS[case["model"]].get("n_experts", 0):
        return {"rel": 1.5e-2, "max": 5e-1}
    return {"rel": 1e-2, "max": 6e-2}
