"""Shared test helpers: oracle-side input preparation and the comparison rules of the parity tests."""
import numpy as np

import synth_inputs as si
from oracle import forward as of


def oracle_drafts(cfg, w_or, kv_or, tokens0, ctx_len, k, noise_std, temperature, seed):
    """Draft tokens and draft distributions the way the workloads define them:
    q_i = softmax((target logits of the prefix + N(0, noise_std)) / T), x_i ~ q_i, with the target
    logits taken from the ORACLE run autoregressively (inputs may come from the oracle, never from
    the HIP path).  Returns tokens [B, k+1] (row 0 = tokens0) and q [B, k, V] fp32."""
    rng = np.random.Generator(np.random.Philox(int(seed) + 4))
    B, V = len(tokens0), cfg["vocab"]
    toks = np.asarray(tokens0, dtype=np.int32).reshape(B, 1)
    q = np.zeros((B, k, V), dtype=np.float32)
    for i in range(k):
        logits, _ = of.verify_forward(cfg, w_or, kv_or, toks, ctx_len)
        qi = si.noisy_draft_distribution(logits[:, -1, :], rng.standard_normal((B, V)) * noise_std, temperature)
        q[:, i, :] = qi
        toks = np.concatenate([toks, si.draw_from(qi, rng).reshape(B, 1)], axis=1)
    return toks.astype(np.int32), q


def sampler_exemptions(pqu, keys, ratio_tol=1e-3, tie_tol=1e-4):
    """Which trials may legitimately differ between fp32 kernels and the fp64 oracle.

    near_threshold[b]: some evaluated accept test had |u - P/Q| < ratio_tol (the exemption the
    build's target states); near_tie[b]: the two best race keys differ by less than tie_tol relative."""
    B, k, _ = pqu.shape
    near_threshold = np.zeros(B, dtype=bool)
    for b in range(B):
        for i in range(k):
            P, Q, u = pqu[b, i]
            if np.isnan(u):
                continue
            if Q > 0 and abs(u - P / Q) < ratio_tol:
                near_threshold[b] = True
    near_tie = (keys[:, 1] > 0) & ((keys[:, 0] - keys[:, 1]) <= tie_tol * keys[:, 0])
    return near_threshold, near_tie


def assert_sampler_parity(n_gpu, out_gpu, n_or, out_or, pqu, keys, max_exempt_frac=0.05, exact=False):
    """Bit-exact accept lengths and tokens except counted near-threshold / near-tie trials.

    exact: no exemption at all - for the sampler on its own, where both sides get identical inputs and the kernels
    decide in fp64 like the oracle (the near-* counts are still reported); the exemptions remain for whole steps, whose
    logits carry the forward pass's error."""
    near_threshold, near_tie = sampler_exemptions(pqu, keys)
    B = len(n_or)
    used = 0
    for b in range(B):
        same = n_gpu[b] == n_or[b] and np.array_equal(out_gpu[b], out_or[b])
        if same:
            continue
        if exact:
            raise AssertionError("sampler mismatch at b=%d (no exemptions): gpu n=%d %s, oracle n=%d %s, P/Q/u=%s keys=%s" %
                                 (b, n_gpu[b], out_gpu[b], n_or[b], out_or[b], pqu[b], keys[b]))
        if near_threshold[b]:
            used += 1
            continue
        if near_tie[b] and n_gpu[b] == n_or[b] and np.array_equal(out_gpu[b][:n_or[b]], out_or[b][:n_or[b]]):
            used += 1
            continue
        raise AssertionError("sampler mismatch at b=%d: gpu n=%d %s, oracle n=%d %s, P/Q/u=%s keys=%s" %
                             (b, n_gpu[b], out_gpu[b], n_or[b], out_or[b], pqu[b], keys[b]))
    assert used <= max(2, max_exempt_frac * B), "too many exempted trials: %d of %d" % (used, B)
    return dict(trials=B, near_threshold=int(near_threshold.sum()), near_tie=int(near_tie.sum()), exempt_used=used)


def logits_close(got, want, abs_tol, rel_tol):
    got = np.asarray(got, dtype=np.float64)
    want = np.asarray(want, dtype=np.float64)
    err = np.abs(got - want)
    bound = abs_tol + rel_tol * np.abs(want)
    worst = float((err - bound).max())
    return worst <= 0.0, float(err.max()), worst


def random_norm_gains(weights, seed):
    """RMSNorm gains 1 + 0.3 N(0,1) in the weights' own type (the generator's are all 1, which would hide a gain
    applied at the wrong place or taken from the wrong layer)."""
    import torch
    g = torch.Generator().manual_seed(int(seed) + 4242)
    for name, t in weights.items():
        if name.endswith("norm"):
            weights[name] = (1.0 + 0.3 * torch.randn(t.shape, generator=g)).to(t.dtype).to(t.device)
    return weights


def gemm_shape(N, K, M, w8=False, f16=False, whole=False, swiglu=False):
    """The tile the library takes for a GEMM of N columns at M rows: dict(mb = 32-row blocks, tile_nb = 32-column blocks, kunit, m_tiles, n_tiles, wide,
    one_block), under the tuning parameters as they are.  Needs no GPU.  f16: one fp16 value per activation; whole: K is never split (the head)."""
    import ctypes

    from paper_2604_26779_amd import binding

    class PackedW(ctypes.Structure):
        _fields_ = [("data", ctypes.c_void_p)] + [(n, ctypes.c_int32) for n in ("N", "K", "n_blocks", "k_steps", "w8", "f16")] + \
                   [("scale", ctypes.c_void_p), ("whole", ctypes.c_int32)]

    class GemmShape(ctypes.Structure):
        _fields_ = [(n, ctypes.c_int) for n in ("mb", "tile_nb", "kunit", "m_tiles", "n_tiles")] + [("wide", ctypes.c_bool), ("one_block", ctypes.c_bool)]

    fn = binding.lib()["_ZN5specv10gemm_shapeERKNS_7PackedWEib"]
    fn.restype, fn.argtypes = GemmShape, [ctypes.POINTER(PackedW), ctypes.c_int, ctypes.c_bool]
    g = fn(ctypes.byref(PackedW(None, N, K, -(-N // 32), K // 16, int(w8), int(f16), None, int(whole))), M, swiglu)
    return {n: getattr(g, n) for n, _ in GemmShape._fields_}
