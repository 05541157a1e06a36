"""The race kernels evaluate an entry's key in fp64 only where its fp32 bounds let it win: parity with the oracle (every key in
fp64) where those bounds are at their limits - vocabularies around a round of the scan and rows that cannot be read in 16-byte
words, weights beyond the range of fp32, residuals that cancel to rounding noise or vanish."""
import numpy as np
import pytest
import torch

from oracle import sampler as oracle_sampler
from tests.test_gpu_sampler import _run_gpu

pytestmark = pytest.mark.gpu

SIZES = [3, 1023, 4096, 16384, 16388, 65541, 70000]


def _softmax(z):
    e = np.exp(z - z.max(-1, keepdims=True))
    return e / e.sum(-1, keepdims=True)


@pytest.mark.parametrize("V", SIZES)
@pytest.mark.parametrize("temperature,offset", [(1.0, 0.0), (0.02, 0.0), (0.7, 5000.0)])
@pytest.mark.parametrize("draft_kind", ["loose", "noise", "zero", "one-hot"])
def test_reject_races_at_the_limits_of_their_bounds(V, temperature, offset, draft_kind):
    B, k = 4, 2
    rng = np.random.default_rng(V)
    logits = (rng.standard_normal((B, k + 1, V)) * 3 + offset).astype(np.float32)
    p = _softmax(logits[:, :k].astype(np.float64) / temperature)
    if draft_kind == "loose":
        q = _softmax((logits[:, :k].astype(np.float64) + rng.standard_normal((B, k, V))) / temperature).astype(np.float32)
    elif draft_kind == "zero":                      # q above p everywhere: the residual is identically zero
        q = (3.0 * p + 1e-30).astype(np.float32)
    else:
        q = p.astype(np.float32)
    draft = rng.integers(0, V, size=(B, k)).astype(np.int32)
    draft[:, 0] = logits[:, 0].argmax(-1)
    if draft_kind == "noise":                       # p - q is rounding noise except where the rejected draft sits
        np.put_along_axis(q, draft[..., None], (2.5 * np.take_along_axis(p, draft[..., None], -1)).astype(np.float32), -1)
    if draft_kind == "one-hot":
        explicit = np.zeros_like(q)
        np.put_along_axis(explicit, draft[..., None], 1.0, -1)
        from paper_2604_26779_amd import binding as sv
        dl, dd = torch.from_numpy(logits).cuda(), torch.from_numpy(draft).cuda()
        n, out = torch.empty(B, dtype=torch.int32, device="cuda"), torch.empty((B, k + 1), dtype=torch.int32, device="cuda")
        ws = torch.empty(sv.spec_sample_workspace_bytes(B, k), dtype=torch.uint8, device="cuda")
        sv.spec_reject_sample(B, k, V, dl, None, dd, temperature, 77, 4, n, out, None, ws)
        n_gpu, out_gpu = n.cpu().numpy(), out.cpu().numpy()
        q = explicit
    else:
        n_gpu, out_gpu, _ = _run_gpu(logits, q, draft, temperature, 77, 4)
    n_or, out_or = oracle_sampler.reject_sample(logits, q, draft, temperature, 77, 4)
    assert np.array_equal(n_gpu, n_or) and np.array_equal(out_gpu, out_or)


@pytest.mark.parametrize("V", SIZES)
@pytest.mark.parametrize("temperature", [1.0, 0.02])
@pytest.mark.parametrize("mapped", [False, True])
def test_draft_draw_at_the_limits_of_its_bounds(V, temperature, mapped):
    from paper_2604_26779_amd import binding as sv
    B = 3
    rng = np.random.default_rng(V + 1)
    logits = (rng.standard_normal((B, V)) * 3).astype(np.float32)
    token_map = np.arange(V, dtype=np.int32) * 2 + 1
    width = 2 * V + 1 if mapped else V
    dl = torch.from_numpy(logits).cuda()
    tok, q = torch.empty(B, dtype=torch.int32, device="cuda"), torch.full((B, width), -1.0, device="cuda")
    if mapped:
        sv.spec_draft_sample_mapped(B, V, dl, V, temperature, 5, 2, 1, tok, 1, None, 1, q, width, torch.from_numpy(token_map).cuda(), width)
        x_or, q_or = oracle_sampler.draft_sample_mapped(logits, token_map, width, temperature, 5, 2, 1)[:2]
    else:
        sv.spec_draft_sample(B, V, dl, V, temperature, 5, 2, 1, tok, 1, None, 1, q, V)
        x_or, q_or = oracle_sampler.draft_sample(logits, temperature, 5, 2, 1)[:2]
    x_or, q_or = (x_or, q_or) if np.ndim(x_or) == 1 else (q_or, x_or)
    assert np.array_equal(tok.cpu().numpy(), x_or)
    # q is an fp64 softmax rounded to fp32 on both sides: at most one unit apart (below the smallest normal number: flushed)
    got = q.cpu().numpy()
    assert np.all(np.abs(got - q_or) <= 2.0 ** -23 * q_or + 1.2e-38)


def _run_one_hot(logits, draft, temperature, seed, step):
    """No q array: one-hot drafts."""
    from paper_2604_26779_amd import binding as sv
    B, k1, V = logits.shape
    dl, dd = torch.from_numpy(logits).cuda(), torch.from_numpy(draft).cuda()
    n, out = torch.empty(B, dtype=torch.int32, device="cuda"), torch.empty((B, k1), dtype=torch.int32, device="cuda")
    ws = torch.empty(sv.spec_sample_workspace_bytes(B, k1 - 1), dtype=torch.uint8, device="cuda")
    sv.spec_reject_sample(B, k1 - 1, V, dl, None, dd, temperature, seed, step, n, out, None, ws)
    return n.cpu().numpy(), out.cpu().numpy()


def _check_draft_draw(logits, temperature, mapped):
    from paper_2604_26779_amd import binding as sv
    B, V = logits.shape
    token_map = np.arange(V, dtype=np.int32) * 2 + 1
    width = 2 * V + 1 if mapped else V
    dl = torch.from_numpy(logits).cuda()
    tok, q = torch.empty(B, dtype=torch.int32, device="cuda"), torch.full((B, width), -1.0, device="cuda")
    if mapped:
        sv.spec_draft_sample_mapped(B, V, dl, V, temperature, 5, 2, 1, tok, 1, None, 1, q, width, torch.from_numpy(token_map).cuda(), width)
        x_or, q_or = oracle_sampler.draft_sample_mapped(logits, token_map, width, temperature, 5, 2, 1)[:2]
    else:
        sv.spec_draft_sample(B, V, dl, V, temperature, 5, 2, 1, tok, 1, None, 1, q, V)
        x_or, q_or = oracle_sampler.draft_sample(logits, temperature, 5, 2, 1)[:2]
    assert np.array_equal(tok.cpu().numpy(), x_or)
    # q is an fp64 softmax rounded to fp32 on both sides: at most one unit apart (below the smallest normal number: flushed)
    got = q.cpu().numpy()
    assert np.all(np.abs(got - q_or) <= 2.0 ** -23 * q_or + 1.2e-38)


# (temperature, spread of the logits): infinite; near fp32's largest number, with logits that still matter there; where log2(e) / T or T
# itself leaves fp32's normal range, with logits of every size beside it
EXTREME_T = [(np.inf, 3.0), (3e38, 5e37), (1e30, 3.0), (1e30, 1e30), (1e-37, 1e-37), (1e-38, 3.0), (1e-39, 2e-39), (1e-39, 3.0),
             (1e-45, 3.0), (1e-45, 1e31)]


@pytest.mark.parametrize("V", [1023, 16388])
@pytest.mark.parametrize("temperature,spread", EXTREME_T)
@pytest.mark.parametrize("draft_kind", ["explicit", "one-hot"])
def test_reject_at_extreme_temperatures(V, temperature, spread, draft_kind):
    B, k = 6, 2
    rng = np.random.default_rng(V)
    logits = (rng.standard_normal((B, k + 1, V)) * spread).astype(np.float32)
    t64 = np.float64(np.float32(temperature))
    q = _softmax((logits[:, :k].astype(np.float64) + rng.standard_normal((B, k, V)) * spread) / t64).astype(np.float32)
    draft = rng.integers(0, V, size=(B, k)).astype(np.int32)
    draft[:, 0] = logits[:, 0].argmax(-1)
    if draft_kind == "one-hot":
        q = np.zeros_like(q)
        np.put_along_axis(q, draft[..., None], 1.0, -1)
    n_or, out_or = oracle_sampler.reject_sample(logits, q, draft, temperature, 77, 4)
    if draft_kind == "one-hot":
        n_gpu, out_gpu = _run_one_hot(logits, draft, temperature, 77, 4)
    else:
        n_gpu, out_gpu, _ = _run_gpu(logits, q, draft, temperature, 77, 4)
    assert np.array_equal(n_gpu, n_or) and np.array_equal(out_gpu, out_or)
    assert np.all(np.take_along_axis(out_gpu, n_gpu[:, None].astype(np.int64), 1) >= 0)


@pytest.mark.parametrize("V", [1023, 16388])
@pytest.mark.parametrize("temperature,spread", EXTREME_T)
@pytest.mark.parametrize("mapped", [False, True])
def test_draft_draw_at_extreme_temperatures(V, temperature, spread, mapped):
    rng = np.random.default_rng(V + 1)
    _check_draft_draw((rng.standard_normal((5, V)) * spread).astype(np.float32), temperature, mapped)


@pytest.mark.parametrize("V", [3, 1023, 16388, 70000])
@pytest.mark.parametrize("temperature", [0.7, np.inf])
@pytest.mark.parametrize("row", ["+inf", "all -inf"])
@pytest.mark.parametrize("mapped", [False, True])
def test_draft_row_without_a_distribution_gives_nan_and_is_rejected(V, temperature, row, mapped):
    """A draft that overflowed: token -1 and a q of NaN, not numbers that look like probabilities; the verifier then rejects the -1 and
    emits from the target's own distribution (for NaN the residual is identically zero)."""
    from paper_2604_26779_amd import binding as sv
    B = 3
    rng = np.random.default_rng(V)
    logits = (rng.standard_normal((B, V)) * 3).astype(np.float32)
    good = logits.copy()
    logits[1] = -np.inf if row == "all -inf" else logits[1]
    if row == "+inf":
        logits[1, rng.integers(0, V)] = np.inf
    dl = torch.from_numpy(logits).cuda()
    tok, q = torch.empty(B, dtype=torch.int32, device="cuda"), torch.full((B, V), -1.0, device="cuda")
    if mapped:
        sv.spec_draft_sample_mapped(B, V, dl, V, temperature, 5, 2, 1, tok, 1, None, 1, q, V, torch.arange(V, dtype=torch.int32, device="cuda"), V)
    else:
        sv.spec_draft_sample(B, V, dl, V, temperature, 5, 2, 1, tok, 1, None, 1, q, V)
    got = q.cpu().numpy()
    assert tok[1].item() == -1 and np.all(np.isnan(got[1]))
    x_or, q_or = oracle_sampler.draft_sample(good, temperature, 5, 2, 1)
    for b in (0, 2):
        assert tok[b].item() == x_or[b] and np.all(np.abs(got[b] - q_or[b]) <= 2.0 ** -23 * q_or[b] + 1.2e-38)
    target = (rng.standard_normal((B, 2, V)) * 3).astype(np.float32)
    draft = tok.cpu().numpy().reshape(B, 1)
    n_gpu, out_gpu, _ = _run_gpu(target, got.reshape(B, 1, V), draft, temperature, 77, 4)
    n_or, out_or = oracle_sampler.reject_sample(target, got.reshape(B, 1, V), np.maximum(draft, 0), temperature, 77, 4)
    assert n_gpu[1] == 0 and np.array_equal(n_gpu, n_or) and np.array_equal(out_gpu, out_or)


@pytest.mark.parametrize("V", [3, 1023, 16388])
@pytest.mark.parametrize("mask", [-np.inf, np.finfo(np.float32).min])
@pytest.mark.parametrize("kept", [1, 2, 700])
def test_masked_rows(V, mask, kept):
    """Rows masked with -inf or with the type's lowest value but for a few entries, one of them wholly -inf in some ranges of the scan;
    a target row that is -inf throughout, or holds +inf, emits -1 as the oracle does."""
    B, k = 5, 2
    rng = np.random.default_rng(V + kept)
    logits = np.full((B, k + 1, V), mask, dtype=np.float32)
    for b in range(B):
        for i in range(k + 1):
            at = rng.permutation(V)[:kept]
            logits[b, i, at] = rng.standard_normal(len(at)) * 3
    for b, x in ((3, np.inf), (4, -np.inf)):
        logits[b, 0, :] = -np.inf
        logits[b, 0, V // 2] = x
    draft = logits[:, :k].argmax(-1).astype(np.int32)
    q = np.full((B, k, V), 1.0 / V, dtype=np.float32)
    n_or, out_or = oracle_sampler.reject_sample(logits, q, draft, 0.7, 77, 4)
    n_gpu, out_gpu, _ = _run_gpu(logits, q, draft, 0.7, 77, 4)
    assert np.array_equal(n_gpu, n_or) and np.array_equal(out_gpu, out_or)
    assert np.all(out_gpu[3:, 0] == -1)


@pytest.mark.parametrize("V", [1023, 16388, 70000])
@pytest.mark.parametrize("draft_kind", ["elsewhere", "top", "one-hot", "tiny residual", "tiny residual in one range"])
def test_reject_races_of_peaked_rows(V, draft_kind):
    """A few entries far above the rest, whose weights lie below fp32's range, and residuals of nothing but such weights: the race's
    supposed lower bound holds, or does not and everything is looked at again."""
    B, k, temperature = 6, 2, 0.2
    rng = np.random.default_rng(V)
    logits = (rng.standard_normal((B, k + 1, V)) * 2).astype(np.float32)
    top = rng.integers(0, V, size=(B, k + 1))
    np.put_along_axis(logits, top[..., None], 25.0, -1)
    p = _softmax(logits[:, :k].astype(np.float64) / temperature)
    draft = rng.integers(0, V, size=(B, k)).astype(np.int32)
    q = np.zeros((B, k, V), dtype=np.float32)
    if draft_kind == "elsewhere" or draft_kind == "one-hot":
        np.put_along_axis(q, draft[..., None], 1.0, -1)
    elif draft_kind == "top":                      # rejected at the top entry: what is left is of the order of 1e-35 and below
        draft = top[:, :k].astype(np.int32)
        np.put_along_axis(q, draft[..., None], np.float32(3e8), -1)
    else:                                          # q covers everything but entries of tiny weight
        q = (1.5 * p + 1e-20).astype(np.float32)
        if draft_kind == "tiny residual":
            q[p < 1e-31] = 0.0
        else:
            q[..., V - 300:][p[..., V - 300:] < 1e-31] = 0.0
        draft = top[:, :k].astype(np.int32)
        np.put_along_axis(q, draft[..., None], np.float32(3e8), -1)
    n_or, out_or = oracle_sampler.reject_sample(logits, q, draft, temperature, 77, 4)
    if draft_kind == "one-hot":
        n_gpu, out_gpu = _run_one_hot(logits, draft, temperature, 77, 4)
    else:
        n_gpu, out_gpu, _ = _run_gpu(logits, q, draft, temperature, 77, 4)
    assert np.array_equal(n_gpu, n_or) and np.array_equal(out_gpu, out_or)


@pytest.mark.parametrize("V", [1023, 16388, 70000])
@pytest.mark.parametrize("top", [25.0, 60.0])
def test_draft_draw_whose_map_leaves_out_the_top(V, top):
    """The most probable entry maps outside the target's vocabulary: the draw is decided among keys far below the bound it gives."""
    from paper_2604_26779_amd import binding as sv
    B, temperature = 4, 0.2
    rng = np.random.default_rng(V)
    logits = (rng.standard_normal((B, V)) * 2).astype(np.float32)
    logits[:, V // 3] = top
    token_map = np.arange(V, dtype=np.int32)
    token_map[V // 3] = V + 5
    tok, q = torch.empty(B, dtype=torch.int32, device="cuda"), torch.full((B, V), -1.0, device="cuda")
    sv.spec_draft_sample_mapped(B, V, torch.from_numpy(logits).cuda(), V, temperature, 5, 2, 1, tok, 1, None, 1, q, V,
                                torch.from_numpy(token_map).cuda(), V)
    p = _softmax(logits.astype(np.float64) / temperature)
    for b in range(B):
        key = np.array([p[b, v] / -np.log(oracle_sampler.uniform_draft(5, 2, b, 1, v)) for v in range(V)])
        key[V // 3] = -1.0
        assert tok[b].item() == int(key.argmax())
    want = p.copy()
    want[:, V // 3] = 0.0
    assert np.all(np.abs(q.cpu().numpy() - want) <= 2.0 ** -23 * want + 1.2e-38)


@pytest.mark.parametrize("V", [50, 1003, 16384, 140000])
@pytest.mark.parametrize("nan_bits", [0x7FC00000, 0x7F800001, 0xFF800001])
@pytest.mark.parametrize("temperature", [1.0, 0.01])
def test_nan_beside_the_largest_logit(V, nan_bits, temperature):
    """A NaN among a row's finite logits, quiet or signalling, is left out: the same draws as with -inf in its place, also where the row's largest logit stands
    right beside it (on either side, at any place of a group of four) and nothing else counts."""
    from paper_2604_26779_amd import binding as sv
    B, k = 12, 1
    rng = np.random.default_rng(V)
    logits = rng.standard_normal((B, k + 1, V)).astype(np.float32)
    holes = np.zeros(logits.shape, dtype=bool)
    for b in range(B):
        for i in range(k + 1):
            at = int(rng.integers(0, V - 8)) // 4 * 4 + b % 4
            logits[b, i, at] = 30.0
            holes[b, i, at + 1 if b % 2 or at == 0 else at - 1] = True
            holes[b, i, rng.integers(0, V)] |= b >= 8
            holes[b, i, at] = False
    q = _softmax(rng.standard_normal((B, k, V))).astype(np.float32)
    draft = rng.integers(0, V, size=(B, k)).astype(np.int32)
    draft[::2, 0] = logits[::2, 0].argmax(-1)
    outcome = []
    for fill in (nan_bits, 0xFF800000):
        L = logits.copy()
        L.view(np.uint32)[holes] = fill
        dl = torch.from_numpy(L.view(np.int32)).cuda().view(torch.float32)
        n, out = torch.empty(B, dtype=torch.int32, device="cuda"), torch.empty((B, k + 1), dtype=torch.int32, device="cuda")
        ws = torch.empty(sv.spec_sample_workspace_bytes(B, k), dtype=torch.uint8, device="cuda")
        sv.spec_reject_sample(B, k, V, dl, torch.from_numpy(q).cuda(), torch.from_numpy(draft).cuda(), temperature, 77, 4, n, out, None, ws)
        tok, qd = torch.empty(B, dtype=torch.int32, device="cuda"), torch.empty((B, V), device="cuda")
        sv.spec_draft_sample(B, V, dl, (k + 1) * V, temperature, 5, 2, 1, tok, 1, None, 1, qd, V)
        outcome.append([n.cpu().numpy(), out.cpu().numpy(), tok.cpu().numpy(), qd.cpu().numpy()[~holes[:, 0]]])
    for a, b in zip(*outcome):
        assert np.array_equal(a, b)
    assert np.array_equal(outcome[0][2], logits[:, 0].argmax(-1)) or temperature == 1.0
