"""Attention of bf16 models with head_dim 32 on the matrix cores: parity with
the oracle at the edges of its tiles (32-key sub-blocks, 128-key stages,
16/32-query waves, 64/128/256-candidate items), and items of every size giving
the same bits."""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_00422_amd import upr
from synth import make_inputs

from .gpu_util import GpuRun, assert_cache_match, assert_scores_match, say

pytestmark = pytest.mark.gpu

SMALL = [
    # (history lens, candidate lens, d, H, L, F)
    ([0, 1, 31, 32, 33, 127, 128, 129, 300], [1, 129, 64, 65, 63, 128, 5, 0, 257], 128, 4, 2, 256),
    ([257, 0, 640], [17, 16, 15], 64, 2, 1, 128),
]


@pytest.mark.parametrize("case", range(len(SMALL)))
def test_edges_match_oracle(case):
    n, k, d, H, L, F = SMALL[case]
    inp = make_inputs(n, k, d, H, L, F, dtype="bf16", seed=600 + case, variant="perturbed")
    say(f"[gpu] head32 case {case}: d={d} H={H} L={L} histories {n} candidates {k}")
    run = GpuRun(inp)
    run.encode()
    run.rank()
    ref_cache = oracle.encode(inp.weights, d, H, L, F, inp.hist_emb, inp.hist_offsets)
    assert_cache_match(run.cache_np(), ref_cache, np.arange(sum(n)), "head32 cache")
    ref = oracle.rank(inp.weights, d, H, L, F, ref_cache, inp.hist_offsets, inp.cand_emb, inp.cand_offsets)
    err = assert_scores_match(run.scores_np(), ref, "head32")
    say(f"[gpu] head32 case {case}: max |score err| {err:.3e}")


@pytest.mark.parametrize("n,k,U,d,H", [(300, 1000, 16, 256, 8),      # 128-candidate items
                                       (4200, 4130, 2, 512, 16)])    # 256-candidate items
def test_item_sizes_agree_bit_for_bit(n, k, U, d, H):
    """A batch against its users one by one (64-candidate items)."""
    hl = [n + 37 * (u % 3) for u in range(U)]
    inp = make_inputs(hl, [k] * U, d, H, 1, 128, dtype="bf16", seed=610, variant="perturbed")
    say(f"[gpu] head32 items: {U} users x {k} candidates, histories {n}+")
    run = GpuRun(inp)
    run.encode()
    run.rank()
    batch = run.scores_np().copy()
    assert np.all(np.isfinite(batch))
    ho, co = inp.hist_offsets, inp.cand_offsets
    for u in (0, U - 1):
        run.scores.fill_(float("nan"))
        run.rank(hoff=np.array([ho[u], ho[u + 1]], np.int32), coff=np.array([co[u], co[u + 1]], np.int32))
        assert np.array_equal(run.scores_np()[co[u]:co[u + 1]], batch[co[u]:co[u + 1]]), f"user {u}"
    rows = co[U - 1] + np.arange(0, k, 211)
    cache = run.cache_np()
    ref = oracle.rank(inp.weights, d, H, 1, 128, cache, inp.hist_offsets, inp.cand_emb, inp.cand_offsets,
                      users=[U - 1], cand_rows=rows)
    err = assert_scores_match(batch[rows], ref[rows], "head32 items, on the GPU's cache")
    say(f"[gpu] head32 items: max |score err| {err:.3e} over {rows.size} sampled candidates")


def test_exact_redo(monkeypatch):
    """The exact two-pass softmax (a testing hook forces it) matches the oracle."""
    inp = make_inputs([200, 5], [70, 33], 128, 4, 1, 256, dtype="bf16", seed=620, variant="sharp")
    run = GpuRun(inp)
    monkeypatch.setenv("UPR_ATTN_EXACT", "1")
    run.encode()
    run.rank()
    got = run.scores_np()
    ref = oracle.rank(inp.weights, 128, 4, 1, 256, run.cache_np(), inp.hist_offsets, inp.cand_emb,
                      inp.cand_offsets)
    assert_scores_match(got, ref, "head32 exact redo, on the GPU's cache", scale=2.0)


def _attention_of(monkeypatch, Wq, bq, X, K, V):
    """Attention output [R, H, D] (float64) of a one-layer d 64 model with 32-value
    heads, query projection Wq, bq and no key or value of a candidate's own
    (own logit 0, own value 0), for candidates X over one user's history K, V
    [H, n, D], and the queries it used.  The rank call is stopped after the
    attention (UPR_STOP_AFTER)."""
    d, H, D, F, R, n = 64, 2, 32, 64, X.shape[0], K.shape[1]
    zero = np.zeros
    blob = [np.ones(d), zero(d), Wq, bq, zero((d, d)), zero(d), zero((d, d)), zero(d),                  # LN1, Wq, Wk, Wv
            np.eye(d), zero(d), np.ones(d), zero(d), zero((F, d)), zero(F), zero((d, F)), zero(d),      # Wo, LN2, W1, W2
            np.ones(d), zero(d), np.ones(d), zero(1)]
    model = upr.Model(upr.make_config(d, H, 1, F, "bf16"),
                      np.concatenate([np.ravel(x) for x in blob]).astype(np.float32))
    cache = model.new_cache(n)
    cache[0, 0], cache[0, 1] = K.cuda(), V.cuda()
    hoff, coff = np.array([0, n], np.int32), np.array([0, R], np.int32)
    hd, cd = torch.from_numpy(hoff).cuda(), torch.from_numpy(coff).cuda()
    scores = torch.empty(R, dtype=torch.float32, device="cuda")
    ws = model.workspace(upr.upr_rank_workspace_bytes(model.handle, upr.segments(hoff, hd), upr.segments(coff, cd)))
    monkeypatch.setenv("UPR_STOP_AFTER", "3")   # LayerNorm and work list, q|k|v, attention
    model.rank(cache, hoff, hd, X.cuda(), coff, cd, scores, ws=ws)
    torch.cuda.synchronize()
    assert R * d % 128 == 0                     # whole 256-byte blocks: no gaps between
    at = R * d * 4 + R * d * 2                  # past the residual and LN1
    q = ws[at:at + R * 3 * d * 2].view(torch.bfloat16).double().cpu().reshape(R, 3, H, D)[:, 0]
    at += R * 3 * d * 2
    return ws[at:at + R * d * 2].view(torch.float16).double().cpu().reshape(R, H, D), q


def test_probabilities_weigh_values_in_fp32(monkeypatch):
    """Two history keys of nearly equal logits with opposite values A: the
    attention output A (p0 - p1) / (1 + p0 + p1) is the probabilities' error
    but for 2^-13 of A, and fp16 storage keeps 11 bits of that.  Against
    float64 on the GPU's own queries."""
    d, H, D, R, A = 64, 2, 32, 700, 1024.0
    rng = np.random.default_rng(630)
    k0 = torch.from_numpy(rng.uniform(0.07, 0.12, (H, D)).astype(np.float32)).to(torch.bfloat16)
    k1 = k0.clone()
    k1[:, ::8] += 2.0 ** -11                    # one or two units of bf16 in four of 32 values
    V = torch.tensor([A, -A], dtype=torch.bfloat16)[None, :, None].expand(H, 2, D)
    X = torch.from_numpy(rng.standard_normal((R, d)).astype(np.float32)).to(torch.bfloat16)
    o, q = _attention_of(monkeypatch, np.eye(d) / 8, np.zeros(d), X, torch.stack([k0, k1], 1), V)
    p0, p1 = (torch.exp2((q * k.double()).sum(-1)) for k in (k0, k1))
    ref = (A * (p0 - p1) / (1 + p0 + p1))[..., None]
    # logits: sums of 32 products, below 0.5 in all, at 2^-24 a rounding; the
    # exponential another 2^-23: 2^-22 of A for the pair with room to spare.
    # (Two bf16 terms per probability leave up to 2^-18 of it.)
    err = (o - ref).abs()
    bound = A * 2.0 ** -22 + ref.abs() * 2.0 ** -11
    assert ref.abs().max() < A * 2.0 ** -9
    say(f"[gpu] head32 probabilities: worst error {float((err / A).max()):.2e} of A, of the bound {float((err / bound).max()):.2f}")
    assert bool((err <= bound).all())


@pytest.mark.parametrize("excess", [[120, 0.5], [127, 0.875], [127, 0.99609375, 0.00244140625], [127, 2], [127, 127]])
def test_logits_far_above_the_own(monkeypatch, excess):
    """A history logit up to 2^128 and more above the candidate's own, which the
    softmax takes as its reference: just below where the probability overflows
    as bf16, between that and fp32's largest, and beyond.  The history's value
    takes all of the weight."""
    d, H, D, R = 64, 2, 32, 4
    K = torch.zeros(H, 3, D, dtype=torch.bfloat16)
    K[:, 1, :len(excess)] = torch.tensor(excess, dtype=torch.bfloat16)
    V = torch.tensor([1.0, 3.0, -2.0], dtype=torch.bfloat16)[None, :, None].expand(H, 3, D)
    bq = np.full(d, np.sqrt(32) * np.log(2))    # queries of 1 (pre-scaled by log2(e) / sqrt(32))
    o, q = _attention_of(monkeypatch, np.zeros((d, d)), bq, torch.zeros(R, d, dtype=torch.bfloat16), K, V)
    assert bool((q == 1).all())
    say(f"[gpu] head32 logits {sum(excess)} above the own: {o.min().item()}..{o.max().item()}")
    assert bool((o == 3).all())
