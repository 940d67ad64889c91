"""Attention of bf16 models with head_dim 32 on the matrix cores: parity with
the oracle at the edges of its tiles (32-key sub-blocks, 128-key stages,
16/32-query waves, 64/128/256-candidate items), and items of every size giving
the same bits."""
import numpy as np
import pytest

import oracle
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
