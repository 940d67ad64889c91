"""Attention of fp32 models on the matrix cores, at the edges of its tiles
(16-key blocks, 64/128-key stages, the two key halves, 16-query waves,
32-query items), and the calls that keep the one-wave-per-row kernel: a
workspace without room for the work list."""
import numpy as np
import pytest

import oracle
from paper_2606_00422_amd import upr
from synth import make_inputs

from .gpu_util import GpuRun, say

pytestmark = pytest.mark.gpu

# Sums of up to n + d terms of order 1 in fp32, a few layers deep: 2^-24 times
# a few hundred roundings stays below 1e-4 of the O(1) scores and cache values.
TOL = 1e-4

CASES = [
    # (history lens, candidate lens, d, H, L, F)
    ([0, 1, 15, 16, 17, 31, 32, 33, 63, 64], [1, 33, 16, 15, 17, 32, 5, 0, 31, 64], 128, 2, 2, 128),
    ([65, 127, 128, 129, 500], [48, 1, 16, 47, 90], 128, 2, 2, 128),
    ([0, 1, 63, 64, 65, 127, 128, 129, 300], [3, 33, 16, 15, 17, 32, 5, 0, 70], 128, 4, 2, 128),
]


@pytest.mark.parametrize("variant", ["perturbed", "sharp"])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_edges_match_oracle(case, variant):
    n, k, d, H, L, F = CASES[case]
    inp = make_inputs(n, k, d, H, L, F, dtype="f32", seed=800 + case, variant=variant)
    say(f"[gpu] f32 attention case {case}/{variant}: d={d} H={H} histories {n} candidates {k}")
    run = GpuRun(inp)
    run.encode()
    run.rank()
    ref_cache = oracle.encode(inp.weights, d, H, L, F, inp.hist_emb, inp.hist_offsets)
    err = np.abs(run.cache_np() - ref_cache)
    assert err.max() <= TOL * (1 + np.abs(ref_cache).max()), f"cache: {err.max():.3e}"
    ref = oracle.rank(inp.weights, d, H, L, F, ref_cache, inp.hist_offsets, inp.cand_emb, inp.cand_offsets)
    e = np.abs(run.scores_np() - ref)
    assert e.max() <= TOL * (1 + np.abs(ref).max()), f"scores: {e.max():.3e}"
    say(f"[gpu] f32 attention case {case}/{variant}: cache {err.max():.2e}, scores {e.max():.2e}")


# (history lens, candidate lens, d, H, L, F, most): relative error (2-norm, mean of
# four seeds) of the scores against the float64 oracle, at most what one wave
# per row and FMA projections in sequence, the kernels these models once ran
# on, left on the same inputs (their own roundings, not a bound on any)
@pytest.mark.parametrize("n,k,d,H,L,F,most", [([1957], [74], 64, 1, 2, 256, 3.66e-7),
                                              ([400, 300], [300, 500], 256, 4, 2, 1024, 1.00e-6),
                                              ([64], [128], 64, 2, 1, 256, 4.61e-7)])
def test_error_against_64_bits(n, k, d, H, L, F, most):
    errors = []
    for seed in range(840, 844):
        inp = make_inputs(n, k, d, H, L, F, dtype="f32", seed=seed, variant="perturbed")
        run = GpuRun(inp)
        run.encode()
        run.rank()
        ref = oracle.rank(inp.weights, d, H, L, F, run.cache_np(), inp.hist_offsets, inp.cand_emb, inp.cand_offsets)
        errors.append(np.linalg.norm(run.scores_np() - ref) / np.linalg.norm(ref))
    say(f"[gpu] f32 error d={d} n={n}: {np.mean(errors):.3e} ({', '.join(f'{e:.2e}' for e in errors)})")
    assert np.mean(errors) <= most


@pytest.mark.parametrize("dt,H", [("f32", 2), ("f32", 4), ("bf16", 4)])
def test_workspace_without_room_for_the_list(dt, H):
    """A workspace a few bytes short of the reported size, as one sized before
    these models had a work list: encode and rank still run and agree."""
    import torch
    d, L, F = 128, 2, 256
    inp = make_inputs([70, 0, 129], [130, 5, 64], d, H, L, F, dtype=dt, seed=820, variant="perturbed")
    run = GpuRun(inp)
    run.encode()
    run.rank()
    want, want_cache = run.scores_np().copy(), run.cache_np().copy()
    hs, cs = upr.segments(run.hoff, run.hoff_d), upr.segments(run.coff, run.coff_d)
    need = upr.upr_rank_workspace_bytes(run.model.handle, hs, cs)
    enc = upr.upr_encode_workspace_bytes(run.model.handle, hs)
    run.cache.zero_()
    run.scores.fill_(float("nan"))
    run.model.encode(run.X, run.hoff, run.hoff_d, run.cache,
                     ws=torch.empty(enc - 1, dtype=torch.uint8, device="cuda"))
    run.model.rank(run.cache, run.hoff, run.hoff_d, run.C, run.coff, run.coff_d, run.scores,
                   ws=torch.empty(need - 1, dtype=torch.uint8, device="cuda"))
    tol = 1e-4 if dt == "f32" else 2e-2
    assert np.abs(run.cache_np() - want_cache).max() <= tol * (1 + np.abs(want_cache).max())
    assert np.abs(run.scores_np() - want).max() <= tol * (1 + np.abs(want).max())
    rows = int(run.coff[-1])
    short = 4 * d * rows                    # less than the residual stream alone: still refused
    with pytest.raises(upr.UprError):
        run.model.rank(run.cache, run.hoff, run.hoff_d, run.C, run.coff, run.coff_d, run.scores,
                       ws=torch.empty(short, dtype=torch.uint8, device="cuda"))


@pytest.mark.parametrize("dt,H", [("f32", 2), ("f32", 4), ("bf16", 4)])
def test_cache_off_the_16_byte_boundaries(dt, H):
    """A cache 4 bytes past a 16-byte boundary runs on the kernels that read
    single values, in encode and in ranking: the bits of a call whose workspace
    has no room for the work list."""
    import torch
    d, L, F = 128, 2, 256
    inp = make_inputs([70, 0, 129], [130, 5, 64], d, H, L, F, dtype=dt, seed=821, variant="perturbed")
    run = GpuRun(inp)
    hs, cs = upr.segments(run.hoff, run.hoff_d), upr.segments(run.coff, run.coff_d)
    need = upr.upr_rank_workspace_bytes(run.model.handle, hs, cs)
    enc = upr.upr_encode_workspace_bytes(run.model.handle, hs)
    run.model.encode(run.X, run.hoff, run.hoff_d, run.cache, ws=run.model.workspace(enc - 1))
    run.model.rank(run.cache, run.hoff, run.hoff_d, run.C, run.coff, run.coff_d, run.scores,
                   ws=run.model.workspace(need - 1))
    want, want_cache = run.scores_np().copy(), run.cache_np().copy()
    assert np.all(np.isfinite(want))
    off = 1 if dt == "f32" else 2
    flat = torch.zeros(run.cache.numel() + 16, dtype=run.cache.dtype, device="cuda")
    run.cache = flat[off:off + run.cache.numel()].view(run.cache.shape)
    assert run.cache.data_ptr() % 16 == 4
    run.scores.fill_(float("nan"))
    run.encode()
    run.rank()
    assert np.array_equal(run.cache_np(), want_cache)
    assert np.array_equal(run.scores_np(), want)
    assert not flat[:off].any() and not flat[off + run.cache.numel():].any()
