"""The MXFP8 variant runs what follows the attention as one kernel in calls of
enough rows and as separate launches in smaller ones: the same candidates get
the same bits either way, whichever tile a row falls in (whole tiles keep the
residual in another order than the call's last, partial one), before the
score head and before action heads.  Nor does the height of a projection's
tile change a bit."""
import numpy as np
import pytest
import torch

from synth import make_heads, make_inputs

from .gpu_util import GpuRun, say

pytestmark = pytest.mark.gpu

# (d, H, L, F, rows): one, two and sixteen hidden chunks; 64-row and 128-row
# tiles, the last of 1, 63, 65 or 128 rows
CASES = [
    (512, 8, 2, 2048, 16384 + 1),
    (512, 8, 2, 128, 8192 + 64 + 63),
    (512, 8, 1, 256, 20000 // 128 * 128 + 65),
    (256, 4, 3, 1024, 16384 + 128),
    (256, 4, 1, 128, 1024 + 1),
    (512, 8, 1, 512, 4096 + 1),
    (256, 4, 2, 256, 33000),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_tail_gives_the_bits_of_the_separate_launches(case):
    d, H, L, F, top = CASES[case]
    inp = make_inputs([70], [top], d, H, L, F, dtype="bf16", seed=800 + case, variant="perturbed")
    run = GpuRun(inp, model_dtype="bf16_mxfp8")
    run.encode()
    say(f"[gpu] mx tail d={d} F={F}: {top} rows")
    run.rank()
    ref = run.scores_np().copy()
    assert np.all(np.isfinite(ref))
    for lo, hi in ((0, 200), (top // 2, min(top, top // 2 + 1000)), (top - 300, top)):
        say(f"[gpu] mx tail d={d} F={F}: rows {lo}..{hi}")
        run.scores.fill_(float("nan"))
        run.rank(coff=np.array([lo, hi], np.int32))
        assert np.array_equal(run.scores_np()[lo:hi], ref[lo:hi]), f"rows {lo}..{hi}"


def test_tail_before_action_heads():
    from tests.test_gpu_heads import _run_actions
    d, H, L, F, top, C, Fh = 256, 4, 2, 512, 16384 + 77, 3, 64
    inp = make_inputs([70], [top], d, H, L, F, dtype="bf16", seed=820, variant="perturbed")
    hb = make_heads(d, C, Fh, dtype="bf16", seed=821, variant="perturbed")
    uw = np.array([1.0, 0.5, -2.0], dtype=np.float32)
    run = GpuRun(inp, model_dtype="bf16_mxfp8")
    run.encode()
    say(f"[gpu] mx tail before heads: {top} rows")
    ref = np.asarray(_run_actions(run, hb, C, Fh, uw)[0]).copy()
    for lo, hi in ((0, 300), (top - 200, top)):
        run.coff = np.array([lo, hi], np.int32)
        run.coff_d = torch.from_numpy(run.coff).to("cuda")
        got = np.asarray(_run_actions(run, hb, C, Fh, uw)[0])
        assert np.array_equal(got[lo:hi], ref[lo:hi]), f"rows {lo}..{hi}"


def test_mx_tile_height_does_not_change_scores():
    """Projections on 256-column tiles of 64, 128, 192 or 256 rows by the size
    of the call (d = 768: no tail), last tiles partial: the same bits."""
    d, H, L, F, top = 768, 12, 1, 896, 33000
    inp = make_inputs([37], [top], d, H, L, F, dtype="bf16", seed=830, variant="perturbed")
    run = GpuRun(inp, model_dtype="bf16_mxfp8")
    run.encode()
    run.rank()
    ref = run.scores_np().copy()
    assert np.all(np.isfinite(ref))
    for lo, hi in ((5, 6), (63, 390), (100, 4100), (7, 6107), (1000, 13011), (11, 22000)):
        say(f"[gpu] mx tiles d={d} F={F}: rows {lo}..{hi}")
        run.scores.fill_(float("nan"))
        run.rank(coff=np.array([lo, hi], np.int32))
        assert np.array_equal(run.scores_np()[lo:hi], ref[lo:hi]), f"rows {lo}..{hi}"
