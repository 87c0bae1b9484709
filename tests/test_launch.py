"""What a call launches (larger tiles, items split along their spans) covers the same pairs as the
schedules of whole items: each visible (query, key) pair once, nothing else, in every head."""
import numpy as np
import pytest

import oracle
from paper_2606_13872_amd import sra
from sra_inputs import SampleGeom, box_token_mask, workload

SCHEDS = (sra.SCHED_FORWARD, sra.SCHED_BWD_DQ, sra.SCHED_BWD_DKDV)
TOKENS = tuple(int(v) for v in np.random.default_rng(3).random(4 * 130) >= 0.3)
GEOMS = {
    "one_item": [SampleGeom(1, 8, 8, 1, 8, 8)],
    "long_keys": [SampleGeom(2, 20, 20, 3, 13, 11)],
    "ragged": [SampleGeom(3, 17, 13, 5, 9, 7, group_frames=2, frame_valid=(1, 0, 1, 1, 1))],
    "window": [SampleGeom(6, 13, 17, 3, 11, 13, gen_window=1)],
    "tokens": [SampleGeom(2, 14, 15, 4, 10, 13, ref_token_valid=TOKENS)],
    "varlen": [SampleGeom(2, 15, 21, 3, 15, 21), SampleGeom(1, 31, 33, 0, 1, 1),
               SampleGeom(2, 9, 9, 4, 12, 12, ref_token_valid=box_token_mask(4, 12, 12, 5))],
    "many": [SampleGeom(4, 24, 24, 3, 24, 24)],
}


@pytest.mark.parametrize("heads,dim", [(1, 64), (1, 128), (3, 128), (8, 64)])
@pytest.mark.parametrize("name", list(GEOMS))
@pytest.mark.parametrize("which", SCHEDS)
def test_launches_cover_the_mask(name, which, heads, dim):
    samples = GEOMS[name]
    for b, s in enumerate(samples):
        want = oracle.visibility_mask(s).astype(np.uint8)
        for h in {0, heads - 1}:
            got = sra.launch_mask(samples, which, b, h, heads=heads, head_dim=dim)
            assert np.array_equal(got, want), (b, h, np.argwhere(got != want)[:5])


@pytest.mark.parametrize("which", SCHEDS)
def test_gen_only_launches_cover_the_gen_rows(which):
    samples = GEOMS["long_keys"]
    want = oracle.visibility_mask(samples[0]).astype(np.uint8)
    want[samples[0].n_gen:] = 0
    got = sra.launch_mask(samples, which, 0, 0, heads=2, flags=sra.FLAG_GEN_QUERIES_ONLY)
    assert np.array_equal(got, want)


def test_the_rules_choose_both_ways():
    """Few long items are split, one round of short ones and long launches are not; long launches
    take the forward's large tile."""
    info = lambda s, h, d: sra.launch_info(s, sra.SCHED_FORWARD, heads=h, head_dim=d)
    n, tile, split = info(GEOMS["long_keys"], 3, 128)
    assert tile == 256 and split > 0 and n > split
    assert info(GEOMS["one_item"], 1, 64)[2] == 0
    for d, large in ((64, 512), (128, 384)):
        n, tile, split = info(workload("480p").samples, 40, d)
        assert tile == large and split == 0


@pytest.mark.parametrize("heads,dim", [(1, 64), (3, 128), (5, 128), (12, 128), (24, 128)])
def test_partial_results_leave_the_allocation_free_forward_its_calls(heads, dim):
    """Splitting may not take a call past the static scratch that whole items leave it under."""
    for samples in list(GEOMS.values()) + [workload("480p").samples, [SampleGeom(12, 33, 37, 9, 33, 37)]]:
        if any(s.ref_token_valid is not None for s in samples):
            continue
        assert sra.Problem(samples, heads, dim).workspace_size(False) <= sra.noalloc_workspace_max()
