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


PARTIAL_BYTES = 256 << 20  # a backward's partial results
LONG_GROUPS = {
    "1x24x24|9x52x30": ([SampleGeom(1, 24, 24, 9, 52, 30, group_frames=9)], 1),
    "1x16x16|4x60x60": ([SampleGeom(1, 16, 16, 4, 60, 60, group_frames=4)], 2),
    "4x17x1|16x60x49": ([SampleGeom(4, 17, 1, 16, 60, 49, group_frames=8)], 1),
    "two": ([SampleGeom(1, 13, 21, 19, 23, 7, group_frames=9), SampleGeom(1, 5, 37, 21, 54, 51, group_frames=12)], 1),
    "1x8x8|9x45x80": ([SampleGeom(1, 8, 8, 9, 45, 80, group_frames=9)], 1),
    "mixed": ([SampleGeom(1, 8, 8, 9, 30, 52, group_frames=9), SampleGeom(5, 30, 52, 9, 30, 52, group_frames=9)], 1),
}


def _random_long_group(rng):
    def sample():
        rf = int(rng.integers(1, 22))
        return SampleGeom(int(rng.integers(1, 5)), int(rng.integers(1, 25)), int(rng.integers(1, 25)), rf,
                          int(rng.integers(1, 61)), int(rng.integers(1, 61)), group_frames=int(rng.integers(1, rf + 1)))
    return [sample() for _ in range(int(rng.integers(1, 4)))]


def test_backward_partial_results_stay_within_their_bound():
    """Few gen rows and groups as long as the clip: the pieces of a key tile's gen and reference queries
    are counted as they are cut. Beside the partial results the workspace holds the tables (under
    4 MiB here) and two values per row and head."""
    rng = np.random.default_rng(17)
    calls = list(LONG_GROUPS.values()) + [(_random_long_group(rng), int(rng.integers(1, 4))) for _ in range(300)]
    split = 0
    for samples, heads in calls:
        for flags in (0, sra.FLAG_GEN_QUERIES_ONLY):
            rows = sum(s.n_gen + s.n_ref for s in samples)
            need = sra.Problem(samples, heads, 128, flags=flags).workspace_size(True)
            assert need <= PARTIAL_BYTES + (4 << 20) + 8 * heads * rows, (samples, heads, flags)
        split += sra.launch_info(samples, sra.SCHED_BWD_DKDV, heads=heads)[2] > 0
    assert split >= 100  # the calls are ones that are split


@pytest.mark.parametrize("flags", [0, sra.FLAG_GEN_QUERIES_ONLY])
@pytest.mark.parametrize("gen,ref", [((1, 8, 8), (4, 16, 33)), ((1, 3, 11), (6, 11, 17)), ((2, 9, 13), (3, 29, 21))])
def test_few_gen_rows_and_long_groups_launch_no_empty_pieces(gen, ref, flags):
    """The expansion refuses an item without spans, so each piece has some; and covers the mask."""
    samples = [SampleGeom(*gen, *ref, group_frames=ref[0])]
    want = oracle.visibility_mask(samples[0]).astype(np.uint8)
    if flags:
        want[samples[0].n_gen:] = 0
    for which in SCHEDS:
        got = sra.launch_mask(samples, which, 0, 0, heads=1, flags=flags)
        assert np.array_equal(got, want), which
    assert sra.launch_info(samples, sra.SCHED_BWD_DKDV, heads=1)[2] > 0


@pytest.mark.parametrize("name,heads", [("long_keys", 3), ("varlen", 3), ("one_item", 1)])
def test_the_hooks_show_the_tables_of_a_joint_gradient_launch(name, heads):
    """dQ and dK/dV items of one launch share its span table; the slots of each kind's pieces are
    0 .. n - 1, each once."""
    tables = [sra.launch_export(GEOMS[name], which, heads=heads) for which in SCHEDS[1:]]
    assert np.array_equal(tables[0][1], tables[1][1])
    for (items, spans), which in zip(tables, SCHEDS[1:]):
        n, _, split = sra.launch_info(GEOMS[name], which, heads=heads)
        assert len(items) == n and set(items[:, 0]) <= {0, 1}
        assert np.all(items[:, 5] > 0) and np.all(items[:, 4] + items[:, 5] <= len(spans))
        slots = np.sort(items[items[:, 7] > 0, 7])
        assert np.array_equal(slots, np.arange(1, len(slots) + 1)) and (len(slots) > 0) == (split > 0)


def _gen_work(samples, which, heads, dim, flags):
    """(head, start, length) of gen query items and pieces -> their spans, and the split items' pieces
    in order (slots are numbered per launch)."""
    items, spans = sra.launch_export(samples, which, heads=heads, head_dim=dim, flags=flags)
    out = {}
    for it in items[np.argsort(items[:, 7], kind="stable")]:
        if it[0] == 0:
            out.setdefault(tuple(it[1:4]), []).append(spans[it[4]:it[4] + it[5]].tolist())
    return out


def _random_batch(rng):
    samples = []
    for _ in range(int(rng.integers(1, 4))):
        rf = int(rng.integers(0, 13))
        n = int(rng.integers(4, 60)), int(rng.integers(4, 60))
        tok = None
        if rf and rng.random() < 0.2:
            tok = box_token_mask(rf, *n, int(rng.integers(99)))
        samples.append(SampleGeom(int(rng.integers(1, 7)), *(n if rng.random() < 0.5 else n[::-1]), rf, *n,
                                  group_frames=int(rng.integers(1, rf + 2)), ref_token_valid=tok))
    return samples


def test_gen_only_launches_run_the_gen_rows_as_the_call_of_all_rows():
    """Cached reference K/V: the gen rows' sums run over the same spans in the same order whether or not
    the reference rows are queries too, so their results are the same bits."""
    rng = np.random.default_rng(23)
    calls = [([SampleGeom(6, 33, 54, 9, 33, 54, group_frames=18)], 16, 64),
             ([SampleGeom(1, 16, 16, 12, 40, 40, group_frames=12), SampleGeom(4, 40, 40, 2, 40, 40)], 16, 128)]
    calls += [(_random_batch(rng), int(rng.choice([3, 8, 16, 24])), int(rng.choice([64, 128]))) for _ in range(120)]
    split = 0
    for samples, heads, dim in calls:
        for which in SCHEDS[:2]:
            full = _gen_work(samples, which, heads, dim, 0)
            gen = _gen_work(samples, which, heads, dim, sra.FLAG_GEN_QUERIES_ONLY)
            assert gen == full, (samples, heads, dim, which)
            split += any(len(v) > 1 for v in gen.values())
    assert 20 < split < 200  # both kinds


@pytest.mark.parametrize("flags", [sra.FLAG_GEN_WINDOW, sra.FLAG_GEN_WINDOW | sra.FLAG_GEN_QUERIES_ONLY])
@pytest.mark.parametrize("gen_frames,ref_frames", [(300, 2400), (280, 3000), (300, 3400), (330, 2800), (100, 3800)])
def test_long_span_lists_leave_the_allocation_free_forward_its_calls(gen_frames, ref_frames, flags):
    """Window tiles that each list a thousand and more one-token runs: 3 to 8 MB of tables, beside which the
    partial results have to fit."""
    valid = tuple(int(i % 2 == 0) for i in range(ref_frames))
    samples = [SampleGeom(gen_frames, 1, 2, ref_frames, 1, 1, frame_valid=valid, gen_window=0)]
    assert sra.Problem(samples, 1, 128, flags=flags).workspace_size(False) <= sra.noalloc_workspace_max()


@pytest.mark.parametrize("which", SCHEDS)
def test_launched_phases_cut_spans_at_tile_ends(which):
    """Long launches with heads pinned to XCDs start a gen span part way in: at a whole number of the
    kernels' 64-row tiles, since a part that ends elsewhere costs a ragged tile of its own."""
    samples = [SampleGeom(11, 35, 41, 5, 35, 41)]
    items, spans = sra.launch_export(samples, which, heads=24)
    first = spans[np.unique(items[items[:, 0] >= 0, 4])]
    assert np.all(first[first[:, 0] == 0, 1] % 64 == 0)
    assert (first[first[:, 0] == 0, 1] > 0).sum() >= 3


@pytest.mark.parametrize("dim,rows,whole,split", [(64, 64, 24, 25), (64, 129, 16, 17), (128, 128, 13, 14), (128, 129, 8, 9)])
def test_short_forwards_stay_whole(dim, rows, whole, split):
    """A launch that ends within the host's part of a call is not split; items of up to 128 rows take 0.7
    of the time."""
    def info(steps):
        g = SampleGeom(1, 1, rows, steps - (rows + 63) // 64, 8, 8)
        return sra.launch_info([g], sra.SCHED_FORWARD, heads=2, head_dim=dim)
    assert info(whole)[2] == 0
    assert info(split)[2] > 0


def test_kinds_of_gradient_items_divide_evenly():
    """dQ items of 26 steps, dK/dV items of 13 (gen keys) and 21: no piece length that is a whole part of
    the longest item's cuts these into pieces of 13, 6.5 and 7, one round of the compute units."""
    g = [SampleGeom(11, 8, 9, 11, 8, 9, group_frames=3)]
    items, spans = sra.launch_export(g, sra.SCHED_BWD_DKDV, heads=8, head_dim=64)
    steps = [int((-(-spans[i[4]:i[4] + i[5], 2] // 64)).sum()) for i in items]
    assert max(steps) <= 8
    assert len(items) + sra.launch_info(g, sra.SCHED_BWD_DQ, heads=8, head_dim=64)[0] <= 256
