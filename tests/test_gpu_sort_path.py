"""The sorting pipeline on race checks, plain and warp-aware: the parity tests of
these calls once more, on contexts whose every size class has a launch shape, so
that nothing is counted by group.  The stage times of each call say that it
sorted.  (Barrier and fitness checks, traces of more than 2^27 records, the
no-allocation call and every call that the grouped count does not hold take the
same pipeline.)"""
import pytest

import test_gpu_filter
import test_gpu_parity
import test_gpu_warp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture()
def sorting(monkeypatch):
    """pkg.Context, with a shape for every size class; yields one of them."""
    import paper_1905_01833_amd as pkg

    class Sorting(pkg.Context):
        def __init__(self, device=0, **kw):
            if not kw.get("graphs"):
                kw["profile"] = True
            super().__init__(device, **kw)
            self.sorted = 0
            for k in range(pkg.SIM_SIZE_CLASSES):
                self.set_tuning(k, {"scatter_threads": 512 if k % 2 else 256})

        def _looked(self, got):
            t = self.stage_times()
            assert t["filter_count"][1] == 0
            self.sorted += t["keygen"][1] > 0
            return got

        def check_traces(self, *a, **kw):
            return self._looked(super().check_traces(*a, **kw))

        def check_traces_device(self, *a, **kw):
            return self._looked(super().check_traces_device(*a, **kw))

        def check_traces_warp_device(self, *a, **kw):
            return self._looked(super().check_traces_warp_device(*a, **kw))

    monkeypatch.setattr(pkg, "Context", Sorting)
    c = Sorting(0)
    yield c
    c.close()


P, W, F = test_gpu_parity, test_gpu_warp, test_gpu_filter


RUNS = {
    "c0": lambda c: P.test_c0_tree_reduction(c),
    "tree family": lambda c: P.test_tree_family_batched(c),
    "truth table": lambda c: P.test_truth_table_batched(c),
    "tiny batch": lambda c: P.test_random_tiny_batch(c),
    "tile boundaries": lambda c: [P.test_tile_boundaries(c, n) for n in (4095, 4096, 4097, 12411, 45055)],
    "host records": lambda c: P.test_host_entry_point(c),
    "one location": lambda c: P.test_mega_location(c),
    "uniform groups": lambda c: P.test_uniform_groups(c),
    "output grows": lambda c: P.test_many_racing_locations_grow_output(c),
    "location lengths": lambda c: P.test_location_lengths_across_threads(c),
    "mixed sizes": lambda c: P.test_batched_mixed_sizes(c),
    "permutation": lambda c: P.test_permutation_invariance(c),
    "errors": lambda c: P.test_error_paths_leave_context_usable(c),
    "2^24": lambda c: P.test_c1_full_size(c),
    "two-word keys": lambda c: P.test_two_word_keys(c),
    "warp patterns": lambda c: [W.test_hand_patterns(c, name) for name in sorted(W.hand_patterns())],
    "warp patterns batched": lambda c: W.test_hand_patterns_batched(c),
    "warp tiny batch": lambda c: [W.test_random_tiny_batch(c, seed) for seed in (1, 2)],
    "warp across tiles": lambda c: [W.test_generated_traces_across_tiles(c, n) for n in (1, 4, 32)],
    "warp two-word keys": lambda c: W.test_two_word_keys(c),
    "warp 2^24": lambda c: W.test_c1_full_size(c),
    "warp batch": lambda c: F.test_warp_aware(c),
    "block sizes": lambda c: [F.test_block_sizes(c, *s) for s in ((1, 4096), (32, 300), (96, 100), (1000, 17), (1 << 20, 5))],
    "empty traces": lambda c: [F.test_tile_edges_and_empty_traces(c, e) for e in (-1, 0, 1)],
    "contents": lambda c: [F.test_contents(c, f) for f in ("reads", "atomics", "private writes", "all race", "one word",
                                                           "wide units", "far units", "half race")],
    "hot words": lambda c: [F.test_hot_words(c, h) for h in ("read", "written", "many")],
    "recovery": lambda c: F.test_invalid_record_and_recovery(c),
}


@pytest.mark.parametrize("run", list(RUNS.values()), ids=list(RUNS))
def test_sorted(sorting, run):
    run(sorting)
    assert sorting.sorted


@pytest.mark.parametrize("run", [P.test_short_traces_sorted_in_lds, lambda: P.test_widest_keys_and_mixed_pass_counts(None),
                                 P.test_graph_replays_match_eager],
                         ids=["short", "widest", "replays"])
def test_sorted_on_contexts_of_their_own(sorting, run):
    """Tests that make their contexts themselves: what a context remembers from
    call to call (passes, key width), and replays."""
    run()

