"""The figures of the benchmark's line that come from statistics (no GPU)."""
import bench


def stats(variant, rounds, counted):
    n = [1000 >> r for r in range(rounds)]
    z = [100 * x for x in n] if counted else [0] * rounds
    return dict(traversal_variant=variant, rounds=rounds, components=n, queries_round=[1000] * rounds,
                child_tests_round=z, leaf_tests_round=z, records_touched_round=z, child_tests=sum(z),
                leaf_tests=sum(z), dist_evals=sum(z))


def test_a_run_without_a_tree_reports_no_counts_of_a_traversal():
    timed, counted = stats(-1, 5, False), stats(13, 6, True)
    rounds, roof, table = bench.traversal_report("uniform2d_10k", 2, timed, counted, 1.0, 10, [0.1] * 5)
    assert rounds == 5 and len(table) == 5 and roof["launches_per_step"] == 5
    assert roof["kernel"] == "k_flat_search" and roof["avg_launch_ms"] == 0.1
    for key in ("achieved", "frac", "traffic", "traffic_frac"):
        assert roof[key] is None
    for key in ("logical", "records_touched_per_launch", "children_examined_per_query_round", "algorithmic_bytes"):
        assert key not in roof
    assert all(row["child_tests_per_query"] is None and row["records_loaded"] is None for row in table)
    assert [row["components"] for row in table] == timed["components"]


def test_a_run_with_a_tree_reports_the_counting_runs():
    timed, counted = stats(13, 6, False), stats(13, 6, True)
    rounds, roof, table = bench.traversal_report(None, 3, timed, counted, 6.0, 6, [1.0] * 6)
    assert rounds == 6 and roof["kernel"] == "k_traverse_fast" and roof["traffic"] is None
    touched = counted["records_touched_round"]
    unique = sum(64 * t + 28 * 1000 for t in touched) / 6
    assert roof["algorithmic_bytes_per_launch"] == int(unique)
    assert roof["achieved"] == round(unique / 1e-3 / 1e9, 1)
    assert [row["records_loaded"] for row in table] == touched
