"""The bench's multi-source byte lower bound for levels of the gather form,
counted by hand."""
import bench


def test_gather_levels():
    n, k = 1000, 64
    recs = [
        {"width": 64, "queue": 9, "queue_slices": 90, "new_pairs": 640, "gather": 1},
        {"width": 64, "queue": 2, "queue_slices": 10, "new_pairs": 40, "gather": 0},
    ]
    levels = 2 * k * n                        # one int16 per (source, vertex)
    gather = 125 + 8 * n                      # front bits; 8 B of visited words per vertex
    gather += 640 // 8 + 3 * 640 // 8 + 640 // 8  # frontier words read; three words and a plane written
    gather += 4 * 10                          # at least ten vertices, a column each
    queue = (4 + 1) * 10 + 8 * 8 * 2 + 40 // 8 + 3 * 40 // 8 + 2 * 40
    assert bench.ms_algorithmic_bytes(recs, n, 125, 8, 4, k) == levels + gather + queue
