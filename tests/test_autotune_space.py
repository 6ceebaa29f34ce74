"""The shapes that the autotuner times (no GPU needed)."""
from paper_2511_16576_amd import autotune


def test_no_shape_twice():
    """blocks_per_cu is tried only where a launch depends on it."""
    s = autotune.DEFAULT_SPACE
    plain = len(s["persistent"]) * len(s["block_threads"]) * len(s["hash_block"]) * len(s["lds_edges"]) \
        * len(s["samples_per_lane"])
    tried = list(autotune.shapes(s, 20_000, 128))
    assert len(tried) == plain and len({tuple({**c, "blocks_per_cu": 0}.values()) for c in tried}) == plain


def test_queued_shapes_by_blocks():
    s = {"persistent": [1, 0], "block_threads": [512], "hash_block": [0, 1], "lds_edges": [256],
         "samples_per_lane": [1], "blocks_per_cu": [8, 16]}
    tried = list(autotune.shapes(s, 20_000, 1000))          # 20 M items of one hash
    assert len(tried) == 5 and [c for c in tried if c["blocks_per_cu"] == 16] == [
        {"persistent": 1, "block_threads": 512, "hash_block": 1, "lds_edges": 256, "samples_per_lane": 1,
         "blocks_per_cu": 16}]
