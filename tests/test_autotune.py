"""The tuner's records (tile_cache.json) are shapes that it tries itself, with times that it measured:
running it again can find them."""
from paper_1405_3331_amd import autotune


def test_records_are_candidates():
    cache = autotune.load_cache()
    assert cache
    for name, r in cache.items():
        tried = (autotune.default_batch_candidates() if name.startswith("batch:")
                 else autotune.default_candidates())
        shape = (r["block_steps"], r["cols_per_lane"], r["height"])
        # a height of 0 is recorded as the planner's own, which is one more than those listed
        listed = {c[:2] for c in tried if c[2] == 0}
        assert shape in tried or shape[:2] in listed, (name, shape)
        us = r["seconds_per_step"] * 1e6
        assert us > 0 and abs(us * 100 - round(us * 100)) > 1e-9, (name, us)   # as measured
