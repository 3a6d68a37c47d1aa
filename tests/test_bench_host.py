"""What bench.py reports beside its measurements, without a GPU."""
import os

import bench

ROOT = os.path.dirname(os.path.abspath(bench.__file__))


def test_counted_traffic_goes_with_the_launch_that_was_counted():
    """A launch that merges its key ranges inside moves the partials twice: it never gets the bytes of one that leaves them to a
    second launch (nor the other way round), and a launch that was not counted gets none.  The bytes are the profile's."""
    from paper_2602_21780_amd.inputs import CONFIGS
    spec = CONFIGS[2]
    algorithmic = bench.algorithmic_work(spec, 4096, 4096, 2722)["attend_bytes"]
    partials = 5 * spec.n_heads * spec.tokens_per_frame * 144
    outputs = 2 * spec.tokens_per_frame * spec.n_heads * spec.head_dim
    second, inside = (bench.traffic_from_profile(240, m, algorithmic) for m in (False, True))
    assert abs(second["write_bytes"] - partials) < 0.05 * partials
    assert abs(inside["write_bytes"] - partials - outputs) < 0.05 * partials
    assert abs(inside["fetch_bytes"] - second["fetch_bytes"] - partials) < 0.1 * partials
    assert bench.traffic_from_profile(224, True, algorithmic) is None
    for t in (second, inside):
        assert t["ratio_to_algorithmic"] == round((t["fetch_bytes"] + t["write_bytes"]) / algorithmic, 2)
        text = open(os.path.join(ROOT, t["file"])).read()
        for x in ("fetch_bytes", "write_bytes"):
            assert f"{t[x] / 1e6:.1f} MB" in text
