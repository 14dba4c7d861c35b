"""The line bench.py prints by default: short enough to survive where only the end of the output is kept (host only)."""
import json

import bench


def test_the_headline_is_short_and_complete():
    shapes = {f"{i}->{i}": {"us": {"dd_fwd": 1.0 / 3}} for i in range(100)}
    out = {"metric": "m", "value": 106.93442591194133, "ms_per_step": 24.044363600000196, "steps": 20, "roofline": {"frac": 0.667},
           "breakdown": {"ms_per_step_by_entry_point": {"dd_fwd": 8.2}, "stack_shapes": shapes, "configs": {"vitl": [shapes] * 9},
                         "dense_stack_ms": {"fwd": 9.45, "fwd_dgrad_wgrad": 35.3, "solutions": shapes}}}
    line = bench.headline(out)
    assert len(json.dumps(line)) < 2000
    assert line["breakdown"] == {"ms_per_step_by_entry_point": {"dd_fwd": 8.2}, "dense_stack_ms": {"fwd": 9.45, "fwd_dgrad_wgrad": 35.3}}
    assert {k: v for k, v in line.items() if k != "breakdown"} == {k: v for k, v in out.items() if k != "breakdown"}
    assert len(out["breakdown"]["configs"]["vitl"]) == 9  # what was measured is untouched
