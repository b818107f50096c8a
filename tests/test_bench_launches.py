"""What the benchmark makes of the step's operations (CPU): launches, their peaks, and the time taken off for events."""
import numpy as np

import bench

OPS = [("conv1", 12), ("conv2", 26), ("conv3", 5), ("heads", 1)]
PIPES = ["i8x3", "f16x2", "f16x2", "bf16x3"]


def test_two_layers_in_one_launch():
    runs = bench.launches(OPS, PIPES, ["conv12_split", "conv12_split", "conv_image_split", "heads"])
    assert [r["name"] for r in runs] == ["conv1+conv2", "conv3", "heads"]
    assert [r["flops"] for r in runs] == [38, 5, 1] and runs[0]["pipe"] == "i8x3+f16x2"
    assert [r["index"] for r in runs] == [[0, 1], [2], [3]]
    # at its peak the launch takes what the two layers take at theirs
    assert np.isclose(38 / runs[0]["peak"], 12 / bench.PEAK_TOPS["i8x3"] + 26 / bench.PEAK_TOPS["f16x2"])
    assert runs[1]["peak"] == bench.PEAK_TOPS["f16x2"]


def test_every_operation_a_launch():
    kernels = ["conv1_i8", "conv_image_split", "conv_image_split", "heads"]
    runs = bench.launches(OPS, PIPES, kernels)
    assert [(r["name"], r["flops"]) for r in runs] == OPS and [r["kernel"] for r in runs] == kernels
    assert [r["peak"] for r in runs] == [bench.PEAK_TOPS[p] for p in PIPES]
    assert all(r["index"] == [i] for i, r in enumerate(runs))


def test_cost_of_an_event():
    event_ms = np.array([0.040, 0.019, 0.008])
    ms, cost = bench.launch_times(event_ms, 0.061)
    assert np.isclose(cost, 0.002) and np.isclose(ms.sum(), 0.061)
    assert bench.launch_times(event_ms, 0.1)[1] == 0.0
    assert np.isclose(bench.launch_times(event_ms, 0.001)[1], 0.004)  # (at most half of the shortest)
