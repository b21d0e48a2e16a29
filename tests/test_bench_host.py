"""bench.py on the CPU: the timing loop and the lookup of the committed traffic counters."""
import time

import pytest
import torch

import bench


def test_short_repeats_are_timed_again_with_more_blocks(monkeypatch):
    monkeypatch.setattr(torch.cuda, "synchronize", lambda: None)
    blocks, times = bench.timed_repeats(lambda: time.sleep(1e-4), 1, 3, 2.0)
    assert blocks > 1 and len(times) == 3 and min(times) >= 2e-3


@pytest.mark.parametrize("kernel", ["stack_product_kernel", "fused_kernel"])
def test_traffic_counters_scale_with_the_layers_of_a_launch(kernel):
    one = bench.measured_traffic("phi3-medium-mlp-stack-bf16", 0.3, kernel, 1)
    algorithmic = 2 * 1536 * 17920 * 2
    assert algorithmic <= one <= 1.05 * algorithmic
    assert bench.measured_traffic("phi3-medium-mlp-stack-bf16", 0.3, kernel, 40) == 40 * one
    assert bench.measured_traffic("phi3-medium-mlp-stack-bf16", 0.5, kernel, 1) is None
