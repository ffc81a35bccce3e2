"""The training line's peak rate: a mixture of products that cost six bf16 products and products that cost three."""
import dataclasses

import bench
from paper_2404_18911_amd import inputs as I


def test_peak_of_a_training_step_weighs_both_kinds_of_products():
    s = I.SHAPES["7b"]
    T, d, V = 256, s.d_model, s.vocab
    head, rest = 2.0 * T * 3 * V * d, 2.0 * T * 12 * d * d
    seconds = head / (2500.0 / 3) + rest / (2500.0 / 6)
    assert abs(bench.training_peak_tflops(s, T, head + rest) - (head + rest) / seconds) < 1e-9
    assert 600 < bench.training_peak_tflops(s, T, head + rest) < 640
    # the head alone, nothing against tiles, and one of three head products against tiles
    assert abs(bench.training_peak_tflops(s, T, head) - 2500.0 / 3) < 1e-9
    f32 = dataclasses.replace(s, dtype="f32")
    assert abs(bench.training_peak_tflops(f32, T, head + rest) - 2500.0 / 6) < 1e-9
    own = dataclasses.replace(s, adapter=I.ADAPTER_MLP)
    assert abs(bench.training_peak_tflops(own, T, head) - head / (head / 3 / (2500.0 / 3) + 2 * head / 3 / (2500.0 / 6))) < 1e-9
