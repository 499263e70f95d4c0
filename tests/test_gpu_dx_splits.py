"""GPU parity of dX where its contraction is cut: wide tiles whose number does not divide 256 (20, 44, 72 of them), last splits
shorter than the others (test_plan.py checks that they are), one split written straight to the output and one that is added to it; the 64 x 64 tiles with one
row, one tile, ragged rows and classes, and more than 256 workgroups."""
import pytest

from paper_2011_09208_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU; there is no CPU fallback")
    from tests import gpu_harness
    return gpu_harness


SHAPES = [                               # B, D, widths
    (1100, 1024, [64 * 141 - 5]),        # 20 wide tiles, 141 k-steps: 9 splits of 16, the last of 13
    (2600, 1024, [64 * 30 + 7]),         # 656 small tiles, one split
    (2600, 1024, [64 * 60 + 7]),         # 44 wide ones: 4 splits of 16, the last of 13
    (2300, 2048, [64 * 40 - 3]),         # 72: 2 splits
    (1000, 2048, [5000]),                # 32: 5 splits of 16, the last of 15
    (1, 64, [1, 40]),                    # one small tile
    (64, 64, [64 * 70 + 1]),             # 1: 18 splits of 4 k-steps, the last of 3
    (65, 128, [64 * 200]),               # 4, one row in the second: 29 splits of 7, the last of 4
    (130, 64, [2561]),                   # 3: 14 splits of 3, the last of 2
    (700, 192, [64 * 21]),               # 33
    (2300, 576, [64 * 19 + 1]),          # 324, in one launch with dW
    (1500, 832, [64 * 40 + 3]),          # 312: 2 splits of 21, the last of 20
    (1100, 1024, [64 * 3, 64 * 2 + 9]),  # 288: one split, the second shard added to the first
    (4500, 64, [130]),                   # 71, 3 k-steps
    (300, 128, [500, 130]),              # in one launch with dW, the second shard added to the first
    (90, 320, [64 * 16, 64 * 16 + 1]),   # 16 and 17 k-steps in one launch with dW
    (90, 320, [64 * 20 + 1]),            # 21 in splits of their own: 7 of 3
]


@pytest.mark.parametrize("B,D,widths", SHAPES)
def test_dx_splits(H, B, D, widths):
    C = sum(widths)
    shards = [(sum(widths[:i]), w) for i, w in enumerate(widths)]
    p = inputs.make_inputs("dx-splits", B, D, C, x_sigma=1.0, w_sigma=0.3, bias_sigma=1.0, seed=B + C)
    shape = f"B={B} D={D} widths={widths}"
    H.say(f"[parity] dX splits: {shape}")
    got = H.run_step(p.X_bits, p.W_bits, p.bias, p.labels, shards, g=1.0 / B)
    ref = H.oracle_step(p.X_bits, p.W_bits, p.bias, p.labels, shards, g=1.0 / B)
    rep = H.compare(got, ref, p.labels, shards, shape, gate="fp32_floor")
    H.record(f"dX splits {shape}", f"{shape} gate=fp32_floor", rep)
