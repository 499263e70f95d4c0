"""GPU parity of dX where its contraction is cut so that the workgroups fit one round of the 256 compute units: tile counts
that do not divide 256 (20, 27, 72, 132 tiles), more splits than k-steps, last splits shorter than the others, one split
written straight to the output and one that is added to it."""
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


@pytest.mark.parametrize("B,D,widths", [
    (1100, 1024, [64 * 141 - 5]),        # 20 tiles, 141 k-steps: 12 splits of 12, the last of 9
    (1100, 1024, [64 * 3]),         # 3 k-steps: as many splits
    (2300, 576, [64 * 19 + 1]),          # 27 tiles, 20 k-steps: 7 splits of 3, the last of 2
    (2100, 1984, [64 * 10]),             # 72 tiles: 2 splits
    (2700, 2880, [300, 64 * 7 + 9]),     # 132 tiles: one split, the second shard added to the first
])
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
