"""GPU parity of the dW kernel's tile stream at the sizes where it can go wrong: the shortest contractions of each of
its store schedules (4, 6 and 10 k-steps of 64 rows), one more and one less, ragged row counts, feature tiles that
hang over the edge (D = 64, 320), ragged class edges, workgroups with one tile, with two, and with none."""
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


@pytest.mark.parametrize("B,D,C", [
    (192, 64, 300),                  # 3 k-steps: one short of a stream
    (193, 320, 700),                 # 4: two feature tiles, the second 64 wide
    (256, 64, 256 * 258 + 9),        # 4: 259 tiles, three workgroups with a second one
    (321, 128, 256 * 256),           # 6: exactly one tile each
    (384, 64, 256 * 257 - 250),      # 6: the last class tile 6 wide
    (577, 320, 256 * 140 + 1),       # 10: 282 tiles, ragged in rows, features and classes
    (639, 576, 256 * 100 - 7),       # 10: three feature tiles, the last 64 wide
    (1025, 64, 40),                  # 17: a single ragged tile
])
def test_dw_stream_schedules_and_edges(H, B, D, C):
    p = inputs.make_inputs("stream", B, D, C, x_sigma=1.0, w_sigma=0.3, bias_sigma=1.0, seed=B + C)
    shape = f"B={B} D={D} C={C}"
    H.say(f"[parity] dW stream: {shape}")
    got = H.run_step(p.X_bits, p.W_bits, p.bias, p.labels, [(0, C)], g=1.0 / B)
    ref = H.oracle_step(p.X_bits, p.W_bits, p.bias, p.labels, [(0, C)], g=1.0 / B)
    rep = H.compare(got, ref, p.labels, [(0, C)], shape, gate="fp32_floor")
    H.record(f"dW stream {shape}", f"{shape} gate=fp32_floor", rep)


def test_dw_stream_with_prefetch(H):
    """dz and W together beyond 256 MiB, a contraction of 7 k-steps: the stream that touches dz lines ahead (the
    full-size workloads run it with 4 and 16 k-steps)."""
    B, D, C = 400, 2048, 60_001
    p = inputs.make_inputs("prefetch", B, D, C, x_relu=True, w_sigma=0.01, seed=6)
    H.say(f"[parity] dW stream with prefetch: B={B} D={D} C={C}")
    got = H.run_step(p.X_bits, p.W_bits, None, p.labels, [(0, C)], g=1.0)
    ref = H.oracle_step(p.X_bits, p.W_bits, None, p.labels, [(0, C)], g=1.0)
    rep = H.compare(got, ref, p.labels, [(0, C)], "prefetch", gate="fp32_floor")
    H.record("dW stream with prefetch", f"B={B} D={D} C={C} gate=fp32_floor", rep)
