"""GPU parity of the dW kernel at the sizes where its tile stream can go wrong: the shortest contractions of each of
its store schedules (4, 6 and 10 k-steps of 64 rows), ragged row counts, feature tiles that hang over the edge (D = 320,
576), ragged class edges, workgroups with two tiles, with one and with none; and at the sizes next to them that take one
workgroup per tile (three k-steps, one feature tile, up to 256 tiles)."""
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
    (192, 320, 256 * 128 + 1),       # 3: 258 tiles
    (193, 320, 700),                 # 4: two feature tiles, the second 64 wide; six tiles
    (193, 320, 256 * 128),           # 4: 256 tiles, one short of a stream
    (193, 320, 256 * 128 + 1),       # 4: 258 tiles, two workgroups with a second one
    (256, 64, 256 * 258 + 9),        # 4: 259 tiles of one feature tile
    (256, 576, 256 * 91 - 3),        # 4: 273 tiles, three feature tiles; 35 to an XCD, 28 on the last: workgroups with none
    (321, 128, 256 * 256),           # 6: exactly one tile each
    (321, 320, 256 * 130 - 250),     # 6: 260 tiles, the last class tile 6 wide
    (384, 64, 256 * 257 - 250),      # 6: the same with one feature tile
    (576, 320, 256 * 129),           # 9: the longest of its schedule
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
