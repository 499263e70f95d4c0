"""GPU parity of the logits kernels that walk lists of tiles, at the sizes where the lists can go wrong: one, two and three
k-steps (loads run two k-steps ahead, over the edge of a tile), rests of one to four units of 32 classes, workgroups with and
without a rest, 1 to 9 and 129 batch tiles (blocks of four, and every remainder), ragged rows and classes, several
workgroups to a compute unit; and a forward call whose workspace holds no more than a partial result per class tile."""
import numpy as np
import pytest

from paper_2011_09208_amd import inputs

pytestmark = pytest.mark.gpu

SHAPES = [                               # B, D, C
    (70, 64, 256 * 65 - 40),             # 1 batch tile, 65 class tiles, 1 k-step; rests of 2 and 3 units; the forward call on tiles
    (257, 64, 256 * 33 - 7),             # 2; 66 tiles; the same
    (300, 128, 256 * 129),               # 2; a whole tile, 8 workgroups of 128 columns with a rest of one unit; the forward call on tiles
    (300, 128, 256 * 161),               # 2; a whole tile and rests of 2 and 3 units
    (513, 1088, 256 * 40),               # 3; 17 k-steps, rests of 3 and 4
    (600, 64, 256 * 170 + 33),           # 3; two whole tiles
    (700, 576, 256 * 86 + 65),           # 3; 9 k-steps, 261 tiles: wide ones, the last 5 as thin tiles
    (700, 576, 256 * 112 + 65),          # 3; 339 tiles: a whole one and rests of 2 and 3 units
    (600, 640, 256 * 170 + 33),          # 3; 513 tiles, 10 k-steps: lists
    (1000, 576, 256 * 136),              # 4; 544 and a tail of 32: lists
    (1000, 576, 256 * 137),              # 548, one of 36: tiles
    (1000, 192, 256 * 17 + 1),           # 4; 72 tiles, 3 k-steps
    (1100, 128, 256 * 21 + 1),           # 5: a block of four and one; the forward call on tiles
    (1400, 192, 256 * 13 - 100),         # 6
    (1700, 64, 2600),                    # 7; the forward call on tiles
    (2100, 64, 256 * 40 - 31),           # 9: two blocks and one
    (33000, 64, 500),                    # 129 batch tiles, 258 tiles: wide ones
    (70, 192, 256 * 65 - 40),            # forward and dz
    (1100, 192, 256 * 21 + 1),
    (1700, 192, 2600),
    (30000, 128, 1500),                  # 118 batch tiles, three whole tiles and no rest
]


@pytest.fixture(scope="module")
def H():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU; there is no CPU fallback")
    from tests import gpu_harness
    return gpu_harness


@pytest.mark.parametrize("B,D,C", SHAPES)
@pytest.mark.parametrize("g,with_bias", [(1.0, False), (-0.25, True)])
def test_step_on_lists(H, B, D, C, g, with_bias):
    p = inputs.make_inputs("list", B, D, C, x_sigma=1.0, w_sigma=0.3, bias_sigma=1.0 if with_bias else 0.0, seed=B + C)
    bias = p.bias if with_bias else None
    cut = C // 3
    shards = [(0, C)] if g > 0 else [(0, C - cut), (C - cut, cut)]       # labels outside the shard, too; an odd width
    shape = f"B={B} D={D} C={C} g={g}"
    H.say(f"[parity] lists of tiles: {shape}")
    got = H.run_step(p.X_bits, p.W_bits, bias, p.labels, shards, g=g)
    ref = H.oracle_step(p.X_bits, p.W_bits, bias, p.labels, shards, g=g)
    rep = H.compare(got, ref, p.labels, shards, shape, gate="fp32_floor")
    H.record(f"lists of tiles {shape}", f"{shape} gate=fp32_floor", rep)


def test_forward_with_a_partial_result_per_class_tile(H):
    """66 tiles in 128 ranges need more room than 33 class tiles; the tiles do without.  The maximum and the label's logit are
    the same numbers, the sums differ in their order only (two fp32 roundings per merge of the 33 and 128 partial sums)."""
    import torch
    from paper_2011_09208_amd import binding as ws
    B, D, C = 257, 192, 256 * 33 - 7
    p = inputs.make_inputs("list", B, D, C, x_sigma=1.0, w_sigma=0.3, seed=1)
    X, W, y = H.dev_bf16(p.X_bits), H.dev_bf16(p.W_bits), torch.from_numpy(np.ascontiguousarray(p.labels, dtype=np.int32)).cuda()
    least, full = 2 * 33 * 512 * 4, ws.fwd_workspace_bytes(B, D, C)
    assert full == 2 * 128 * 512 * 4 > least
    out = []
    for n in (full, least):
        m, s, t = (torch.empty(B, device="cuda") for _ in range(3))
        work = torch.empty(n, dtype=torch.uint8, device="cuda").fill_(0xFF)
        ws.split_fc_fwd(X, W, None, y, 0, m, s, t, work)
        out.append((m, s, t))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][2], out[1][2])
    assert (out[0][1] - out[1][1]).abs().max() <= 2.0 ** -24 * 2 * (33 + 128) * out[0][1].max()
    with pytest.raises(ws.WhaleSplitError):
        ws.split_fc_fwd(X, W, None, y, 0, m, s, t, work[:least - 16])


@pytest.mark.parametrize("B,D,C", [(50000, 128, 600), (600, 640, 256 * 170 + 33), (700, 576, 256 * 112 + 65), (64, 192, 140000)])
def test_wide_tiles_add_in_the_order_of_the_step(H, B, D, C):
    """Lists of several whole tiles, which alternate their direction, one of them with a single range, and a step of 64 x 64 tiles,
    which do not: the arg-max's logit (wide tiles) is the forward call's maximum, and with that class as the label its label logit, bit for bit."""
    import torch
    from paper_2011_09208_amd import binding as ws
    H.say(f"[parity] lists and wide tiles: B={B} D={D} C={C}")
    gen = torch.Generator(device="cuda").manual_seed(B)
    X, W = (torch.randn((n, D), device="cuda", generator=gen).to(torch.bfloat16) for n in (B, C))
    m, s, t, top = (torch.empty(B, device="cuda") for _ in range(4))
    y = torch.empty(B, device="cuda", dtype=torch.int32)
    work = torch.empty(ws.fwd_workspace_bytes(B, D, C), dtype=torch.uint8, device="cuda")
    ws.split_fc_top1(X, W, None, 0, top, y, work)
    ws.split_fc_fwd(X, W, None, y, 0, m, s, t, work)
    assert torch.equal(m, top) and torch.equal(t, top)
