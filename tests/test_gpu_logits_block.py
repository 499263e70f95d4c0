"""GPU parity of the logits kernels in 64 x 64 tiles at the sizes where they can go wrong: one row, a full and a ragged block of
rows, one class, ragged classes, fewer k-steps than the four that are loaded ahead and more, the lines to the small-batch
kernels and to the wider tiles, and a forward call whose workspace holds no more than a partial result per 256 classes."""
import numpy as np
import pytest

from oracle import oracle
from paper_2011_09208_amd import inputs

pytestmark = pytest.mark.gpu

SHAPES = [                               # B, D, widths
    (17, 64, [8192, 8193]),              # the small-batch kernels; here
    (32, 576, [8193, 32768, 32769]),     # arg-max of the last there
    (1, 2112, [1, 65]),                  # one row, one class; 33 k-steps
    (33, 64, [1, 63, 64]),
    (40, 256, [129]),                    # four k-steps
    (63, 320, [66, 200]),                # five
    (64, 384, [65, 3]),                  # six
    (64, 192, [64 * 1280, 64 * 1280 + 1]),   # the last: arg-max on wide tiles
    (20, 2112, [64 * 1280, 64 * 1280 + 1]),  # the last: the step in lists, the rest on wide tiles
    (65, 320, [100, 1]),                 # a block of one row
    (127, 64, [333]),
    (200, 128, [64 * 128 - 5, 64 * 128 + 1]),    # 512 tiles; 516: the step on wide ones
    (260, 192, [64 * 205 - 1]),          # 1025: the step in lists, the rest on wide ones
    (500, 64, [64 * 128]),               # 1024: the step and the arg-max on wide ones
    (1000, 448, [257]),                  # 16 blocks of rows
]


@pytest.fixture(scope="module")
def H():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU; there is no CPU fallback")
    from tests import gpu_harness
    return gpu_harness


@pytest.mark.parametrize("B,D,widths", SHAPES)
@pytest.mark.parametrize("g,with_bias", [(1.0, False), (-0.25, True)])
def test_step(H, B, D, widths, g, with_bias):
    C = sum(widths)
    shards = [(sum(widths[:i]), w) for i, w in enumerate(widths)]
    p = inputs.make_inputs("block", B, D, C, x_sigma=1.0, w_sigma=0.3, bias_sigma=1.0 if with_bias else 0.0, seed=B + C)
    bias = p.bias if with_bias else None
    shape = f"B={B} D={D} widths={widths} g={g}"
    H.say(f"[parity] logits in 64 x 64 tiles: {shape}")
    got = H.run_step(p.X_bits, p.W_bits, bias, p.labels, shards, g=g)
    ref = H.oracle_step(p.X_bits, p.W_bits, bias, p.labels, shards, g=g)
    rep = H.compare(got, ref, p.labels, shards, shape, gate="fp32_floor")
    H.record(f"logits in 64 x 64 tiles {shape}", f"{shape} gate=fp32_floor", rep)


@pytest.mark.parametrize("B,D,widths", SHAPES)
def test_probabilities_and_top1(H, B, D, widths):
    """Bounds as for the small-batch kernels: one bf16 rounding of a probability, z and lse within fp32 sums, probabilities
    below 2^-126 flushed to zero; an arg-max whose logit is the largest within those sums."""
    import torch
    from paper_2011_09208_amd import binding as ws
    C = sum(widths)
    p = inputs.make_inputs("block", B, D, C, x_sigma=1.0, w_sigma=0.3, bias_sigma=1.0, seed=B + C + 1)
    H.say(f"[parity] probabilities and top-1 in 64 x 64 tiles: B={B} D={D} widths={widths}")
    X, W, b = H.dev_bf16(p.X_bits), H.dev_bf16(p.W_bits), torch.from_numpy(p.bias).cuda()
    Z = oracle.logits(inputs.bf16_bits_to_f64(p.X_bits), inputs.bf16_bits_to_f64(p.W_bits), p.bias.astype(np.float64))
    zmax = max(1.0, float(np.abs(Z).max()))
    lse64 = np.log(np.exp(Z - Z.max(1, keepdims=True)).sum(1)) + Z.max(1)
    lse = torch.from_numpy(lse64.astype(np.float32)).cuda()
    pitch = (C + 15) // 8 * 8                                       # at least one padding column, which must stay as it is
    off = 0
    for w in widths:
        P = torch.full((B + 1, pitch), 7.0, device="cuda", dtype=torch.bfloat16)
        ws.split_fc_predict(X, W[off:off + w], b[off:off + w], lse, P[:B, :w])
        got = H.bf16_to_f64(P)
        ref = np.exp(Z[:, off:off + w] - lse64[:, None])
        assert (got[:B, w:] == 7.0).all() and (got[B] == 7.0).all()
        assert (np.abs(got[:B, :w] - ref) <= (2.0 ** -8 + 2 * H.LSE_ABS * zmax) * ref + 2.0 ** -126).all()
        best = Z[:, off:off + w].max(1)
        least = 2 * ((w + 255) // 256) * ((B + 255) // 256 * 256) * 4
        values = []
        for n in (ws.fwd_workspace_bytes(B, D, w), least):          # with the latter, wide tiles above 64 rows
            work = torch.empty(n, dtype=torch.uint8, device="cuda").fill_(0xFF)
            tv, tc = torch.empty(B, device="cuda"), torch.empty(B, device="cuda", dtype=torch.int32)
            ws.split_fc_top1(X, W[off:off + w], b[off:off + w], off, tv, tc, work)
            values.append((tv, tc))
            tv, tc = tv.cpu().numpy(), tc.cpu().numpy()
            assert ((tc >= off) & (tc < off + w)).all() and (np.abs(tv - best) <= H.LSE_ABS * zmax).all()
            assert (Z[np.arange(B), tc] >= best - 2 * H.LSE_ABS * zmax).all()
        assert torch.equal(values[0][0], values[1][0]) and torch.equal(values[0][1], values[1][1])
        off += w


def test_top1_ties(H):
    """Equal logits everywhere: the lowest class id of the shard."""
    import torch
    from paper_2011_09208_amd import binding as ws
    for B in (40, 64, 130):
        X = torch.ones((B, 128), device="cuda", dtype=torch.bfloat16)
        W = torch.ones((500, 128), device="cuda", dtype=torch.bfloat16)
        work = torch.empty(ws.fwd_workspace_bytes(B, 128, 500), dtype=torch.uint8, device="cuda")
        tv, tc = torch.empty(B, device="cuda"), torch.empty(B, device="cuda", dtype=torch.int32)
        ws.split_fc_top1(X, W, None, 40, tv, tc, work)
        assert (tc == 40).all() and (tv == 128.0).all()


@pytest.mark.parametrize("B,D,C", [(128, 320, 1001), (70, 1024, 900), (300, 2112, 1900), (300, 64, 5001)])
def test_forward_with_a_partial_result_per_256_classes(H, B, D, C):
    """The wide tiles do without the larger workspace (which up to 64 rows is none): the maximum and the label's logit are the same numbers, the sums
    differ in their order only (two fp32 roundings per merge of the partial sums)."""
    import torch
    from paper_2011_09208_amd import binding as ws
    p = inputs.make_inputs("block", B, D, C, x_sigma=1.0, w_sigma=0.3, bias_sigma=1.0, seed=1)
    X, W, b = H.dev_bf16(p.X_bits), H.dev_bf16(p.W_bits), torch.from_numpy(p.bias).cuda()
    y = torch.from_numpy(np.ascontiguousarray(p.labels, dtype=np.int32)).cuda()
    least, full = 2 * ((C + 255) // 256) * ((B + 255) // 256 * 256) * 4, ws.fwd_workspace_bytes(B, D, C)
    assert full == 2 * ((C + 63) // 64) * ((B + 63) // 64 * 64) * 4 > least
    out = []
    for n in (full, least):
        m, s, t = (torch.empty(B, device="cuda") for _ in range(3))
        work = torch.empty(n, dtype=torch.uint8, device="cuda").fill_(0xFF)
        ws.split_fc_fwd(X, W, b, y, 0, m, s, t, work)
        out.append((m, s, t))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][2], out[1][2])
    parts = (C + 63) // 64 + (C + 255) // 256
    assert ((out[0][1] - out[1][1]).abs() <= 2.0 ** -24 * (2 * parts + 128) * out[0][1]).all()
    with pytest.raises(ws.WhaleSplitError):
        ws.split_fc_fwd(X, W, b, y, 0, m, s, t, work[:least - 16])
