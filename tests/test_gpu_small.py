"""GPU parity of the logits kernels for small batches (up to 32 rows and 2048 features: statistics, dz, probabilities,
arg-max) at the edges of their 16-row blocks, of the 32 classes they take at a time and of the workgroups' ranges, and
with contractions shorter and longer than one round of their waves; and of batches of up to 65 rows, which take 64 x 64 tiles."""
import numpy as np
import pytest

from oracle import oracle
from paper_2011_09208_amd import inputs

pytestmark = pytest.mark.gpu

SHAPES = [                               # B, D, widths
    (1, 64, [5, 27]),                    # one wave has work; a few classes and one short of 32
    (16, 512, [32, 33]),                 # eight k-steps: one per wave
    (17, 576, [31, 64, 1]),              # nine; the second 16-row block has one row
    (31, 128, [97]),
    (32, 1088, [700, 65]),               # seventeen k-steps
    (33, 1024, [63, 129]),               # sixteen; here and below, with 33 rows or more, 64 x 64 tiles
    (64, 192, [1000]),
    (5, 128, [256 * 32, 256 * 32 + 1]),  # 256 ranges of 32 classes; ranges of 40, walked 32 and 8
    (20, 64, [256 * 57 + 3]),            # too many classes for more than 16 rows: 64 x 64 tiles
    (12, 64, [256 * 57 + 3]),            # ranges of 64, the last 35 classes
    (64, 2048, [256 * 64 + 1]),
    (16, 2048, [256 * 64 + 1]),          # all registers full; ranges of 72: 32, 32, 8
    (65, 192, [1000]),
    (40, 2112, [300]),
    (16, 2112, [300]),                   # one k-step too many: 64 x 64 tiles
    (40, 704, [6000, 6150]),
    (64, 1024, [24576, 24577]),
    (33, 192, [24576, 24577]),
    (50, 64, [256 * 48, 256 * 97]),
    (36, 768, [256 * 256 + 9]),
    (20, 128, [256 * 224, 256 * 224 + 1]),   # the arg-max here, ranges of 224 and 232, the rest in 64 x 64 tiles
]


@pytest.fixture(scope="module")
def H():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU; there is no CPU fallback")
    from tests import gpu_harness
    return gpu_harness


@pytest.mark.parametrize("B,D,widths", SHAPES)
@pytest.mark.parametrize("g", [1.0, -0.25])
def test_small_batch_step(H, B, D, widths, g):
    C = sum(widths)
    shards = [(sum(widths[:i]), w) for i, w in enumerate(widths)]
    p = inputs.make_inputs("small", B, D, C, x_sigma=1.0, w_sigma=0.3, bias_sigma=1.0, seed=B + C)
    shape = f"B={B} D={D} widths={widths} g={g}"
    H.say(f"[parity] small batch: {shape}")
    got = H.run_step(p.X_bits, p.W_bits, p.bias, p.labels, shards, g=g)
    ref = H.oracle_step(p.X_bits, p.W_bits, p.bias, p.labels, shards, g=g)
    rep = H.compare(got, ref, p.labels, shards, shape, gate="fp32_floor")
    H.record(f"small batch {shape}", f"{shape} gate=fp32_floor", rep)


@pytest.mark.parametrize("B,D,widths", SHAPES)
def test_small_batch_probabilities_and_top1(H, B, D, widths):
    import torch
    from paper_2011_09208_amd import binding as ws
    C = sum(widths)
    p = inputs.make_inputs("small", B, D, C, x_sigma=1.0, w_sigma=0.3, bias_sigma=1.0, seed=B + C + 1)
    H.say(f"[parity] small batch, probabilities and top-1: B={B} D={D} widths={widths}")
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
        # one bf16 rounding, and z and lse within fp32 sums; at D = 2048 the logits spread over 100 and probabilities below
        # the smallest normal fp32 and bf16 number, 2^-126, are flushed to zero
        assert (np.abs(got[:B, :w] - ref) <= (2.0 ** -8 + 2 * H.LSE_ABS * zmax) * ref + 2.0 ** -126).all()
        work = torch.empty(ws.fwd_workspace_bytes(B, D, w), dtype=torch.uint8, device="cuda").fill_(0xFF)
        tv, tc = torch.empty(B, device="cuda"), torch.empty(B, device="cuda", dtype=torch.int32)
        ws.split_fc_top1(X, W[off:off + w], b[off:off + w], off, tv, tc, work)
        tv, tc = tv.cpu().numpy(), tc.cpu().numpy()
        best = Z[:, off:off + w].max(1)
        assert ((tc >= off) & (tc < off + w)).all() and (np.abs(tv - best) <= H.LSE_ABS * zmax).all()
        assert (Z[np.arange(B), tc] >= best - 2 * H.LSE_ABS * zmax).all()
        off += w


def test_small_batch_top1_ties(H):
    """Equal logits everywhere: the lowest class id of the shard."""
    import torch
    from paper_2011_09208_amd import binding as ws
    for B in (1, 20, 64):
        X = torch.ones((B, 128), device="cuda", dtype=torch.bfloat16)
        W = torch.ones((500, 128), device="cuda", dtype=torch.bfloat16)
        work = torch.empty(ws.fwd_workspace_bytes(B, 128, 500), dtype=torch.uint8, device="cuda")
        tv, tc = torch.empty(B, device="cuda"), torch.empty(B, device="cuda", dtype=torch.int32)
        ws.split_fc_top1(X, W, None, 40, tv, tc, work)
        assert (tc == 40).all() and (tv == 128.0).all()
