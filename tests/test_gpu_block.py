"""GPU parity of dW where its output is small: the 64 x 64 tiles at the edges of their class tiles and of their five stages of the
contraction (1, 4, 5, 6 k-steps), with ragged last k-steps, and either side of the lines to the wide and thin tiles (192 and
512 of them, 20 k-steps); and launches of less than one round of thin tiles.  Plain and with the fused update."""
import numpy as np
import pytest

from paper_2011_09208_amd import inputs

pytestmark = pytest.mark.gpu

SHAPES = [                               # B, D, C
    (65, 64, 1),                         # 2 k-steps, one class
    (60, 128, 63),                       # 1
    (66, 2112, 65),                      # 2; 33 feature tiles, the second class tile one class wide
    (256, 64, 64),                       # 4: all stages but one
    (257, 320, 200),                     # 5: every stage once
    (384, 192, 129),                     # 6
    (700, 64, 64 * 192),                 # 11; 192 tiles, as many as are taken for any contraction
    (700, 64, 64 * 192 + 1),             # 193: 49 wide tiles, thin above 11 k-steps
    (1217, 256, 64 * 128),               # 20; 512 tiles
    (1216, 256, 64 * 128),               # 19: 32 thin tiles
    (1217, 256, 64 * 128 + 1),           # 513: 33 thin tiles
    (300, 1024, 2200),                   # 36 tiles of 5 k-steps, thin
    (300, 1024, 2600),                   # 44, wide
]


@pytest.fixture(scope="module")
def H():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU; there is no CPU fallback")
    from tests import gpu_harness
    return gpu_harness


@pytest.mark.parametrize("B,D,C", SHAPES)
def test_dw_of_small_outputs(H, B, D, C):
    import torch
    from paper_2011_09208_amd import binding as ws
    p = inputs.make_inputs("block", B, D, C, x_sigma=1.0, w_sigma=0.3, bias_sigma=1.0, seed=B + C)
    shape = f"B={B} D={D} C={C}"
    H.say(f"[parity] dW of small outputs: {shape}")
    got = H.run_step(p.X_bits, p.W_bits, p.bias, p.labels, [(0, C)], g=1.0 / B)
    ref = H.oracle_step(p.X_bits, p.W_bits, p.bias, p.labels, [(0, C)], g=1.0 / B)
    rep = H.compare(got, ref, p.labels, [(0, C)], shape, gate="fp32_floor")
    H.record(f"dW of small outputs {shape}", f"{shape} gate=fp32_floor", rep)

    # the fused update takes the same gradient: W - lr * dW in fp32, rounded once (a fused multiply-add: no second rounding)
    X, W = H.dev_bf16(p.X_bits), H.dev_bf16(p.W_bits)
    b, y = torch.from_numpy(p.bias).cuda(), torch.from_numpy(np.ascontiguousarray(p.labels, dtype=np.int32)).cuda()
    work = torch.empty(ws.bwd_workspace_bytes(B, D, C), dtype=torch.uint8, device="cuda").fill_(0xFF)
    lse = torch.logsumexp(X.float() @ W.float().T + b, 1)
    dX, dW, db = torch.empty((B, D), device="cuda"), torch.empty_like(W), torch.empty(C, device="cuda")
    ws.split_fc_bwd(X, W, b, lse, y, 0, 1.0, dX, False, dW, db, work)
    W1, b1 = W.clone(), b.clone()
    ws.split_fc_bwd_sgd(X, W1, b1, lse, y, 0, 1.0, 0.25, dX, False, work.fill_(0xFF))
    assert torch.equal(W1, (W.double() - 0.25 * dW.double()).float().bfloat16())
    assert torch.equal(b1, torch.addcmul(b.double(), db.double(), torch.full_like(db, -0.25).double()).float())
