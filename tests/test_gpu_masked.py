"""GPU: classes masked through their bias, by -inf, the lowest float and numbers in between, in groups that fill a lane's, a wave's
and a tile's share of the classes, for every kind of logits kernel; and a shard of nothing but masked classes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SHAPES = [                               # B, D, C
    (5, 128, 5000),                      # small-batch kernels
    (32, 128, 5000),
    (40, 128, 5000),                     # 64 x 64 tiles
    (300, 1024, 800),
    (1100, 192, 3000),                   # thin tiles
    (300, 128, 12000),                   # lists, rests alone
    (700, 128, 40000),                   # lists, whole tiles first
    (1024, 1024, 12500),                 # wide tiles
    (256, 1024, 256 * 272),              # wide and thin tiles
]


@pytest.mark.parametrize("B,D,C", SHAPES)
def test_masked_classes_count_nothing(B, D, C):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU; there is no CPU fallback")
    from paper_2011_09208_amd import binding as ws
    print(f"[masked] B={B} D={D} C={C}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(C)
    X = torch.randn((B, D), device="cuda", generator=gen).to(torch.bfloat16)
    W = (0.05 * torch.randn((C, D), device="cuda", generator=gen)).to(torch.bfloat16)
    y = torch.randint(0, 20, (B,), device="cuda", generator=gen, dtype=torch.int32)       # never masked
    z = X.double() @ W.double().t()
    cut = C // 3 * 2
    work = torch.empty(max(ws.fwd_workspace_bytes(B, D, C), ws.bwd_workspace_bytes(B, D, C)), dtype=torch.uint8, device="cuda")
    for low in (-1e4, -1e10, -1e30, float(np.finfo(np.float32).min), float("-inf")):
        bias = torch.zeros(C, device="cuda")
        for n, at in ((1, 30), (8, 64), (32, 96), (64, 192), (300, 300)):                 # masked classes, from
            bias[at:at + n] = low
        bias[cut:] = low                                                                 # the second shard is masked altogether
        lse64 = torch.logsumexp(z + bias.double(), 1)
        m, s, t = (torch.empty((2, B), device="cuda") for _ in range(3))
        lse, loss = torch.empty(B, device="cuda"), torch.empty(B, device="cuda")
        for i, (a, e) in enumerate(((0, cut), (cut, C))):
            ws.split_fc_fwd(X, W[a:e], bias[a:e], y, a, m[i], s[i], t[i], work)
        ws.combine_partials(m, s, t, lse, loss, None)
        assert not torch.isnan(s).any() and not torch.isnan(m).any(), low
        # fp32 sums of D products and of C exponentials: some 1e-6 of logits of up to about 10
        assert (lse.double() - lse64).abs().max() <= 2e-5, low
        assert (m[1].double() - (z + bias.double())[:, cut:].max(1).values).abs().nan_to_num(0.0).max() <= 2.0 ** -23 * max(10.0, abs(low) if np.isfinite(low) else 0.0)
        one = torch.empty((B,), device="cuda")
        ws.split_fc_fwd(X, W, bias, y, 0, m[0], s[0], t[0], work)
        ws.combine_partials(m[:1], s[:1], t[:1], one, loss, None)
        assert (one.double() - lse64).abs().max() <= 2e-5, low
        dX = torch.empty((B, D), device="cuda")
        dW, db = torch.empty_like(W), torch.empty(C, device="cuda")
        ws.split_fc_bwd(X, W, bias, one, y, 0, 1.0, dX, False, dW, db, work)
        assert torch.isfinite(dX).all() and torch.isfinite(dW).all()
        assert (db[bias == low] == 0.0).all() and (dW[bias == low] == 0.0).all(), low
