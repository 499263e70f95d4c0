"""GPU parity of the kernels that merge statistics across shards, at the batch and workgroup edges of their loops:
combine_partials loads eight shards at a time, merge_class_tiles eight partials for each of 64 threads per row, 8 rows per
workgroup, merge_top1 deals candidates to 64 threads per row and 16 rows per workgroup, or one thread to a row for up to
twelve candidates."""
import numpy as np
import pytest

from oracle import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ws():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU; there is no CPU fallback")
    from paper_2011_09208_amd import binding
    return binding


@pytest.mark.parametrize("S,B", [(1, 1), (7, 63), (8, 64), (9, 65), (16, 200), (17, 130)])
def test_combine_partials_batches_of_shards(ws, S, B):
    import torch
    rng = np.random.default_rng(100 * S + B)
    m = rng.normal(0, 4, (S, B)).astype(np.float32)
    s = rng.uniform(1, 500, (S, B)).astype(np.float32)
    t = np.zeros((S, B), np.float32)
    t[rng.integers(0, S, B), np.arange(B)] = rng.normal(0, 4, B)
    if S > 1:
        m[S - 1, ::3], s[S - 1, ::3] = -np.inf, 0.0                # a shard without classes for these rows
    dm, ds, dt = (torch.from_numpy(x).cuda() for x in (m, s, t))
    lse, loss = torch.empty(B, device="cuda"), torch.empty(B, device="cuda")
    ws.combine_partials(dm, ds, dt, lse, loss, None)
    m64 = m.astype(np.float64)
    ref = np.log((s * np.exp(m64 - m64.max(0))).sum(0)) + m64.max(0)
    # fp32: the sum of S terms (each an exp of 2 ulp), a log, one add; loss subtracts t
    tol = 2.0 ** -23 * (S + 6) + 2.0 ** -23 * np.maximum(np.abs(ref), np.abs(t.sum(0)))
    assert (np.abs(lse.cpu().numpy() - ref) <= tol).all()
    assert (np.abs(loss.cpu().numpy() - (ref - t.sum(0))) <= 2 * tol).all()


@pytest.mark.parametrize("S,B", [(1, 1), (2, 15), (8, 63), (9, 64), (12, 65), (13, 65), (63, 16), (64, 17), (65, 33), (391, 2),
                                 (513, 16)])
def test_combine_top1_groups_of_candidates(ws, S, B):
    import torch
    rng = np.random.default_rng(100 * S + B)
    v = rng.integers(-3, 4, (S, B)).astype(np.float32)             # many ties: the lowest class id wins
    c = np.stack([rng.permutation(10 * S)[:S] for _ in range(B)], 1).astype(np.int32)
    v[:, B // 2] = -np.inf                                         # all candidates of one row alike
    dv, dc = torch.from_numpy(v).cuda(), torch.from_numpy(c).cuda()
    bv, bc = torch.empty(B, device="cuda"), torch.empty(B, device="cuda", dtype=torch.int32)
    ws.combine_top1(dv, dc, bv, bc)
    rv, rc = oracle.combine_top1(list(v.astype(np.float64)), list(c.astype(np.int64)))
    assert (bv.cpu().numpy() == rv).all() and (bc.cpu().numpy() == rc).all()


@pytest.mark.parametrize("B", [1, 1023, 1025, 1792, 1793, 2048, 2049])
@pytest.mark.parametrize("S", [1, 8, 9])
def test_mean_in_the_combine_launch(B, S):
    """Up to 1792 rows and 8 shards one workgroup does it all: rows bit for bit as without the mean, the mean within the
    rounding of its B fp32 additions."""
    import torch
    from paper_2011_09208_amd import binding as ws
    g = torch.Generator(device="cuda").manual_seed(B + S)
    m, t = (torch.empty((S, B), device="cuda").normal_(0.0, 3.0, generator=g) for _ in range(2))
    s = torch.empty((S, B), device="cuda").uniform_(1.0, 9.0, generator=g)
    m[0, 0] = float("-inf")                                        # an empty shard
    s[0, 0] = 0.0 if S > 1 else 1.0
    if S == 1:
        m[0, 0] = 0.0
    out = [torch.empty(B, device="cuda") for _ in range(4)]
    mean = torch.empty(1, device="cuda")
    ws.combine_partials(m, s, t, out[0], out[1], None)
    ws.combine_partials(m, s, t, out[2], out[3], mean)
    assert torch.equal(out[0], out[2]) and torch.equal(out[1], out[3])
    loss = out[1].double()
    assert (mean.double() - loss.mean()).abs() <= 2.0 ** -24 * (12 + B / 1024) * loss.abs().mean()


@pytest.mark.parametrize("B,parts", [(1, 1), (17, 129), (24, 511), (33, 512), (40, 513), (63, 65), (64, 1025), (17, 1100)])
def test_forward_statistics_of_many_partial_results(ws, B, parts):
    """64 x 64 tiles (one row: the small-batch kernel): a partial result for every 64 classes, the last of them of three.  Small integers, so the
    logits are exact; a sum is up to 8 logits of a lane, 3 merges in a tile, 8 of a batch's turns of 8 and 15 merges of 64 threads."""
    import torch
    D, C = 64, 64 * parts - 61
    g = torch.Generator(device="cuda").manual_seed(parts)
    X = torch.randint(-1, 2, (B, D), device="cuda", generator=g).to(torch.bfloat16)
    W = torch.randint(-1, 2, (C, D), device="cuda", generator=g).to(torch.bfloat16)
    bias = torch.zeros(C, device="cuda")
    bias[64:192] = float("-inf")                                   # whole tiles without a class
    y = torch.randint(0, min(C, 64), (B,), device="cuda", generator=g, dtype=torch.int32)
    m, s, t = (torch.empty(B, device="cuda") for _ in range(3))
    ws.split_fc_fwd(X, W, bias, y, 0, m, s, t, torch.empty(ws.fwd_workspace_bytes(B, D, C), dtype=torch.uint8, device="cuda"))
    z = X.double() @ W.double().t() + bias.double()
    top = z.max(1).values
    assert torch.equal(m.double(), top) and torch.equal(t.double(), z.gather(1, y.long()[:, None])[:, 0])
    ref = torch.exp(z - top[:, None]).sum(1)
    # per term: an addition at each of up to 40 places, an exponential and its argument's rounding at each of up to 22
    tol = 2.0 ** -24 * (40 + 22 * (2 + 2 * z[z > -1e9].abs().max()))
    assert ((s.double() - ref).abs() <= tol * ref).all()
