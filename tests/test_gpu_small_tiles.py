"""Matrix products on few tokens: 128 x 128 tiles with four LDS stages, their
two-stage form when there are more tiles than compute units, and products whose
K is split over workgroups, against fp64.

Tolerances: a bf16 result (8 significant bits) differs from fp64 by its own rounding, 2^-8 of its
value, plus fp32 sums of K <= 600 products (below 600 * 2^-24); an fp32 one by
the sums alone."""
import numpy as np
import pytest
import torch

from paper_2510_02483_amd import configs, inputs, lib as L

from gpu_util import GRAD_TOL, OUT_TOL, bf16_randn, f64, fro_rel, max_rel, need_gpu, oracle_block, say

pytestmark = pytest.mark.gpu

BF16_TOL = 2.0 ** -8 + 1e-4
F32_TOL = 600 * 2.0 ** -24

# edges of the 128 x 128 tile; K: 1..9 whole k tiles of 64 (fewer than the four
# stages, exactly four, one pass of the unrolled loop and every remainder) and ragged ones
MN = [(8, 8), (120, 136), (128, 128), (136, 264), (264, 120)]
KS = [8, 64, 72, 128, 192, 256, 264, 320, 384, 448, 512, 520, 576]


@pytest.mark.parametrize("K", KS)
def test_small_products(K):
    need_gpu()
    for M, N in MN:
        say(f"small products M={M} N={N} K={K}")
        A, B = bf16_randn((M, K), 1), bf16_randn((N, K), 2)
        ref = f64(A) @ f64(B).T
        C = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
        L.ls_gemm_nt(A, B, C)
        torch.cuda.synchronize()
        assert max_rel(f64(C), ref) < BF16_TOL
        C.fill_(float("nan"))
        L.ls_gemm_nn(A, B.t().contiguous(), C)
        torch.cuda.synchronize()
        assert max_rel(f64(C), ref) < BF16_TOL
        F = torch.full((M, N), 0.25, dtype=torch.float32, device="cuda")
        L.ls_gemm_tn(A.t().contiguous(), B.t().contiguous(), F, accumulate=True)
        torch.cuda.synchronize()
        assert max_rel(f64(F) - 0.25, ref) < F32_TOL


# 17 x 21 = 357 tiles of 128 x 128: more than the compute units, fewer than two per unit
@pytest.mark.parametrize("K", [64, 136, 320])
def test_more_tiles_than_units(K):
    need_gpu()
    M, N = 2056, 2568
    say(f"two tiles per unit M={M} N={N} K={K}")
    A, B = bf16_randn((M, K), 3), bf16_randn((N, K), 4)
    ref = f64(A) @ f64(B).T
    C = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    L.ls_gemm_nt(A, B, C)
    torch.cuda.synchronize()
    assert max_rel(f64(C), ref) < BF16_TOL
    L.ls_gemm_nn(A, B.t().contiguous(), C)
    torch.cuda.synchronize()
    assert max_rel(f64(C), ref) < BF16_TOL


# 72 tokens against a width of 4104: every product of the MLP, and those of the
# attention layer whose K is the width (first case: 128-wide heads) or the heads'
# features (second: 64-wide), splits its K; ragged in every dimension
SPLIT_D128 = configs.BlockConfig("split-d128", 31, batch=1, seq=72, hidden=4104, n_q_heads=4, n_kv_heads=2,
                                 head_dim=128, intermediate=4616, rope_theta=1e4)
SPLIT_D64 = configs.BlockConfig("split-d64", 32, batch=2, seq=36, hidden=4104, n_q_heads=72, n_kv_heads=8, head_dim=64,
                                intermediate=264, rope_theta=1e4)


@pytest.mark.parametrize("c", [SPLIT_D128, SPLIT_D64], ids=lambda c: c.name)
def test_split_products(c):
    need_gpu()
    say(f"split products {c.name}")
    host = inputs.make_inputs(c, gamma="random")
    blk = L.Block(c, host)
    blk.step()
    torch.cuda.synchronize()
    fwd, gr = oracle_block(c, inputs.to_f64(host))
    shp = (c.batch, c.seq, c.hidden)
    assert max_rel(f64(blk.y).reshape(shp), fwd["y"]) < OUT_TOL
    assert fro_rel(f64(blk.dx).reshape(shp), gr["dx"]) < GRAD_TOL
    for n in L.WEIGHTS:
        assert fro_rel(f64(blk.grads[n]), gr[n]) < GRAD_TOL, n


def test_mlp_forward_with_and_without_scratch():
    """The MLP forward runs unsplit without a workspace: the same up to the order of its fp32 sums."""
    need_gpu()
    c = SPLIT_D128
    sizes = L.ls_query_sizes(c)
    unsplit = 2 * c.tokens * (2 * c.intermediate + c.hidden) + 4 * (c.tokens + 31) // 8 * c.hidden
    assert sizes["mlp_workspace"] > unsplit  # room for partial sums: some product of this shape splits
    host = inputs.make_inputs(c, gamma="random")
    w = {n: host[n].cuda() for n in L.WEIGHTS}
    x = host["x"].cuda().view(c.tokens, c.hidden)
    out = []
    for ws in (None, torch.empty(sizes["mlp_workspace"], dtype=torch.uint8, device="cuda")):
        y = torch.empty_like(x)
        saved = torch.empty(sizes["mlp_saved"], dtype=torch.uint8, device="cuda")
        L.ls_mlp_fwd(c, x, w, y, saved, ws)
        torch.cuda.synchronize()
        out.append(f64(y))
    # one bf16 unit in the last place (2^-7) where a sum lies at a rounding boundary
    assert np.max(np.abs(out[0] - out[1])) <= 2.0 ** -7 * np.max(np.abs(out[0]))


# q/k/v projections that take 256 x 128 tiles (K = 256: unsplit) or, forced, 256 x 256
ROPE_D128 = configs.BlockConfig("rope-d128", 33, batch=2, seq=1030, hidden=256, n_q_heads=16, n_kv_heads=2, head_dim=128,
                                intermediate=264, rope_theta=1e4)
ROPE_D64 = configs.BlockConfig("rope-d64", 34, batch=2, seq=1030, hidden=256, n_q_heads=24, n_kv_heads=8, head_dim=64,
                               intermediate=264, rope_theta=1e4)


@pytest.mark.parametrize("c", [ROPE_D128, ROPE_D64], ids=lambda c: c.name)
def test_rope_does_not_depend_on_the_tile(c):
    """Unsplit products sum K in the same order in every tile shape, and the rotation rounds
    the same way in every epilogue: the saved state (q, k, v, o) is the same bit for bit."""
    need_gpu()
    say(f"rope by tile shape {c.name}")
    host = inputs.make_inputs(c, gamma="random")
    w = {n: host[n].cuda() for n in L.WEIGHTS}
    x = host["x"].cuda().view(c.tokens, c.hidden)
    sizes = L.ls_query_sizes(c)
    got = []
    try:
        for tile in ((0, 0), (256, 256)):
            L.ls_gemm_tile_override(*tile)
            y = torch.empty_like(x)
            saved = torch.zeros(sizes["attn_saved"], dtype=torch.uint8, device="cuda")
            L.ls_attn_fwd(c, x, w, y, saved, torch.empty(sizes["attn_workspace"], dtype=torch.uint8, device="cuda"))
            torch.cuda.synchronize()
            got.append((saved, y))
    finally:
        L.ls_gemm_tile_override(0, 0)
    assert torch.equal(got[0][0], got[1][0])
    assert torch.equal(got[0][1], got[1][1])


# RMSNorm backward: rows per workgroup 8 (up to 2048 rows), 16, 24 and 32 (from
# 6145 on; past 8192 more than 256 workgroups), each with a ragged last workgroup
@pytest.mark.parametrize("rows", [1, 2047, 2049, 4100, 6150, 8300])
def test_rmsnorm_backward_rows(rows):
    need_gpu()
    hidden = 264
    say(f"rmsnorm backward rows={rows}")
    x, dh, dres = (bf16_randn((rows, hidden), s) for s in (1, 2, 3))
    gamma = bf16_randn((hidden,), 4, 0.1) + 1
    h, r = torch.empty_like(x), torch.empty(rows, dtype=torch.float32, device="cuda")
    L.ls_rmsnorm_fwd(rows, hidden, 1e-5, x, gamma, h, r)
    dx, dg = torch.empty_like(x), torch.full((hidden,), 0.5, dtype=torch.float32, device="cuda")
    ws = torch.empty(L.ls_rmsnorm_bwd_workspace(rows, hidden), dtype=torch.uint8, device="cuda")
    L.ls_rmsnorm_bwd(rows, hidden, x, gamma, r, dh, dres, dx, dg, True, ws)
    torch.cuda.synchronize()
    xf, g, d = f64(x), f64(gamma), f64(dh)
    rr = 1 / np.sqrt(np.mean(xf * xf, 1, keepdims=True) + 1e-5)
    ref = f64(dres) + rr * g * d - xf * rr ** 3 * np.sum(g * d * xf, 1, keepdims=True) / hidden
    assert max_rel(f64(dx), ref) < BF16_TOL
    # r is fp32 (2^-23) and the column sums add at most 8300 terms of random sign in fp32
    assert fro_rel(f64(dg) - 0.5, np.sum(d * xf * rr, 0)) < 1e-5


# in registers and streamed (above 131072 columns)
@pytest.mark.parametrize("V", [264, 131088])
def test_cross_entropy_smallest_gradients(V):
    """Probabilities below 2^-126 (exp(-88) to exp(-91)) reach the bf16 gradients, which go down to 2^-133."""
    need_gpu()
    say(f"cross-entropy smallest gradients V={V}")
    z = torch.full((1, V), -88.0, dtype=torch.bfloat16)
    z[0, 1::2] = -90.0
    z[0, 2::4] = -91.0
    z[0, 5] = 0.0
    p = torch.softmax(z.double(), 1).numpy()
    p[0, 5] -= 1
    zc = z.cuda()
    loss, row = torch.empty(1, device="cuda"), torch.empty(1, device="cuda")
    ws = torch.empty(L.ls_cross_entropy_workspace(1), dtype=torch.uint8, device="cuda")
    ids = torch.zeros(1, dtype=torch.int32, device="cuda")
    L.ls_cross_entropy(zc, 1, ids, torch.full((1,), 5, dtype=torch.int32, device="cuda"), loss, row, ws)
    torch.cuda.synchronize()
    got = zc.cpu().double().numpy()
    # bf16 below 2^-126 steps by 2^-133 (rounding 2^-134), the fp32 exponent (up to 132) is rounded to 2^-17
    assert np.max(np.abs(got - p)) <= 2.0 ** -134 + 2.0 ** -17 * 2.0 ** -126
    assert got[0, 0] > 0 and got[0, 1] > 0 and got[0, 2] > 0
