"""Matrix products on few tokens: 128 x 128 tiles with four LDS stages, their
two-stage form when there are more tiles than compute units, 256 x 128 tiles, and
products whose K is split over workgroups, against fp64 or against the 256 x 256
tiles.  What is named is what runs: the tests ask the library for the plan of
each product and fail where it is another one (as after a change of the
estimate's constants: the shapes then have to be chosen anew).

Tolerances: a bf16 result (8 significant bits) differs from fp64 by its own rounding, 2^-8 of its
value, plus fp32 sums of K <= 600 products (below 600 * 2^-24); an fp32 one by
the sums alone."""
import numpy as np
import pytest
import torch

from paper_2510_02483_amd import configs, inputs, lib as L

from gpu_util import (GRAD_TOL, OUT_TOL, bf16_randn, f64, fro_rel, gemm_plan, max_rel, need_gpu, oracle_block, say,
                      step_plan)

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


# The two-stage 128 x 128 tiles (more tiles than compute units) and the
# three-stage 256 x 128 ones, at a ragged shape that takes them in each layout
TWO_STAGE, THREE_STAGE, FOUR_STAGE = (128, 128, 2), (256, 128, 3), (128, 128, 4)
NARROW = [("nt", TWO_STAGE, 136, 16392), ("nt", THREE_STAGE, 2056, 2568), ("nn", TWO_STAGE, 264, 12296),
          ("nn", THREE_STAGE, 136, 16392), ("tn", TWO_STAGE, 264, 12296), ("tn", THREE_STAGE, 136, 16392)]


@pytest.mark.parametrize("K", KS)
def test_more_tiles_than_units(K):
    need_gpu()
    for layout, kernel, M, N in NARROW:
        say(f"more tiles than units {layout} {kernel} M={M} N={N} K={K}")
        assert gemm_plan(("nt", "nn", "tn").index(layout), M, N, K) == kernel + (1,)
        A, B = bf16_randn((M, K), 3), bf16_randn((K, N), 4)
        ref = A.double() @ B.double()
        if layout == "tn":
            C = torch.full((M, N), 0.25, dtype=torch.float32, device="cuda")
            L.ls_gemm_tn(A.t().contiguous(), B, C, accumulate=True)
            C -= 0.25
        else:
            C = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
            L.ls_gemm_nt(A, B.t().contiguous(), C) if layout == "nt" else L.ls_gemm_nn(A, B, C)
        err = float((C.double() - ref).abs().max() / ref.abs().max())
        assert err < (F32_TOL if layout == "tn" else BF16_TOL), (layout, kernel)


# 72 tokens against a width of 4104: every product of the MLP, and those of the
# attention layer whose K is the width (first case: 128-wide heads) or the heads'
# features (second: 64-wide), splits its K; ragged in every dimension
SPLIT_D128 = configs.BlockConfig("split-d128", 31, batch=1, seq=72, hidden=4104, n_q_heads=4, n_kv_heads=2,
                                 head_dim=128, intermediate=4616, rope_theta=1e4)
SPLIT_D64 = configs.BlockConfig("split-d64", 32, batch=2, seq=36, hidden=4104, n_q_heads=72, n_kv_heads=8, head_dim=64,
                                intermediate=264, rope_theta=1e4)


# forced to 256 x 256 tiles they are unsplit: the small ragged shapes of those epilogues
@pytest.mark.parametrize("tile", [(0, 0), (256, 256)], ids=["split", "256x256"])
@pytest.mark.parametrize("c", [SPLIT_D128, SPLIT_D64], ids=lambda c: c.name)
def test_split_products(c, tile):
    need_gpu()
    say(f"split products {c.name} {tile}")
    for step in ("qkv projection", "dO") + (("gate/up projection", "down projection", "dact", "dh2")
                                            if c is SPLIT_D128 else ("gate/up projection", "dact", "output projection")):
        assert step_plan(c, step)[3] > 1, step
    host = inputs.make_inputs(c, gamma="random")
    blk = L.Block(c, host)
    try:
        L.ls_gemm_tile_override(*tile)
        blk.step()
    finally:
        L.ls_gemm_tile_override(0, 0)
    torch.cuda.synchronize()
    fwd, gr = oracle_block(c, inputs.to_f64(host))
    shp = (c.batch, c.seq, c.hidden)
    assert max_rel(f64(blk.y).reshape(shp), fwd["y"]) < OUT_TOL
    assert fro_rel(f64(blk.dx).reshape(shp), gr["dx"]) < GRAD_TOL
    for n in L.WEIGHTS:
        assert fro_rel(f64(blk.grads[n]), gr[n]) < GRAD_TOL, n


def _sub_layer(tokens, hidden, nq=1, nkv=1, d=64, intermediate=264, batch=1):
    return configs.BlockConfig("instance", 0, batch=batch, seq=tokens // batch, hidden=hidden, n_q_heads=nq, n_kv_heads=nkv,
                               head_dim=d, intermediate=intermediate, rope_theta=1e4)


QKV, OUT, GATE_UP, DOWN = "qkv projection", "output projection", "gate/up projection", "down projection"
SPLIT_256 = (256, 256, 2)
# Every narrow tile and every split with each epilogue that it has, at the
# smallest ragged shapes found that take them: {step: (kernel, split?)}
INSTANCES = [
    ("attn", _sub_layer(35, 520, 64, 8, 128), {QKV: (FOUR_STAGE, 0), OUT: (FOUR_STAGE, 1), "dWo": (TWO_STAGE, 0),
                                               "dWqkv": (THREE_STAGE, 0)}),
    ("attn", _sub_layer(2049, 2048), {QKV: (FOUR_STAGE, 0), OUT: (TWO_STAGE, 0), "dO": (FOUR_STAGE, 1),
                                      "dh1": (THREE_STAGE, 0), "dWo": (FOUR_STAGE, 1), "dWqkv": (FOUR_STAGE, 1)}),
    ("attn", _sub_layer(1373, 3072), {QKV: (FOUR_STAGE, 1), OUT: (TWO_STAGE, 0), "dh1": (TWO_STAGE, 0)}),
    ("attn", _sub_layer(1435, 3072), {OUT: (THREE_STAGE, 0), "dh1": (THREE_STAGE, 0)}),
    ("attn", _sub_layer(391, 256, 64, 8, 128), {QKV: (THREE_STAGE, 0), "dh1": (FOUR_STAGE, 1)}),
    ("attn", _sub_layer(1302, 256, 8, 8, 128, batch=2), {QKV: (TWO_STAGE, 0)}),
    ("attn", _sub_layer(777, 264, 64, 8, batch=3), {QKV: (TWO_STAGE, 0)}),
    ("attn", _sub_layer(915, 264, 64, 8, batch=3), {QKV: (THREE_STAGE, 0)}),
    ("attn", _sub_layer(33, 2048, 1, 1, 128), {QKV: (FOUR_STAGE, 1)}),
    ("attn", _sub_layer(137, 7304, 32, 8, 128), {QKV: (THREE_STAGE, 1)}),
    ("attn", _sub_layer(8288, 7920, batch=4), {QKV: (THREE_STAGE, 1)}),
    ("attn", _sub_layer(1321, 7904, 8, 8, 128), {QKV: (SPLIT_256, 1), "dWo": (THREE_STAGE, 0)}),
    ("attn", _sub_layer(2725, 8040, 8, 8), {QKV: (SPLIT_256, 1)}),
    ("mlp", _sub_layer(35, 256, intermediate=16760), {GATE_UP: (TWO_STAGE, 0), DOWN: (FOUR_STAGE, 1),
                                                      "dh2": (FOUR_STAGE, 1), "dWd": (THREE_STAGE, 0)}),
    ("mlp", _sub_layer(3601, 256, intermediate=1032), {GATE_UP: (THREE_STAGE, 0), "dact": (THREE_STAGE, 0),
                                                       "dWg/dWu": (FOUR_STAGE, 1), "dWd": (FOUR_STAGE, 1)}),
    ("mlp", _sub_layer(273, 256, intermediate=11792), {"dact": (TWO_STAGE, 0), "dWg/dWu": (THREE_STAGE, 0)}),
    ("mlp", _sub_layer(33, 2048), {GATE_UP: (FOUR_STAGE, 1), "dact": (FOUR_STAGE, 1)}),
    ("mlp", _sub_layer(141, 4104, intermediate=16880), {DOWN: (THREE_STAGE, 1), "dact": (SPLIT_256, 1),
                                                        "dh2": (THREE_STAGE, 1)}),
    ("mlp", _sub_layer(285, 4096, intermediate=15976), {DOWN: (TWO_STAGE, 1), "dact": (TWO_STAGE, 0),
                                                        "dh2": (SPLIT_256, 1)}),
    ("mlp", _sub_layer(301, 4104, intermediate=7352), {GATE_UP: (TWO_STAGE, 0), "dh2": (TWO_STAGE, 1)}),
    ("mlp", _sub_layer(387, 4104, intermediate=16208), {DOWN: (SPLIT_256, 1), "dact": (THREE_STAGE, 0)}),
    ("mlp", _sub_layer(7135, 264, intermediate=1920), {"dWg/dWu": (THREE_STAGE, 1), "dWd": (FOUR_STAGE, 1)}),
    ("mlp", _sub_layer(133, 6176, intermediate=5528), {"dact": (THREE_STAGE, 1)}),
    ("mlp", _sub_layer(33, 6952, intermediate=6000), {GATE_UP: (TWO_STAGE, 1)}),
]


def _run_sub_layer(part, c, host, tile, accumulate):
    """Outputs of one forward and backward pass, the weight gradients on top of 0.25 where accumulated."""
    names = ("attn_norm", "wq", "wk", "wv", "wo") if part == "attn" else ("mlp_norm", "wg", "wu", "wd")
    fwd, bwd = (L.ls_attn_fwd, L.ls_attn_bwd) if part == "attn" else (L.ls_mlp_fwd, L.ls_mlp_bwd)
    sizes = L.ls_query_sizes(c)
    x, dy = (host[n].view(c.tokens, c.hidden) for n in ("x", "dy"))
    w = {n: host[n] for n in names}
    saved, ws = (torch.empty(sizes[f"{part}_{n}"], dtype=torch.uint8, device="cuda") for n in ("saved", "workspace"))
    y, dx = torch.full_like(x, float("nan")), torch.full_like(x, float("nan"))
    grads = {n: torch.full(w[n].shape, 0.25 if accumulate else float("nan"), device="cuda") for n in names}
    try:
        L.ls_gemm_tile_override(*tile)
        fwd(c, x, w, y, saved, ws)
        bwd(c, x, w, saved, dy, dx, grads, accumulate, ws)
        torch.cuda.synchronize()
    finally:
        L.ls_gemm_tile_override(0, 0)
    return {"y": y.float() - x.float(), "dx": dx.float() - dy.float(),
            **{n: g - 0.25 if accumulate else g for n, g in grads.items()}}


@pytest.mark.parametrize("part,c,steps", INSTANCES, ids=lambda v: f"{v.tokens}x{v.hidden}x{v.intermediate}"
                         if isinstance(v, configs.BlockConfig) else v if isinstance(v, str) else "")
def test_instances(part, c, steps):
    """The automatic choice (accumulating) against forced 256 x 256 tiles (overwriting), which the
    oracle checks elsewhere, by the norm of every row and every column.

    Only the order of fp32 sums differs, so stored bf16 values round the other way here and
    there, each by at most their spacing, 2^-7 of themselves.  Sums over them (a row of an
    output) are off by at most that in norm where one term of the sum outweighs the rest, and
    by less where the roundings of many average out: 2^-6 is allowed, for two such steps.  An
    output stored with its residual (y, dx) rounds to the spacing of the sum, 2^-8 to 2^-7 of
    it and about 2^-8 in norm where every value flips.  A piece of 8 values (16 bytes) that is
    missing or misplaced moves the norm of a row or column of n values by sqrt(8 / n), over 2^-6
    for all n < 32768."""
    need_gpu()
    for step, (kernel, split) in steps.items():
        plan = step_plan(c, step)
        assert plan[:3] == kernel and (plan[3] > 1) == bool(split), (step, plan)
    say(f"instances {part} tokens={c.tokens} hidden={c.hidden} heads={c.n_q_heads}/{c.n_kv_heads}x{c.head_dim} "
        f"intermediate={c.intermediate}")
    host = inputs.make_inputs(c, seed_base=500, gamma="random", device="cuda")
    got = _run_sub_layer(part, c, host, (0, 0), True)
    want = _run_sub_layer(part, c, host, (256, 256), False)
    for n in want:
        a, b = got[n], want[n]
        res = {"y": host["x"], "dx": host["dy"]}.get(n)
        for dim in range(b.dim()):
            allowed = 2.0 ** -6 * b.norm(dim=dim)
            if res is not None:
                allowed += 2.0 ** -8 * res.view_as(b).float().norm(dim=dim)
            worst = float(((a - b).norm(dim=dim) / allowed).max())
            say(f"  {n} dim {dim}: {worst:.3f} of what is allowed")
            assert worst <= 1, n


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
