"""The forms of the GEMM and its tile map at the sizes where they can go wrong: ragged last tiles
and blocks in both directions, fewer K steps than waves, several Aux steps, rows of Y on and off
64-byte boundaries, even splits of the tiles over the XCDs.  Accumulators and Y against the CPU
oracle, all exact (Aux on its own scale: check_own_scale states the bound)."""
import numpy as np
import pytest
import torch

from gpu_common import B, check_case, check_mlp, check_own_scale, check_plain_y, orc, sample_rows, synth
from paper_2604_04701_amd.synth import Case

pytestmark = pytest.mark.gpu
U = (20.0, 100.0)

# M, K, N and the rows of the output tile of each form.
FORMS = {
    "direct 16x16": (100, 2112, 264, 16), "direct 16x32": (130, 520, 1000, 32), "direct 16x32, one K step": (70, 64, 72, 32),
    "direct 32x32": (333, 1032, 1096, 32), "direct 32x64": (500, 2112, 776, 64), "direct 64x64": (700, 1600, 1400, 64),
    "direct 64x64, long K": (390, 3008, 1992, 64), "direct 32x32, three on a CU": (31, 776, 16424, 32),
    # fewer K steps than waves (with several Aux steps: the list below), or not many more
    "direct 64x64, one K step": (1016, 64, 1024, 64), "direct 64x64, five K steps": (1024, 264, 1000, 64),
    "persistent 128, short K": (2049, 264, 776, 128), "persistent 128, one K step": (1536, 64, 1536, 128),
    # no more tiles than are worked on at one time: split evenly, or one block per XCD
    "persistent 128, even split": (2100, 520, 1544, 128), "persistent 128, block per XCD": (2245, 72, 1288, 128),
    "persistent 256, even split": (3077, 136, 4808, 256), "persistent 256, block per XCD": (4100, 72, 2560, 256),
    # several tiles per workgroup: blocks ragged in both directions (places without a tile are skipped), even splits
    "persistent 256, ragged blocks": (4743, 72, 4272, 256), "persistent 256, even split, more": (5222, 72, 4112, 256),
    "persistent 128, even split, more": (6607, 72, 2312, 128),
}


@pytest.mark.parametrize("x_gran,w_gran,bias_seed", [("tensor", "tensor", None), ("tensor", "channel", 5),
                                                     ("token", "channel", 6)])
@pytest.mark.parametrize("form", FORMS)
def test_gemm_forms(form, x_gran, w_gran, bias_seed):
    M, K, N, tile_rows = FORMS[form]
    assert B.lib().muxq_linear_gelu_slabs(M, K, N) == (M + tile_rows - 1) // tile_rows
    assert B.gemm_kernel(M, K, N) == {64: "k_gemm_i8_direct", 128: "k_gemm_i8_persist4", 256: "k_gemm_i8_persist8"}[max(tile_rows, 64)]
    case = Case("form", M, K, N, min(6, K // 8), U, 800 + M)
    if M * N <= 2000 * 1600:
        check_case(case, x_gran=x_gran, w_gran=w_gran, bias_seed=bias_seed)
    check_plain_y(case, x_gran=x_gran, w_gran=w_gran, bias_seed=bias_seed)


@pytest.mark.parametrize("M,N,tile_rows", [(4743, 4272, 256), (4096, 4104, 128)])
@pytest.mark.parametrize("x_gran,w_gran", [("tensor", "tensor"), ("token", "channel")])
def test_one_k_step_per_tile_and_several_tiles_per_workgroup(M, N, tile_rows, x_gran, w_gran):
    """The stream of K steps runs more than a tile ahead of the products: without Aux steps it needs the tile
    after the next, with one Aux step it changes phase at every step."""
    assert B.lib().muxq_linear_gelu_slabs(M, 64, N) == (M + tile_rows - 1) // tile_rows
    for r_cap in (0, 64):
        check_plain_y(Case("one_step", M, 64, N, 3, U, 880 + r_cap), x_gran=x_gran, w_gran=w_gran, r_cap=r_cap)


@pytest.mark.parametrize("x_gran", ["tensor", "token"])
@pytest.mark.parametrize("shape", [(100, 2112, 264), (130, 520, 1000), (333, 1032, 1096), (500, 2112, 776), (700, 1600, 1400),
                                   (1000, 200, 1024)], ids=lambda s: "x".join(map(str, s)))
def test_direct_forms_several_aux_steps_and_own_scale(shape, x_gran):
    M, K, N = shape
    assert B.gemm_kernel(M, K, N) == "k_gemm_i8_direct"
    check_case(Case("form_aux", M, K, N, 150, U, 820 + M), r_cap=192, e=3, x_gran=x_gran)
    X = np.random.default_rng(M).uniform(-5.0, 5.0, size=(M, K)).astype(np.float32)
    X[:, ::K // 8] *= 1.5
    W = (0.05 * np.random.default_rng(N).standard_normal((K, N))).astype(np.float16)
    check_own_scale(Case("form_own", M, K, N, 0, U, 0), X.astype(np.float16), W, x_gran=x_gran, w_gran="channel")


@pytest.mark.parametrize("shape", [(100, 2112, 264, 72), (333, 1032, 1096, 136), (700, 1600, 1400, 264)],
                         ids=lambda s: "x".join(map(str, s)))
def test_direct_forms_hand_the_column_maxima_over(shape):
    check_mlp(*shape, 840 + shape[0])


@pytest.mark.parametrize("w_gran,x_gran", [("tensor", "tensor"), ("channel", "token")])
@pytest.mark.parametrize("shape,tile_rows", [((1040, 1544, 48, 72), 16), ((2080, 72, 64, 136), 32), ((1041, 1600, 40, 24), 16)],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else f"tile_rows_{v}")
def test_more_than_64_rows_of_tiles(shape, tile_rows, w_gran, x_gran):
    """More rows of tiles than the next layer takes slabs: the column maxima come from a pass over H."""
    M, K, N, N2 = shape
    assert (M + tile_rows - 1) // tile_rows > 64
    assert B.gemm_kernel(M, K, N) == "k_gemm_i8_direct"
    n = check_mlp(M, K, N, N2, 850 + M, w_gran=w_gran, x_gran=x_gran)
    assert n <= 64 and n != (M + tile_rows - 1) // tile_rows


@pytest.mark.parametrize("N,ldy", [(4808, 4808), (4816, 4816), (4832, 4832), (4864, 4864), (4808, 4832), (4832, 4840)])
def test_rows_of_y_on_every_boundary(N, ldy):
    """Rows that start on 16-, 32-, 64- and 128-byte boundaries, by N and by the row stride; nothing past N."""
    rng = np.random.default_rng(N + ldy)
    M, K = 3077, 136
    X, _ = synth.make_x(M, K, 5, U, rng)
    W = synth.make_w(K, N, rng)
    out = torch.full((M, ldy), 7.0, dtype=torch.float16, device="cuda")
    w_q, w_s = B.muxq_quantize_weight(torch.from_numpy(W).cuda())
    B.muxq_linear(torch.from_numpy(X).cuda(), w_q, w_s, N, out=out[:, :N])
    rows = sample_rows(M, 200, 3)
    assert (out[:, :N].cpu().numpy()[rows] == orc.linear(X, W, rows=rows)["y16"]).all()
    assert (out[:, N:] == 7.0).all()


@pytest.mark.parametrize("M,K,N", [(300, 520, 7688), (500, 520, 7680), (129, 712, 16384), (1500, 520, 2056), (3000, 520, 776),
                                   (1000, 520, 3848), (2049, 520, 2056)])
def test_one_block_of_tiles_for_each_xcd(M, K, N):
    """The 128 x 128 form with no more tiles than CUs: eight blocks, ragged in either direction, and sizes
    with no such blocks."""
    check_plain_y(Case("xcd_blocks", M, K, N, 6, U, 860 + M), w_gran="channel", bias_seed=3)
