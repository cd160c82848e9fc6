"""Calls with few tokens, which run as one launch (csrc/muxq_few.hip): every workspace region, the
accumulators and Y against the CPU oracle at the edges of that kernel's ranges -- one row and
the largest row counts, partial 16-row blocks, the shortest and longest K, fewer and more
blocks of 16 output channels than workgroups, list capacities, lists fixed offline, and the
column maxima it hands from layer to layer.  All comparisons are exact (check_mlp states the
one tolerance, that of the GELU)."""
import numpy as np
import pytest
import torch

import test_gpu_parity as T
from gpu_common import B, check_case, check_mlp, check_plain_y, orc, run_gpu, synth
from paper_2604_04701_amd.synth import Case

pytestmark = pytest.mark.gpu
U = (20.0, 100.0)

SHAPES = [(1, 8, 8), (1, 768, 2304), (1, 8192, 520), (2, 72, 24), (15, 4096, 136), (16, 1280, 1288),
          (17, 1000, 264), (24, 5120, 264), (31, 512, 8200), (33, 136, 520), (48, 2048, 72), (64, 64, 16),
          (64, 1024, 264),
          # workgroups of 15, 14, 9 and 13 waves: a row in 5, 7, 9 and 13 pieces
          (3, 2400, 72), (3, 3400, 264), (2, 4360, 72), (5, 6400, 136),
          # the same rows with more blocks of output channels than CUs: 16 waves, of which 1, 2, 7 and 3 hold no row
          (3, 2400, 4104), (2, 3400, 6424), (1, 4360, 4120), (1, 6400, 6424),
          # three pieces to a row: two workgroups of 6 waves on a CU, and 12 waves that walk over N
          (1, 1032, 4104), (4, 1536, 8216), (5, 1032, 4104), (6, 1536, 8200),
          # rows of four pieces and of more beyond N = 16384: 16 waves
          (5, 1544, 16392), (9, 2048, 16456), (9, 2064, 16392),
          # either side of the line to the separate launches: rows in turn, elements with one scale per token, the walk over N
          (7, 5120, 136), (8, 5120, 136), (6, 4400, 72), (6, 4480, 72), (16, 768, 12280), (20, 768, 12280)]
# those of them beyond that line, with one scale per call and per token
SEPARATE = [(15, 4096, 136), (24, 5120, 264), (48, 2048, 72), (64, 1024, 264)]
SEPARATE_TOKEN = SEPARATE + [(64, 64, 16), (5, 6400, 136), (7, 5120, 136), (8, 5120, 136), (6, 4480, 72), (20, 768, 12280)]


@pytest.mark.parametrize("x_gran,w_gran", [("tensor", "tensor"), ("tensor", "channel"), ("token", "channel")])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_few_tokens_all_stages(shape, x_gran, w_gran):
    M, K, N = shape
    assert (B.code_kernel(M, K, N, x_gran=x_gran) == "k_linear_few") == (shape not in (SEPARATE if x_gran == "tensor" else SEPARATE_TOKEN))
    case = Case("few", M, K, N, min(6, K // 8), U, 600 + M)
    check_case(case, x_gran=x_gran, w_gran=w_gran, bias_seed=M if M % 2 else None)
    check_plain_y(case, x_gran=x_gran, w_gran=w_gran, bias_seed=3)


@pytest.mark.parametrize("x_gran", ["tensor", "token"])
@pytest.mark.parametrize("r_cap,r", [(0, 5), (64, 0), (64, 64), (64, 90), (128, 100), (256, 200)])
def test_few_tokens_list_capacity(r_cap, r, x_gran):
    for M, e in ((3, 1), (20, 3)):
        check_case(Case("few_cap", M, 520, 136, r, U, 640 + M), r_cap=r_cap, e=e, x_gran=x_gran)


@pytest.mark.parametrize("x_gran", ["tensor", "token"])
@pytest.mark.parametrize("shape", [(33, 136, 520), (48, 512, 72), (64, 248, 264), (24, 1400, 136), (1, 1600, 6416), (4, 2048, 8200)],
                         ids=lambda s: "x".join(map(str, s)))
def test_few_tokens_long_capacity_and_many_blocks(shape, x_gran):
    """Capacities above 64, with which more rows stay in the one launch (three and four blocks of 16 of them), and more blocks
    of 16 output channels than CUs with few rows, for which two workgroups share a CU."""
    M, K, N = shape
    for r_cap in (64, 128):
        check_case(Case("few_rows", M, K, N, min(80, K // 8), U, 690 + M), r_cap=r_cap, x_gran=x_gran, w_gran="channel", bias_seed=4)


@pytest.mark.parametrize("x_gran,w_gran", [("tensor", "channel"), ("token", "tensor")])
def test_few_tokens_static_lists(x_gran, w_gran):
    for M, K, N in ((1, 264, 136), (24, 5120, 72), (50, 1032, 264)):
        case = Case("few_static", M, K, N, 5, U, 660 + M)
        _, _, planted = synth.make_case(case)
        _lists = ([int(k) for k in planted], [], list(range(0, 200, 2)), [3, 7, 7, K + 1])
        for lst in _lists:
            T._check_static(case, lst, x_gran, w_gran, with_bias=M > 1)


@pytest.mark.parametrize("w_gran,x_gran", [("tensor", "tensor"), ("channel", "token")])
@pytest.mark.parametrize("M,K,N1,N2", [(1, 64, 256, 64), (8, 1280, 5120, 1280), (17, 264, 1048, 264),
                                       (64, 768, 1000, 768), (40, 72, 4104, 72)])
def test_few_tokens_mlp(M, K, N1, N2, w_gran, x_gran):
    check_mlp(M, K, N1, N2, 700 + M, w_gran=w_gran, x_gran=x_gran)


def test_few_tokens_strided_rows_and_the_static_array():
    """Row strides above the row length; the entry point without a workspace; the same
    workspace for calls of shrinking size."""
    dev = "cuda"
    rng = np.random.default_rng(5)
    for M, K, N in ((24, 1280, 520), (3, 200, 72)):
        X, _ = synth.make_x(M, K, 4, U, rng)
        W = synth.make_w(K, N, rng)
        Xd = torch.zeros((M, K + 24), dtype=torch.float16, device=dev)[:, :K]
        Xd.copy_(torch.from_numpy(X))
        out = torch.full((M, N + 16), 7.0, dtype=torch.float16, device=dev)
        w_q, w_s = B.muxq_quantize_weight(torch.from_numpy(W).to(dev))
        B.muxq_linear(Xd, w_q, w_s, N, out=out[:, :N])
        y = B.muxq_linear_noalloc(Xd, w_q, w_s, N)
        o = orc.linear(X, W)
        assert (out[:, :N].cpu().numpy() == o["y16"]).all() and (out[:, N:] == 7.0).all()
        assert (y.cpu().numpy() == o["y16"]).all()


def test_y_in_the_place_of_x():
    """Y may take X's memory (K = N): no workgroup may store before all have read."""
    rng = np.random.default_rng(9)
    M, K = 16, 1280
    X, _ = synth.make_x(M, K, 4, U, rng)
    W = synth.make_w(K, K, rng)
    w_q, w_s = B.muxq_quantize_weight(torch.from_numpy(W).cuda())
    o = orc.linear(X, W)
    for _ in range(5):
        Xd = torch.from_numpy(X).cuda()
        assert (B.muxq_linear(Xd, w_q, w_s, K, out=Xd).cpu().numpy() == o["y16"]).all()


@pytest.mark.parametrize("M,K,N", [(8, 1280, 264), (300, 1032, 136), (70, 4096, 72)])
def test_a_nan_does_not_hide_the_other_channels(M, K, N):
    """One scale per call: a NaN in one row of a quiet channel leaves the other rows as they are
    with a zero in its place (its channel's maximum is not a number and sets no scale)."""
    X, ch = synth.make_x(M, K, 4, U, np.random.default_rng(M))
    c = next(k for k in range(5, K) if k not in set(ch.tolist()))
    X[0, c] = 0
    W = synth.make_w(K, N, np.random.default_rng(K))
    o = orc.linear(X, W)
    Xn = X.copy()
    Xn[0, c] = np.nan
    w_q, w_s = B.muxq_quantize_weight(torch.from_numpy(W).cuda())
    y = B.muxq_linear(torch.from_numpy(Xn).cuda(), w_q, w_s, N).cpu().numpy()
    assert (y[1:] == o["y16"][1:]).all()


@pytest.mark.parametrize("M,K,N", [(8, 1280, 264), (40, 520, 72), (300, 1032, 136), (70, 4096, 72), (300, 200, 72)])
@pytest.mark.parametrize("r", [0, 4])
def test_a_nan_does_not_hide_the_other_channels_of_its_row(M, K, N, r):
    """One scale per token: a NaN in a quiet channel sets no scale itself, and its row keeps the scale
    and the codes of the other channels, with listed channels in the row and without."""
    X, ch = synth.make_x(M, K, r, U, np.random.default_rng(M + r))
    W = synth.make_w(K, N, np.random.default_rng(K))
    quiet = [k for k in range(K) if k not in set(ch.tolist())]
    where = [(0, quiet[5]), (M - 1, quiet[-3])]
    X0, Xn = X.copy(), X.copy()
    for m, k in where:
        X0[m, k] = 0
        Xn[m, k] = -np.float16("nan") if m else np.float16("nan")
    g = run_gpu(Xn, W, x_gran="token", finite=False)
    o = orc.linear(X0, W, x_gran="token")
    assert g["n_outliers"].tolist() == [o["n_used"], o["n_total"]]
    assert (g["x_scale"][0] == o["s_x"]).all() and (g["x_scale"][1] == o["inv_x"]).all()
    keep = np.ones((M, K), bool)
    for m, k in where:
        keep[m, k] = False
    assert (g["body_q"][:, :K] == o["body_q"])[keep].all()
    assert (g["Y"][1:M - 1] == o["y16"][1:M - 1]).all()


@pytest.mark.parametrize("x_gran", ["tensor", "token"])
@pytest.mark.parametrize("M,K,N1,N2", [(8, 2560, 1280, 264), (8, 64, 1000, 72), (8, 264, 1048, 264),
                                       (333, 64, 1000, 136), (333, 1032, 520, 72), (2100, 64, 3000, 72)])
def test_one_workspace_for_both_layers(M, K, N1, N2, x_gran):
    """The column maxima for the next layer may lie inside the workspace of this one, on whatever its
    layout has there: results as with two workspaces."""
    rng = np.random.default_rng(M + K)
    X, _ = synth.make_x(M, K, 4, U, rng)
    Xd = torch.from_numpy(X).cuda()
    wq1, ws1 = B.muxq_quantize_weight(torch.from_numpy(synth.make_w(K, N1, rng)).cuda())
    wq2, ws2 = B.muxq_quantize_weight(torch.from_numpy(synth.make_w(N1, N2, rng)).cuda())
    lay2 = B.workspace_layout(M, N1, N2, 64)
    n1, n2 = B.workspace_bytes(M, K, N1, 64), B.workspace_bytes(M, N1, N2, 64)

    def run(first, second):
        H, n = B.muxq_linear_gelu(Xd, wq1, ws1, N1, workspace=first, next_workspace=second, next_layout=lay2, x_gran=x_gran)
        return H, B.muxq_linear(H, wq2, ws2, N2, workspace=second, absmax_ready=True, absmax_slabs=n, x_gran=x_gran)

    H, Y = run(torch.empty(n1, dtype=torch.uint8, device="cuda"), torch.empty(n2, dtype=torch.uint8, device="cuda"))
    one = torch.empty(max(n1, n2), dtype=torch.uint8, device="cuda")
    for _ in range(5):
        one.fill_(0x5A)
        H1, Y1 = run(one, one)
        assert torch.equal(H, H1) and torch.equal(Y, Y1)


@pytest.mark.parametrize("x_gran", ["tensor", "token"])
@pytest.mark.parametrize("M,K,N", [(16, 2624, 4360), (20, 2048, 24576), (24, 1536, 4360), (32, 1024, 12288), (33, 992, 264),
                                   (40, 816, 264), (48, 512, 8192), (64, 512, 8192)])
def test_longest_rows_and_widest_outputs(M, K, N, x_gran):
    """The longest rows that each number of tokens can run with in the one launch (every weight block of a wave is held), the
    widest outputs, and one row more, eight channels more of either, whichever launches the line gives them to."""
    check_case(Case("few_longest", M, K, N, 5, U, 680 + M), x_gran=x_gran, w_gran="channel", bias_seed=2)
    if N in (8192, 12288, 24576):
        check_plain_y(Case("few_wider", M, K, N + 8, 5, U, 690 + M), x_gran=x_gran, w_gran="channel")
    else:
        check_case(Case("few_longer", M + 1, K + 8, N, 5, U, 690 + M), x_gran=x_gran, w_gran="channel")


# (M, K, N), then what makes it a call for the separate launches: one row ("M"), eight channels of K or of N more
LIMITS = {
    (64, "tensor"): [(8, 5328, 264, "MK"), (16, 2648, 264, "MK"), (20, 2104, 136, "MK"), (24, 1536, 264, "MK"), (32, 1024, 264, "MK"),
                     (33, 992, 264, "MK"), (40, 816, 264, "MK"), (64, 512, 264, "MK"), (9, 2560, 8192, "MK"), (24, 1024, 12288, "MKN"),
                     (48, 512, 8192, "MKN"), (1, 4096, 12288, "N"), (4, 2048, 16384, "MK"), (1, 1544, 24576, "N")],
    (64, "token"): [(4, 8192, 264, "MK"), (8, 3328, 264, "MK"), (12, 2560, 264, "MK"), (16, 1664, 264, "MK"), (24, 1024, 264, "MK"),
                    (48, 512, 264, "MK"), (2, 6144, 8192, "MK"), (6, 2048, 8192, "MK"), (16, 1024, 12288, "KN"), (48, 512, 8192, "MKN")],
    (128, "tensor"): [(16, 2608, 4360, "MK"), (20, 2048, 24576, "MKN"), (24, 1536, 4360, "MK"), (32, 1024, 12288, "MKN"), (40, 816, 264, "MK"),
                      (48, 512, 8192, "KN"), (64, 512, 8192, "MKN")],
    (128, "token"): [(16, 2608, 4360, "MK"), (20, 2048, 24576, "MKN"), (24, 1536, 4360, "MK"), (32, 1024, 12288, "MKN"), (48, 512, 8192, "MKN")],
}


@pytest.mark.parametrize("r_cap,x_gran,M,K,N,ends", [(r, g, *s) for (r, g), shapes in LIMITS.items() for s in shapes])
def test_ends_of_the_one_launch(r_cap, x_gran, M, K, N, ends):
    """The longest rows that each number of tokens runs with (with capacities above 64 every weight block of a wave is held and LDS is
    full), the widest outputs; one row more, eight channels more take the separate launches."""
    beyond = [(M + (e == "M"), K + 8 * (e == "K"), N + 8 * (e == "N")) for e in ends]
    assert B.code_kernel(M, K, N, r_cap, x_gran) == "k_linear_few"
    assert all(B.code_kernel(*s, r_cap, x_gran) != "k_linear_few" for s in beyond)
    kw = dict(x_gran=x_gran, w_gran="channel", r_cap=r_cap)
    check = check_plain_y if K * N > 10_000_000 else check_case        # (every stage, unless the weight is large)
    check(Case("few_longest", M, K, N, 70 if r_cap > 64 else 5, U, 680 + M), bias_seed=2, **kw)
    if N < 16384:
        check(Case("few_longer", *beyond[-1], 5, U, 690 + M), **kw)
