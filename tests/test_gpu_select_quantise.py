"""The quantisers that select the outlier channels for themselves (csrc/muxq_act.hip): pieces of a row
for 1 to 16 waves, rows fewer and more than the workgroups take at once, the abs-max pass with
narrow column blocks or X itself in its place, slabs of a producer below and above the limit,
lists fixed offline and lists the caller gives to the stage entry point.  All exact."""
import numpy as np
import pytest
import torch

import test_gpu_parity as T
from gpu_common import B, check_case, check_plain_y, compare, orc, run_gpu, sample_rows, synth
from paper_2604_04701_amd.synth import Case

pytestmark = pytest.mark.gpu
U = (20.0, 100.0)

SHAPES = [(65, 1032, 72), (66, 8192, 24), (300, 64, 72), (513, 520, 136), (700, 2056, 72), (1000, 1024, 264),
          (2100, 200, 72), (5000, 1032, 40), (257, 4104, 8200), (2051, 5128, 24), (70, 8200, 24)]   # the last one: the separate kernels


@pytest.mark.parametrize("x_gran", ["tensor", "token"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_select_and_quantise_all_stages(shape, x_gran):
    M, K, N = shape
    check_case(Case("act", M, K, N, min(9, K // 8), U, 900 + M), x_gran=x_gran, w_gran="channel")


@pytest.mark.parametrize("x_gran", ["tensor", "token"])
@pytest.mark.parametrize("r_cap,r", [(0, 5), (64, 0), (64, 64), (64, 90), (128, 100), (256, 200)])
def test_select_and_quantise_capacity(r_cap, r, x_gran):
    check_case(Case("act_cap", 333, 712, 136, r, U, 940 + r), r_cap=r_cap, e=3, x_gran=x_gran)


@pytest.mark.parametrize("threshold", [-1.0, -0.0, 0.0, 1e-40, 2.0 ** -25, 2.0 ** -24, 3.5e-5, 2.0 ** -14 - 2.0 ** -25, 2.0 ** -14, 6.0, 6.001,
                                       65503.9, 65504.0, 65519.0, 65520.0, 1e30, float("inf")])
@pytest.mark.parametrize("M", [3, 300])
def test_thresholds(M, threshold):
    """The threshold is any binary32 value, also between two fp16 values, below the smallest or above the largest
    one (the kernels compare fp16 magnitudes with the largest one that is not over it)."""
    X, W, _ = synth.make_case(Case("act_thr", M, 200, 72, 4, U, 980))
    X[:, :8] = 0
    X[0, 1:8] = [2.0 ** -24, 2.0 ** -23, 3.4e-5, 3.6e-5, 6.0, 6.0039, 65504.0]
    X[M - 1, 8:10] = [-6.0, -6.0039]
    kw = dict(threshold=threshold, r_cap=256)
    compare(run_gpu(X, W, **kw), orc.linear(X, W, **kw), 200, 72, 256)


# one scale per row: single rows (2 x 64 chunks to a wave), and 4 rows at a time in pieces of 4 and of 5 x 16 chunks, each with one
# wave to the rows and with several, whole pieces and K padding, M off the groups of 4
ROW_SHAPES = [(40, 1024, 24), (70, 3080, 24), (255, 8192, 24), (8195, 512, 24), (6001, 1032, 24), (2003, 5120, 24), (5002, 640, 24),
              (9001, 600, 24), (12001, 1280, 24), (9999, 8, 24),
              # several steps with rows up to 4 KB: single rows, and 4 rows in one wave and in several, spread evenly over the steps or
              # with a last step of few rows
              (9001, 1000, 24), (16390, 640, 24), (16400, 240, 24), (5125, 1536, 24), (5001, 2040, 24), (12289, 1024, 24)]


@pytest.mark.parametrize("shape", ROW_SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_rows_of_each_form(shape):
    M, K, N = shape
    check_case(Case("act_rows", M, K, N, min(9, K // 8), U, 990), x_gran="token")
    case = Case("act_rows_static", M, K, N, min(5, K // 8), U, 991)
    if M * K < 10_300_000:
        T._check_static(case, [int(k) for k in synth.make_case(case)[2]], "token", "channel", with_bias=True)


@pytest.mark.parametrize("M,K", [(40, 1024), (6001, 520), (9001, 600), (9001, 1000), (5125, 1536)])
def test_rows_with_nan_and_infinity(M, K):
    """A NaN sets no scale (and hides its channel from the list), an infinity makes its row's scale infinite; the codes
    and scales of all other rows are those of the list that results, by the formulas in binary32."""
    X, W, ch = synth.make_case(Case("act_nan", M, K, 24, 3, U, 992))
    hit = [(5, (int(ch[0]) + 1) % K, np.nan), (9, (int(ch[1]) + 1) % K, np.inf), (M - 1, int(ch[2]), np.nan)]
    for r, k, v in hit:
        X[r, k] = v
    got = run_gpu(X, W, x_gran="token", finite=False)
    lst = got["outlier_idx"][:got["n_outliers"][0]]
    assert lst.tolist() == sorted([int(ch[0]), int(ch[1]), hit[1][1]])
    mult = np.ones(K, np.float32)
    mult[lst] = 0.25
    amax = np.nanmax(np.abs(X.astype(np.float32)) * mult, axis=1)
    s_x, inv = amax / np.float32(127), np.float32(127) / amax
    assert (got["x_scale"][0] == s_x).all() and (got["x_scale"][1] == inv).all()
    rows = np.ones(M, bool)
    rows[[5, 9, M - 1]] = False
    want = np.clip(np.rint(X[rows].astype(np.float32) * (inv[rows, None] * mult)), -127, 127)
    assert (got["body_q"][rows][:, :K] == want).all() and (got["aux_q"][rows][:, :len(lst)] == want[:, lst]).all()


@pytest.mark.parametrize("x_gran", ["tensor", "token"])
def test_select_and_quantise_static_lists(x_gran):
    for M, K, N in ((70, 2056, 72), (900, 264, 264)):
        case = Case("act_static", M, K, N, 5, U, 960 + M)
        _, _, planted = synth.make_case(case)
        for lst in ([int(k) for k in planted], [], list(range(0, 200, 2))):
            T._check_static(case, lst, x_gran, "channel", with_bias=True)


def test_given_lists_need_not_ascend_and_any_binary32_maxima():
    """muxq_build_aux: the list in any order, maxima that are no fp16 values."""
    rng = np.random.default_rng(3)
    for M, K in ((5, 72), (300, 1032), (1030, 4096), (130, 8192), (40, 8200)):
        X, ch = synth.make_x(M, K, 6, U, rng)
        lst = np.array([ch[3], ch[0], 1, ch[5]], dtype=np.int32)
        _, first = np.unique(lst, return_index=True)
        lst = lst[np.sort(first)]
        Xd = torch.from_numpy(X).cuda()
        cm, _, _ = B.muxq_detect_outliers(Xd)
        cm = cm * 1.0009765
        idx = torch.full((64,), -1, dtype=torch.int32, device="cuda")
        idx[:len(lst)] = torch.from_numpy(lst).cuda()
        n = torch.tensor([len(lst), len(lst)], dtype=torch.int32, device="cuda")
        body, aux, xs = B.muxq_build_aux(Xd, cm, idx, n, 64, 2)
        mult = np.ones(K, np.float32)
        mult[lst] = 0.25
        amax = (cm.cpu().numpy()[:K] * mult).max()
        inv = np.float32(127.0) / amax
        assert xs.cpu().numpy().tolist() == [amax / np.float32(127.0), inv]
        want = np.clip(np.rint((X.astype(np.float32) * mult) * inv), -127, 127).astype(np.int8)
        got = B.unpack(body, M, B.k_pad(K)).cpu().numpy()
        assert (got[:, :K] == want).all() and (got[:, K:] == 0).all()
        ga = B.unpack(aux, M, 64).cpu().numpy()
        assert (ga[:, :len(lst)] == want[:, lst]).all() and (ga[:, len(lst):] == 0).all()


@pytest.mark.parametrize("M,K,N", [(333, 200, 264), (2049, 1032, 72), (700, 4096, 72)])
def test_slabs_of_a_producer(M, K, N):
    """The maxima left by the GELU kernel, few enough to be folded by every workgroup or not."""
    rng = np.random.default_rng(M)
    Y = torch.from_numpy((3.0 * rng.standard_normal((M, K))).astype(np.float16)).cuda()
    W = synth.make_w(K, N, rng)
    w_q, w_s = B.muxq_quantize_weight(torch.from_numpy(W).cuda())
    ws, lay = B.alloc_workspace(M, K, N, 64), B.workspace_layout(M, K, N, 64)
    ws.fill_(0xCD)
    X = B.muxq_gelu_absmax(Y, ws, lay)
    for x_gran in ("tensor", "token"):
        Yg = B.muxq_linear(X, w_q, w_s, N, workspace=ws, absmax_ready=True, x_gran=x_gran)
        o = orc.linear(X.cpu().numpy(), W, x_gran=x_gran)
        assert (Yg.cpu().numpy() == o["y16"]).all()
        B.muxq_gelu_absmax(Y, ws, lay)


@pytest.mark.parametrize("M,K", [(96_001, 968), (96_001, 1032), (24_001, 4096)])
def test_x_beyond_the_caches(M, K):
    """X of 186 to 198 MB, on both sides of the line to the separate kernels; codes, lists and scales over all
    rows, accumulators and Y on a sample."""
    case = Case("act_big", M, K, 24, 7, U, 970)
    check_case(case, rows=sample_rows(M, 40, 2))


@pytest.mark.parametrize("M,K", [(140_001, 1032), (150_001, 1032), (61_001, 4096), (62_001, 4096), (30_001, 5128), (140_001, 248)])
def test_stages_on_x_beyond_the_caches(M, K):
    """The stage entry points on both sides of their lines, against the same formulas in binary32 (every step is exact
    or correctly rounded here as well: the scales by numpy, the codes by torch on the GPU)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(M + K)
    X = torch.randn(M, K, generator=g, device="cuda", dtype=torch.float16).clamp_(-5.5, 5.5)      # none over 6 by chance
    lst = torch.tensor([3, 40, K - 2], device="cuda")
    X[:, lst] *= 30
    cm, idx, n = B.muxq_detect_outliers(X)
    assert torch.equal(cm, X.abs().amax(0).float())
    assert n.tolist() == [3, 3] and idx[:3].tolist() == lst.tolist() and (idx[3:] == -1).all()
    body, aux, xs = B.muxq_build_aux(X, cm, idx, n, 64, 2)
    mult = torch.ones(K, device="cuda")
    mult[lst] = 0.25
    amax = np.float32((cm * mult).amax().item())
    inv = float(np.float32(127.0) / amax)
    assert xs.tolist() == [float(amax / np.float32(127.0)), inv]
    got = B.unpack(body, M, B.k_pad(K))
    for r0 in range(0, M, 16384):
        want = ((X[r0:r0 + 16384].float() * mult) * inv).round_().clamp_(-127, 127).to(torch.int8)
        assert torch.equal(got[r0:r0 + 16384, :K], want)
        assert torch.equal(B.unpack(aux, M, 64)[r0:r0 + 16384, :3], want[:, lst])
    assert (got[:, K:] == 0).all() and (B.unpack(aux, M, 64)[:, 3:] == 0).all()
