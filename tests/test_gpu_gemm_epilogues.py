"""The epilogues of the persistent GEMM, one kernel for each combination of scales, bias, zero point, GELU and way
of storing Y, on partial tiles in both directions and several tiles per workgroup.  Y against the CPU oracle, exact
(the order of binary32 operations is the same on both sides)."""
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

from gpu_common import B, check_case, check_mlp, check_own_scale, check_plain_y, orc, rows_every_block, sample_rows, say, synth
from paper_2604_04701_amd.synth import Case

pytestmark = pytest.mark.gpu
U = (20.0, 100.0)
# more tiles than workgroups are resident (512 of 128 x 128 and 128 x 256, 256 of 256 x 256), partial in both directions
FORMS = {"128x128": (6607, 72, 2312), "256x256": (5222, 72, 4112), "128x256": (3400, 520, 6304)}
FAR = {"128x128": (129, 712, 16384), "256x256": (200, 264, 65536), "128x256": (129, 2048, 32768)}
KERNELS = {"128x128": "k_gemm_i8_persist4", "256x256": "k_gemm_i8_persist8", "128x256": "k_gemm_i8_persist_half"}


@pytest.mark.parametrize("form", FORMS)
def test_the_shapes_below_take_the_kernels_they_are_listed_for(form):
    (M, K, N), (m, k, n) = FORMS[form], FAR[form]
    assert B.gemm_kernel(M, K, N) == B.gemm_kernel(m, k, n) == KERNELS[form]
    tn, tm = (int(x) for x in form.split("x"))
    assert -(-N // tn) * -(-M // tm) > (256 if form == "256x256" else 512)


def row_strides(N):
    """On 128-byte lines, where Y goes out as a stream, and off 64 bytes, where it goes through L2."""
    return (N + 63) // 64 * 64, N + 8 if (N + 8) % 32 else N + 16


@pytest.mark.parametrize("on_lines", [True, False])
@pytest.mark.parametrize("bias_seed", [None, 7])
@pytest.mark.parametrize("w_gran", ["tensor", "channel"])
@pytest.mark.parametrize("x_gran", ["tensor", "token", "naive"])
@pytest.mark.parametrize("form", FORMS)
def test_every_combination_of_scales_and_bias(form, x_gran, w_gran, bias_seed, on_lines):
    """Rows of Y on 128-byte lines (stored as a stream) and off them (through L2, in another order); nothing past N.
    naive: the plain INT8 pipeline, whose zero point is 0."""
    M, K, N = FORMS[form]
    rows = rows_every_block(M, 11)
    X, W, _ = synth.make_case(Case("epilogue", M, K, N, 5, U, 900 + M))
    bias = None if bias_seed is None else np.random.default_rng(bias_seed).standard_normal(N).astype(np.float16)
    bd = None if bias is None else torch.from_numpy(bias).cuda()
    Xd = torch.from_numpy(X).cuda()
    w_q, w_s = B.muxq_quantize_weight(torch.from_numpy(W).cuda(), w_gran)
    ldy = row_strides(N)[0 if on_lines else 1]
    out = torch.full((M, ldy), 7.0, dtype=torch.float16, device="cuda")
    say(f"[epilogue] {form} x={x_gran} w={w_gran} bias={bias_seed} ldy={ldy}")
    if x_gran == "naive":
        B.muxq_linear_naive_int8(Xd, w_q, w_s, N, w_gran, bias=bd, out=out[:, :N])
        o = orc.linear(X, W, r_cap=0, w_gran=w_gran, bias16=bias, rows=rows)
    else:
        B.muxq_linear(Xd, w_q, w_s, N, w_gran, bias=bd, out=out[:, :N], x_gran=x_gran)
        o = orc.linear(X, W, w_gran=w_gran, bias16=bias, rows=rows, x_gran=x_gran)
    got = out.cpu().numpy()
    assert (got[rows][:, :N] == o["y16"]).all()
    assert (got[:, N:] == 7.0).all()


@pytest.mark.parametrize("on_lines", [True, False])
@pytest.mark.parametrize("bias_seed", [None, 9])
@pytest.mark.parametrize("w_gran", ["tensor", "channel"])
@pytest.mark.parametrize("form", FORMS)
def test_gemm_on_codes_without_a_zero_point(form, w_gran, bias_seed, on_lines):
    """muxq_gemm_i8 on codes of the full range, with Aux steps and without: Y is the product of the codes, exact."""
    M, K, N = FORMS[form]
    rng = np.random.default_rng(M + N)
    rows = np.array(rows_every_block(M, 13))
    kp = B.k_pad(K)
    a = rng.integers(-127, 128, (M, kp), dtype=np.int8)
    aux = rng.integers(-127, 128, (M, 64), dtype=np.int8)
    w_aux = rng.integers(-127, 128, (N, 64), dtype=np.int8)
    a[:, K:] = 0
    aux[:, 5:] = 0
    w_q, w_s = B.muxq_quantize_weight(torch.from_numpy(synth.make_w(K, N, rng)).cuda(), w_gran)
    wn = B.unpack(w_q, N, kp).cpu().numpy()
    bias = None if bias_seed is None else np.random.default_rng(bias_seed).standard_normal(N).astype(np.float16)
    sx = np.float32(0.013)
    dev = lambda t: torch.from_numpy(t).cuda()
    ldy = row_strides(N)[0 if on_lines else 1]
    say(f"[gemm] {form} w={w_gran} bias={bias_seed} ldy={ldy}")
    for with_aux in (False, True):
        out = torch.full((M, ldy), 7.0, dtype=torch.float16, device="cuda")
        extra = dict(aux_q=B.pack(dev(aux)), w_aux=B.pack(dev(w_aux)), r_cap=64, exp=3,
                     n_outliers=torch.tensor([5, 5], dtype=torch.int32, device="cuda")) if with_aux else {}
        B.muxq_gemm_i8(B.pack(dev(a)), M, K, w_q, N, torch.tensor([sx, 1 / sx], device="cuda"), w_s, w_gran,
                       bias=None if bias is None else dev(bias), out=out[:, :N], **extra)
        # whole numbers below 2^53: exact in binary64
        acc = a[rows].astype(np.float64) @ wn.T.astype(np.float64)
        if with_aux:
            acc += 7.0 * (aux[rows].astype(np.float64) @ w_aux.T.astype(np.float64))
        y = (sx * w_s.cpu().numpy()) * acc.astype(np.float32)
        want = (y if bias is None else y + bias.astype(np.float32)).astype(np.float16)
        got = out.cpu().numpy()
        assert (got[rows][:, :N] == want).all()
        assert (got[:, N:] == 7.0).all()


@pytest.mark.parametrize("M,K,N", [(1500, 264, 2056), (3400, 520, 6304)])
@pytest.mark.parametrize("w_gran,x_gran", [("tensor", "tensor"), ("channel", "tensor"), ("tensor", "token"), ("channel", "token")])
def test_gelu_with_every_kind_of_scales(w_gran, x_gran, M, K, N):
    check_mlp(M, K, N, 136, 910, w_gran=w_gran, x_gran=x_gran)


@pytest.mark.parametrize("w_gran,x_gran", [("tensor", "tensor"), ("channel", "tensor"), ("tensor", "token"), ("channel", "token")])
@pytest.mark.parametrize("form", FORMS)
def test_gelu_without_a_bias(form, w_gran, x_gran):
    """The first layer against the oracle, exact; the fused GELU against the stand-alone one on the fp16 values the
    layer stores, bit for bit, and within one unit of the oracle's; its column maxima."""
    M, K, N = FORMS[form]
    rows = rows_every_block(M, 14)
    X, W, _ = synth.make_case(Case("gelu", M, K, N, 5, U, 960 + M))
    Xd = torch.from_numpy(X).cuda()
    w_q, w_s = B.muxq_quantize_weight(torch.from_numpy(W).cuda(), w_gran)
    say(f"[gelu] {form} x={x_gran} w={w_gran}")
    o = orc.linear(X, W, w_gran=w_gran, x_gran=x_gran, rows=rows)
    Y = B.muxq_linear(Xd, w_q, w_s, N, w_gran, x_gran=x_gran)
    assert (Y.cpu().numpy()[rows] == o["y16"]).all()
    lay = B.workspace_layout(M, N, 8, 64)
    ws, ws2 = B.alloc_workspace(M, N, 8, 64), B.alloc_workspace(M, N, 8, 64)
    H, n_slabs = B.muxq_linear_gelu(Xd, w_q, w_s, N, w_gran, x_gran=x_gran, next_workspace=ws, next_layout=lay)
    assert torch.equal(H.view(torch.int16), B.muxq_gelu_absmax(Y, ws2, lay).view(torch.int16))
    slabs = ws[lay.absmax_partial:lay.absmax_partial + n_slabs * lay.k_pad * 2].view(torch.float16).view(n_slabs, -1)
    assert torch.equal(slabs.amax(dim=0)[:N], H.abs().amax(dim=0))
    got, want = H.cpu().numpy()[rows], orc.gelu_tanh(o["y16"])
    assert np.abs(got.view(np.int16).astype(np.int32) - want.view(np.int16).astype(np.int32)).max() <= 1


@pytest.mark.parametrize("M,K,N", [(8190, 2120, 1016), (3400, 520, 6304), (8300, 4104, 2312)])
def test_128x256_tiles(M, K, N):
    """One tile per CU, ragged in both directions; several Aux steps; two tiles for some workgroups and K = 65 steps."""
    rows = rows_every_block(M, 12)
    check_plain_y(Case("half", M, K, N, 150, U, 930 + K), rows=rows, w_gran="channel", bias_seed=3, r_cap=192)
    check_case(Case("half", M, K, N, 3, U, 931 + K), rows=sample_rows(M, 40, 2))


@pytest.mark.parametrize("w_gran,x_gran", [("tensor", "tensor"), ("channel", "tensor"), ("tensor", "token"), ("channel", "token")])
@pytest.mark.parametrize("bias_seed", [None, 8])
@pytest.mark.parametrize("form", FORMS)
def test_aux_on_its_own_scale_with_every_kind_of_scales(form, w_gran, x_gran, bias_seed):
    """With the accumulators exported (a kernel of its own) against the oracle; without, as a program calls it, the same Y."""
    M, K, N = FORMS[form]
    case = Case("epilogue_own", M, K, N, 6, U, 920 + M)
    g, _ = check_own_scale(case, rows=rows_every_block(M, 15), w_gran=w_gran, x_gran=x_gran, bias_seed=bias_seed)
    X, W, _ = synth.make_case(case)
    bias = None if bias_seed is None else torch.from_numpy(np.random.default_rng(bias_seed).standard_normal(N).astype(np.float16)).cuda()
    w_q, w_s = B.muxq_quantize_weight(torch.from_numpy(W).cuda(), w_gran)
    for ldy in row_strides(N):
        out = torch.full((M, ldy), 7.0, dtype=torch.float16, device="cuda")
        B.muxq_linear(torch.from_numpy(X).cuda(), w_q, w_s, N, w_gran, bias=bias, out=out[:, :N], x_gran=x_gran, aux_scale="own")
        got = out.cpu().numpy()
        assert (got[:, :N] == g["Y"]).all() and (got[:, N:] == 7.0).all()


@pytest.mark.parametrize("form,ldy", [("128x128", (1 << 25) - 8), ("128x128", 1 << 25), ("128x128", (1 << 28) - 64),
                                      ("128x128", (1 << 28) - 56), ("256x256", (1 << 28) - 64), ("256x256", 1 << 28),
                                      ("128x256", (1 << 28) - 64), ("128x256", 1 << 28)])
def test_rows_of_y_far_apart(form, ldy):
    """Row strides up to what a buffer's 32-bit offsets reach, and beyond it; 70 to 110 GB that are not touched in between.
    The fused GELU against the same call with rows next to each other."""
    M, K, N = FAR[form]
    torch.cuda.empty_cache()
    rng = np.random.default_rng(ldy)
    X, _ = synth.make_x(M, K, 5, U, rng)
    W = synth.make_w(K, N, rng)
    Xd = torch.from_numpy(X).cuda()
    out = torch.empty((M, ldy), dtype=torch.float16, device="cuda")
    out[:, N:N + 64] = 7.0
    w_q, w_s = B.muxq_quantize_weight(torch.from_numpy(W).cuda())
    B.muxq_linear(Xd, w_q, w_s, N, out=out[:, :N])
    rows = sample_rows(M, 60, 3)
    assert (out[:, :N].cpu().numpy()[rows] == orc.linear(X, W, rows=rows)["y16"]).all()
    assert (out[:, N:N + 64] == 7.0).all()
    if ldy > (1 << 28) - 64:
        B.muxq_linear_gelu(Xd, w_q, w_s, N, out=out[:, :N])
        assert torch.equal(out[:, :N], B.muxq_linear_gelu(Xd, w_q, w_s, N)[0])
        assert (out[:, N:N + 64] == 7.0).all()
    del out
    torch.cuda.empty_cache()


FIRST_LAUNCH = """
import sys, torch
from paper_2604_04701_amd import binding as B
if sys.argv[1] == "init":
    B.muxq_init()
M, K, N = 2048, 1024, 4096
X = torch.randn(M, K, device="cuda").half()
X[:, :5] *= 50
w_q, w_s = B.muxq_quantize_weight((0.02 * torch.randn(K, N, device="cuda")).half())
kinds = [lambda **kw: B.muxq_linear(X, w_q, w_s, N, **kw), lambda **kw: B.muxq_linear(X, w_q, w_s, N, aux_scale="own", **kw),
         lambda **kw: B.muxq_linear_gelu(X, w_q, w_s, N, **kw)[0]]
for kind in kinds:
    out, ws = torch.empty(M, N, dtype=torch.float16, device="cuda"), B.alloc_workspace(M, K, N, 64)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        kind(out=out, workspace=ws)
    for _ in range(3):
        X.copy_(torch.randn(M, K, device="cuda").half())
        graph.replay()
        torch.cuda.synchronize()
        got = out.clone()
        assert torch.equal(got, kind())
        torch.cuda.synchronize()
print("captured", flush=True)
"""


@pytest.mark.parametrize("init", ["init", "plain"])
def test_first_launch_of_each_kind_under_capture(init):
    """A process whose first launch of a kernel, which loads its binary and sets its attribute, is captured into a graph."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", FIRST_LAUNCH, init], capture_output=True, text=True, timeout=100, cwd=root)
    assert r.returncode == 0 and "captured" in r.stdout, r.stderr[-2000:]
