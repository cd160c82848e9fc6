"""The weight quantiser in strips of 64 output channels against the CPU oracle: ragged last strips,
K below, at and above the step of 512 input channels, both granularities, narrower codes, the
difficulty migration, K beyond the line to the other kernels.  Codes, code sums and scales exact."""
import numpy as np
import pytest
import torch

from gpu_common import B, orc, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gran", ["tensor", "channel"])
@pytest.mark.parametrize("K,N", [(8, 8), (64, 72), (504, 64), (512, 136), (520, 1000), (1032, 200), (4104, 264),
                                 (8192, 72), (8200, 72)])
def test_weight_codes_sums_and_scales(K, N, gran):
    rng = np.random.default_rng(K + N)
    W = synth.make_w(K, N, rng)
    W[:, 3] = 0                                          # an all-zero unit
    f = np.exp(rng.uniform(-1.0, 1.0, K)).astype(np.float32)
    for bits, factors in ((8, None), (5, None), (8, f)):
        ref = W if factors is None else (W.astype(np.float32) * f[:, None]).astype(np.float16)
        ld = torch.zeros((K, N + 8), dtype=torch.float16, device="cuda")
        ld[:, :N] = torch.from_numpy(W).cuda()
        w_q, w_s = B.muxq_quantize_weight(ld[:, :N], gran, bits=bits,
                                          factors=None if factors is None else torch.from_numpy(f).cuda())
        o = orc.linear(np.zeros((1, K), np.float16), ref, w_gran=gran, w_bits=bits)
        got = B.unpack(w_q, N, B.k_pad(K)).cpu().numpy()
        assert (got[:, :K] == o["w_q"].T).all() and (got[:, K:] == 0).all()
        assert (w_s.cpu().numpy() == o["s_w"]).all()
        assert (B.wq_row_sums(w_q, K, N).cpu().numpy() == got.astype(np.int64).sum(axis=1)).all()


@pytest.mark.parametrize("gran", ["tensor", "channel"])
@pytest.mark.parametrize("K,N,ldw", [(1032, 8192, 8192), (1032, 8192, 8200), (1032, 8200, 8200), (72, 32768, 32768),
                                     (72, 32776, 32832), (4104, 24, 24), (1024, 1280, 1280), (1024, 1288, 1288),
                                     (1032, 1280, 1280), (1024, 8184, 8184), (264, 16448, 16448), (520, 32704, 32704),
                                     (520, 16448, 16448), (40, 50304, 50304)])
def test_weight_codes_on_both_sides_of_the_line(K, N, ldw, gran):
    """Rows on and off 128-byte lines, few and many strips, short and long K: strips and 64 x 64 tiles."""
    rng = np.random.default_rng(K + ldw)
    W = synth.make_w(K, N, rng)
    ld = torch.zeros((K, ldw), dtype=torch.float16, device="cuda")
    ld[:, :N] = torch.from_numpy(W).cuda()
    w_q, w_s = B.muxq_quantize_weight(ld[:, :N], gran)
    o = orc.quantize_weight(W, gran)
    got = B.unpack(w_q, N, B.k_pad(K)).cpu().numpy()
    assert (got[:, :K] == o["w_q"].T).all() and (got[:, K:] == 0).all()
    assert (w_s.cpu().numpy() == o["s_w"]).all()
    assert (B.wq_row_sums(w_q, K, N).cpu().numpy() == got.astype(np.int64).sum(axis=1)).all()


@pytest.mark.parametrize("K,N", [(5128, 16448), (5128, 16512), (8200, 15936), (8200, 16000), (4104, 33024),
                                 (9224, 16448), (5120, 12296), (3072, 18440), (12296, 12416), (24584, 12288)])
def test_weight_codes_by_rounds_of_strips(K, N):
    """Strips in one round and in several, the last one short, a single strip or full, rows on and off 128-byte lines, and
    the separate launches beside them (the channels are independent: the oracle takes some of each strip, all of the last)."""
    g = torch.Generator(device="cuda").manual_seed(K + N)
    W = (0.02 * torch.randn(K, N, generator=g, device="cuda")).half()
    w_q, w_s = B.muxq_quantize_weight(W, "channel")
    cols = np.unique(np.concatenate([np.arange(0, N, 37), np.arange(N - 64, N)]))
    o = orc.quantize_weight(W[:, torch.from_numpy(cols).cuda()].cpu().numpy(), "channel")
    codes = B.unpack(w_q, N, B.k_pad(K))
    got = codes[torch.from_numpy(cols).cuda()].cpu().numpy()
    assert (got[:, :K] == o["w_q"].T).all() and (got[:, K:] == 0).all()
    assert (w_s.cpu().numpy()[cols] == o["s_w"]).all()
    assert (B.wq_row_sums(w_q, K, N) == codes.sum(dim=1, dtype=torch.int64)).all()


@pytest.mark.parametrize("K", [1032, 1536, 2040, 2048, 2056, 2568, 3080, 4096])
def test_rows_kept_between_the_two_readings_and_rows_read_again(K):
    """Every channel's largest weight in another row, so that each step of 512 rows sets some scale."""
    N = 264
    rng = np.random.default_rng(K)
    W = synth.make_w(K, N, rng)
    W[(np.arange(N) * 131 + K - 1) % K, np.arange(N)] = 0.5
    w_q, w_s = B.muxq_quantize_weight(torch.from_numpy(W).cuda(), "channel")
    o = orc.quantize_weight(W, "channel")
    got = B.unpack(w_q, N, B.k_pad(K)).cpu().numpy()
    assert (got[:, :K] == o["w_q"].T).all() and (got[:, K:] == 0).all()
    assert (w_s.cpu().numpy() == o["s_w"]).all()
    assert (B.wq_row_sums(w_q, K, N).cpu().numpy() == got.astype(np.int64).sum(axis=1)).all()
