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
                                     (72, 32776, 32832), (4104, 24, 24), (1024, 1280, 1280), (1024, 1288, 1288), (40, 50304, 50304)])
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
