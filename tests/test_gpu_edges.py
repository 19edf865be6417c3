"""GPU kernels at the sizes where their tiles end: remainders, the smallest and the largest of a range, and the sizes on
either side of a dispatch rule, against the fp64 oracle.  Every array sits inside a buffer of NaN patterns, so that a value
taken from beyond an array shows in the result."""
import numpy as np
import pytest

import fbq_synth
from helpers import framed_in_nan, make_oracle_layer

pytestmark = pytest.mark.gpu


def t16(a):
    import torch
    return None if a is None else framed_in_nan(torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).cuda())


# ------------------------------------------------------------------ feedback quantizer: blocks of 64 rows, 16 per wave, taps in tiles of 32

@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("N,K,r", [(1, 128, 8), (15, 128, 0), (17, 256, 40), (63, 384, 24), (65, 128, 200), (130, 1280, 256), (64, 256, 32)])
def test_quantizer_tile_edges(bits, N, K, r):
    """Codes, scales and zeros are defined in 64 bits; these sums need fewer than 53 bits, so every word must agree."""
    import torch
    import paper_2501_16385_amd as fbq
    L = make_oracle_layer(fbq_synth.LayerSpec("edge", N, K, r, bits), config=41)
    dev = fbq.quantize_feedback(fbq.Desc(N, K, r, bits), t16(L.W), t16(L.A.T) if r else None, t16(L.B.T) if r else None)
    torch.cuda.synchronize()
    assert np.array_equal(dev.scales.cpu().numpy().view(np.float16), L.scales)
    assert np.array_equal(dev.zeros.cpu().numpy().view(np.float16), L.zeros)
    assert np.array_equal(dev.qweight.cpu().numpy().view(np.uint32), L.words)
