"""The encoder's kernels at the sizes where their split changes: tiles encoded
whole in LDS (up to 128), tiles whose two finest levels run in strips (256 and
512), one and two levels (no second kernel), the deepest level counts, grey
frames, source planes at an odd address, and the quantiser's step range."""
import numpy as np
import pytest
import torch

from oracle import codec
from oracle import wavelet as owv

pytestmark = pytest.mark.gpu

CASES = [  # tile, levels, grey
    (16, 1, False), (16, 4, True), (16, 3, False), (32, 5, True), (64, 4, False), (128, 2, False), (128, 7, True),
    (256, 1, False), (256, 2, True), (256, 5, False), (512, 1, False), (512, 2, False), (512, 3, True),
    (512, 8, False),
]


@pytest.mark.parametrize("wavelet", [owv.W53, owv.W97])
@pytest.mark.parametrize("tile,levels,grey", CASES)
def test_encoder_matches_oracle(tile, levels, grey, wavelet):
    from paper_2208_10859_amd import wv
    wl = wv.W53 if wavelet == owv.W53 else wv.W97
    dec = wv.Decoder(3 * tile, tile, tile, levels, wl, wv.GRAY8 if grey else wv.YUV420)
    rng = np.random.default_rng(tile * 10 + levels)
    src = [rng.integers(0, 256, dec.plane_shape(p), dtype=np.uint8) for p in range(dec.nplanes)]
    src[0][0] = 255 * (np.indices((tile, tile)).sum(0) & 1)      # largest details
    dev = []
    for p in src:                                                # odd addresses
        buf = torch.zeros(p.size + 1, dtype=torch.uint8, device="cuda")
        buf[1:] = torch.from_numpy(p.reshape(-1)).cuda()
        dev.append(buf[1:].view(p.shape))
    for step in (1, 3, 16, 65535):
        dst = [torch.zeros(dec.plane_shape(p), dtype=dec.coef_dtype, device="cuda") for p in range(dec.nplanes)]
        dec.encode_intra(dev, dst, step)
        want = codec.encode_intra(src, levels, wavelet, step)
        for g, w in zip(dst, want):
            got = g.cpu().numpy()
            if wavelet == owv.W53:
                assert np.array_equal(got, w)
            else:
                # float64 on both sides: a value within 1e-10 of a rounding
                # tie may land on the next multiple of the step
                diff = np.abs(got.astype(np.float64) - w)
                assert diff.max() <= step and np.mean(diff > 0) < 1e-4
