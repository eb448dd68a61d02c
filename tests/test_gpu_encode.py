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


@pytest.mark.parametrize("wavelet", [owv.W53, owv.W97])
def test_threads_share_one_context(wavelet):
    """The context's workspace serves one call at a time: two threads with
    streams and planes of their own get what each gets alone."""
    import threading

    from paper_2208_10859_amd import wv
    dec = wv.Decoder(2048, 1024, 256, 4, wv.W53 if wavelet == owv.W53 else wv.W97, wv.GRAY8)
    torch.manual_seed(1)
    src = [torch.randint(0, 256, dec.plane_shape(0), dtype=torch.uint8, device="cuda") for _ in range(2)]
    alone, dst = [[torch.zeros(dec.plane_shape(0), dtype=dec.coef_dtype, device="cuda") for _ in range(2)]
                  for _ in range(2)]
    for s, d in zip(src, alone):
        dec.encode_intra([s], [d], 2)
    torch.cuda.synchronize()
    same = [[], []]

    def work(k):
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            for _ in range(20):
                dst[k].zero_()
                dec.encode_intra([src[k]], [dst[k]], 2, stream=st)
                same[k].append(torch.equal(dst[k], alone[k]))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert same == [[True] * 20] * 2


@pytest.mark.parametrize("tile,levels,grey", CASES)
def test_float_encoder_differs_at_rounding_ties_only(tile, levels, grey):
    """9/7: float64 on both sides, so a coefficient of up to 2^10 is off by a few
    hundred roundings of 2^-53 of it at most, below 1e-10.  An index may differ
    from the oracle's only where |c| / step + 1/2 lies within 1e-9 of a whole
    number, and then by one; every other value is the same float.  (The
    chequerboard's approximation, 127.5 everywhere, is such a tie.)"""
    from paper_2208_10859_amd import wv
    dec = wv.Decoder(3 * tile, tile, tile, levels, wv.W97, wv.GRAY8 if grey else wv.YUV420)
    rng = np.random.default_rng(tile * 10 + levels + 1)
    src = [rng.integers(0, 256, dec.plane_shape(p), dtype=np.uint8) for p in range(dec.nplanes)]
    src[0][0] = 255 * (np.indices((tile, tile)).sum(0) & 1)
    coef = [owv.fwd2d(s, levels, owv.W97) for s in src]
    assert all(np.abs(c).max() < 1024 for c in coef)
    dev = [torch.from_numpy(s).cuda() for s in src]
    for step in (1, 3, 16, 100, 65535):
        dst = [torch.zeros(dec.plane_shape(p), dtype=dec.coef_dtype, device="cuda") for p in range(dec.nplanes)]
        dec.encode_intra(dev, dst, step)
        for g, c in zip(dst, coef):
            got = g.cpu().numpy()
            a = np.abs(c) / step + 0.5
            tie = np.abs(a - np.rint(a)) < 1e-9
            k = np.where(tie, np.rint(a), np.floor(a))
            low = np.where(tie, k - 1, k)
            want = [(step * np.sign(c) * i).astype(np.float32) for i in (k, low)]
            assert np.all((got == want[0]) | (got == want[1]))
            assert tie.mean() < 0.1
