"""The narrow row strips (tiles of 256 and 128) and the whole-tile kernel
(64, 32, 16) against the oracle: every tile size at its shallowest and deepest
level counts, per-tile level drops, frame by frame and as one GOP longer than
a launch, a residual-only tail and a frame without output.

5/3 is exact.  9/7 runs in float32: a sample passes through about 16 roundings
per level (two directions of four lifting steps and two scalings, each a
product and a sum), each within 2^-24 of values up to 512 in the intra frame and
64 in each residual frame, and the colour conversion multiplies chroma errors
by at most 1.772; the errors of a chain of frames add up."""
import numpy as np
import pytest
import torch

from gop import Gop, W53, W97

pytestmark = pytest.mark.gpu

CASES = [  # tile, levels, grey
    (256, 2, False), (256, 5, False), (256, 3, True), (128, 2, False), (128, 5, False), (128, 4, True),
    (64, 1, False), (64, 5, False), (64, 6, True), (32, 2, False), (32, 4, False), (16, 1, True), (16, 3, False),
]


def _check(got, want, wavelet, levels, frame, what):
    if wavelet == W53:
        assert np.array_equal(got, want), what
    else:
        tol = 16 * levels * 2.0 ** -24 * 1.772 * (512 + 64 * frame)
        assert np.max(np.abs(got.astype(np.float64) - want)) <= tol, what


@pytest.mark.parametrize("wavelet", [W53, W97])
@pytest.mark.parametrize("tile,levels,grey", CASES)
def test_small_tiles(tile, levels, grey, wavelet):
    from paper_2208_10859_amd import wv
    n_frames = 10
    gop = Gop(3 * tile, 2 * tile, tile, levels, wavelet, n_frames, seed=tile * 10 + levels, chroma=not grey)
    n = gop.spec.n_tiles
    mask = np.array([1, 0, 1, 1, 1, 1], np.uint8)
    rng = np.random.default_rng(tile + levels)
    lc = rng.integers(0, levels + 1, n).astype(np.uint8)
    lc[0] = levels
    want = gop.oracle([mask] * n_frames, [lc] * n_frames)
    vis = np.nonzero(mask)[0]
    dec = wv.Decoder(3 * tile, 2 * tile, tile, levels, wv.W53 if wavelet == W53 else wv.W97,
                     wv.GRAY8 if grey else wv.YUV420)
    assert dec.variants()[dec.variant].startswith(f"strip{tile}" if tile >= 128 else f"tile{tile}")
    frames = [([torch.from_numpy(p).cuda() for p in f["coeffs"]], f["intra"], f["step"]) for f in gop.frames]
    for form in ("gop", "frames", "tail"):
        ref = wv.Reference(dec)
        outs = [torch.full(dec.out_shape(len(vis)), 77, dtype=dec.sample_dtype, device="cuda")
                for _ in range(n_frames)]
        outs[1] = None
        if form == "gop":
            dec.decode_gop(frames, 0, mask, ref, outs, lc)
        else:
            first = n_frames if form == "frames" else 3
            for t, (planes, intra, step) in enumerate(frames[:first]):
                dec.decode_viewport(planes, t, intra, step, mask, ref, outs[t], lc)
            if form == "tail":               # a GOP call that starts with a residual frame
                dec.decode_gop(frames[first:], first, mask, ref, outs[first:], lc)
        torch.cuda.synchronize()
        for t in range(n_frames):
            if outs[t] is not None:
                _check(outs[t].cpu().numpy(), want[t][1], wavelet, levels, t, (form, t))
        for p, w in zip(ref.planes, want[-1][2]):
            got = p.cpu().numpy()
            _check(got[vis], w, wavelet, levels, n_frames - 1, (form, "reference"))
            assert not got[1].any()          # the tile outside the mask is untouched


def test_sets_still_need_512_sample_tiles():
    from paper_2208_10859_amd import wv
    for tile in (256, 128, 64):
        dec = wv.Decoder(2 * tile, tile, tile, 3, wv.W53, wv.YUV420)
        bands = [torch.zeros(dec.set_shape(2, p), dtype=torch.int16, device="cuda") for p in range(3)]
        out = torch.empty(dec.out_shape(2), dtype=torch.uint8, device="cuda")
        with pytest.raises(wv.WvError) as e:
            dec.decode_set(bands, 2, (1, 1), 0, np.ones(2, np.uint8), [out])
        assert e.value.status == wv.EUNSUPPORTED


def test_grey_calls_of_few_and_of_many_tiles():
    """Grey 5/3 frames of 512-sample tiles take another variant up to 24 tiles:
    both sides of the line give the same bytes as a chosen variant, and a
    choice holds for every call."""
    from paper_2208_10859_amd import wv
    dec = wv.Decoder(5 * 512, 5 * 512, 512, 3, wv.W53, wv.GRAY8)
    first = dec.variant
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    coef = [torch.randint(-40, 40, dec.plane_shape(0), generator=gen, device="cuda", dtype=torch.int16)]
    for n_vis in (24, 25):
        mask = np.zeros(25, np.uint8)
        mask[:n_vis] = 1
        res = []
        for pick in (None, first, dec.variants().index("strip_r16_w4_L3_chain_grid")):
            d = wv.Decoder(5 * 512, 5 * 512, 512, 3, wv.W53, wv.GRAY8)
            if pick is not None:
                d.variant = pick
            ref = wv.Reference(d)
            outs = [torch.empty(d.out_shape(n_vis), dtype=torch.uint8, device="cuda") for _ in range(3)]
            d.decode_viewport(coef, 0, True, 3, mask, ref, outs[0])
            d.decode_gop([(coef, False, 1), (coef, False, 2)], 1, mask, ref, outs[1:])
            assert pick is None or d.variant == pick
            torch.cuda.synchronize()
            res.append(outs + [ref.planes[0]])
        for r in res[1:]:
            for a, b in zip(r, res[0]):
                assert torch.equal(a, b)


@pytest.mark.parametrize("tile,n", [(16, 8), (16, 9), (16, 15), (16, 17), (16, 35), (16, 360), (16, 361), (16, 730),
                                    (512, 9), (512, 13)])
def test_mixed_level_counts_in_launches_of_any_size(tile, n):
    """Tiles of different level counts are dealt over a launch: each is decoded
    once and lands in its own slot (against the plain path, which takes them
    in order)."""
    from paper_2208_10859_amd import wv
    levels = 3
    mask = np.ones(n + 3, np.uint8)
    mask[[1, 4, n]] = 0
    lc = np.random.default_rng(n).integers(0, levels + 1, n + 3).astype(np.uint8)
    res = []
    for path in (wv.PATH_FUSED, wv.PATH_PLAIN):
        dec = wv.Decoder((n + 3) * tile, tile, tile, levels, wv.W53, wv.YUV420)
        dec.set_path(path)
        gen = torch.Generator(device="cuda")
        gen.manual_seed(n)
        coef = [[torch.randint(-40, 40, dec.plane_shape(p), generator=gen, device="cuda", dtype=torch.int16)
                 for p in range(3)] for _ in range(3)]
        ref = wv.Reference(dec)
        outs = [torch.empty(dec.out_shape(n), dtype=torch.uint8, device="cuda") for _ in range(3)]
        dec.decode_viewport(coef[0], 0, True, 3, mask, ref, outs[0], lc)
        dec.decode_gop([(coef[1], False, 1), (coef[2], False, 2)], 1, mask, ref, outs[1:], lc)
        torch.cuda.synchronize()
        res.append(outs + list(ref.planes))
    for a, b in zip(*res):
        assert torch.equal(a, b)


@pytest.mark.parametrize("tile,levels,grey", CASES)
def test_float_tiles_round_at_random(tile, levels, grey):
    """9/7: the bound above adds every rounding up with one sign.  Rounding errors
    of values below 512 are spread over 2^-15, a standard deviation of 2^-15 / sqrt(12)
    each; the 16 of each level add up as the square root of their number, and the
    colour conversion adds a chroma error times 1.772 to a luma error, a factor of
    sqrt(1 + 1.772^2).  The largest of a few million samples lies 5 to 6 such
    deviations out: 7.5 are allowed in every frame of a chain (the reference is
    clipped, not transformed: a frame adds the rounding of one sum)."""
    from paper_2208_10859_amd import wv
    n_frames = 10
    gop = Gop(3 * tile, 2 * tile, tile, levels, W97, n_frames, seed=tile * 10 + levels, chroma=not grey)
    mask = np.array([1, 0, 1, 1, 1, 1], np.uint8)
    want = gop.oracle([mask] * n_frames, [np.full(6, levels, np.uint8)] * n_frames)
    dec = wv.Decoder(3 * tile, 2 * tile, tile, levels, wv.W97, wv.GRAY8 if grey else wv.YUV420)
    frames = [([torch.from_numpy(p).cuda() for p in f["coeffs"]], f["intra"], f["step"]) for f in gop.frames]
    ref = wv.Reference(dec)
    outs = [torch.empty(dec.out_shape(5), dtype=dec.sample_dtype, device="cuda") for _ in range(n_frames)]
    dec.decode_gop(frames, 0, mask, ref, outs)
    tol = 7.5 * 2.0 ** -15 * np.sqrt(16 * levels / 12) * (1.0 if grey else np.sqrt(1 + 1.772 ** 2))
    for t in range(n_frames):
        err = float(np.max(np.abs(outs[t].cpu().numpy().astype(np.float64) - want[t][1])))
        assert err <= tol, (t, err, tol)
