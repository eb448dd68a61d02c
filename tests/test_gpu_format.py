"""GPU parity of the sparse-format rebuild (wv_sparse_rebuild) and of the
decode that follows it, against the oracle (oracle/paperformat.py).

The rebuilt dense planes must equal the oracle's exactly (the kernel and the
oracle dequantise with the same float32 operations); the decode of them is
bit-exact for 5/3 and within max-abs 1e-3 for 9/7.  Frames are encoded by
the oracle's encoder from seeded synthetic sources.
"""
import numpy as np
import pytest
import torch

import wvinputs
from oracle import paperformat as pf
from oracle.wavelet import W53, W97, fwd2d

pytestmark = pytest.mark.gpu

TOL97 = 1e-3


def _wv():
    from paper_2208_10859_amd import fmt, wv
    return wv, fmt


def _frame(width, height, tile, levels, wavelet, tiles, seed, alpha, poles):
    """Oracle-encoded planes of a synthetic frame (only `tiles` carry content),
    from the forward transform of the wavelet the frame is decoded with."""
    spec = wvinputs.FrameSpec(width, height, tile, seed)
    src = wvinputs.source_planes(spec, tiles=tiles)
    enc, edges = [], []
    for p, s in enumerate(src):
        s = s.numpy().reshape(-1, *s.shape[2:]).astype(np.float64)
        c = fwd2d(s, levels, wavelet).astype(np.float32)
        ph = height if p == 0 else height // 2
        enc.append(pf.encode_plane(c, levels, width // tile, ph, alpha, poles))
        edges.append(s.shape[-1])
    return enc, edges


def _run(dec, enc, mask, lc):
    wv, fmt = _wv()
    planes = [fmt.DevicePlane(e) for e in enc]
    dense = [torch.zeros(dec.plane_shape(p), dtype=dec.coef_dtype, device="cuda")
             for p in range(dec.nplanes)]
    fmt.rebuild(dec, planes, mask, dense, lc)
    nvis = int(np.count_nonzero(mask))
    out = torch.empty(dec.out_shape(nvis), dtype=dec.sample_dtype, device="cuda")
    ref = wv.Reference(dec)
    dec.decode_viewport(dense, 0, True, 1, mask, ref, out, lc)
    torch.cuda.synchronize()
    return [d.cpu().numpy() for d in dense], out.cpu().numpy()


@pytest.mark.parametrize("wavelet,levels,alpha,poles,foveate", [
    (W97, 5, 0.1, True, False),
    (W97, 4, 0.25, False, True),
    (W53, 5, 0.1, True, True),
    (W53, 3, 0.0, False, False),
])
def test_rebuild_and_decode_equal_oracle(wavelet, levels, alpha, poles, foveate):
    """2048 x 1024 (4 x 2 tiles of 512), a ragged viewport of 5 tiles; the
    format made with the paper's HQ / LQ thresholds (0.1 / 0.25), the lossless
    limit, with and without the pole factor, foveated and not."""
    wv, fmt = _wv()
    W, H, tile = 2048, 1024, 512
    mask = np.array([1, 1, 0, 1, 0, 1, 1, 0], np.uint8)
    vis = np.nonzero(mask)[0]
    enc, edges = _frame(W, H, tile, levels, wavelet, vis, 300 + levels, alpha, poles)
    lc = None
    if foveate:
        lc = np.full(8, levels, np.uint8)
        lc[[1, 5]] = levels - 1
        lc[6] = levels - 2
    wl = wv.W53 if wavelet == W53 else wv.W97
    dec = wv.Decoder(W, H, tile, levels, wl, wv.YUV420)
    dense, out = _run(dec, enc, mask, lc)
    lcv = np.full(8, levels) if lc is None else lc
    vis_w, want, _, want_dense = pf.decode_viewport(enc, edges, mask, levels, wavelet, lcv)
    for p in range(3):
        assert np.array_equal(dense[p][vis], want_dense[p]), f"plane {p}: rebuilt coefficients differ"
        others = np.setdiff1d(np.arange(8), vis)
        assert not dense[p][others].any(), "tiles outside the mask were written"
    if wavelet == W53:
        assert np.array_equal(out, want)
    else:
        assert float(np.max(np.abs(out.astype(np.float64) - want))) <= TOL97


def test_grey_small_tiles():
    """256 x 256 grey, 64-sample tiles (one block per chroma-sized plane is
    not involved; 2 x 2 blocks per tile), 3 levels, every tile visible."""
    wv, fmt = _wv()
    W = H = 256
    spec = wvinputs.FrameSpec(W, H, 64, 17, chroma=False)
    s = wvinputs.source_planes(spec)[0].numpy().reshape(-1, 64, 64).astype(np.float64)
    c = fwd2d(s, 3, W97).astype(np.float32)
    enc = [pf.encode_plane(c, 3, 4, H, 0.05, True)]
    mask = np.ones(16, np.uint8)
    dec = wv.Decoder(W, H, 64, 3, wv.W97, wv.GRAY8)
    dense, out = _run(dec, enc, mask, None)
    _, want, _, want_dense = pf.decode_viewport(enc, [64], mask, 3, W97)
    assert np.array_equal(dense[0], want_dense[0])
    assert float(np.max(np.abs(out.astype(np.float64) - want))) <= TOL97


def test_hostile_records_are_ignored():
    """Indices outside their block and block ends past the record count are
    skipped by the kernel's own checks; the valid records still land."""
    wv, fmt = _wv()
    dec = wv.Decoder(128, 128, 64, 2, wv.W97, wv.GRAY8)
    nb = 4
    block_end = np.zeros(4 * nb, np.uint32)
    block_end[0] = 3                 # tile 0, block 0: three records
    block_end[1:] = 1 << 30          # every later block claims records that do not exist
    enc = {"block_end": block_end, "values": np.array([255, 0, 255], np.uint8),
           "index": np.array([0, 5000, 33], np.uint16),
           "bounds": np.array([0.0, 10.0, -1.0, 1.0], np.float32)}
    plane = fmt.DevicePlane(enc)
    dense = [torch.zeros(dec.plane_shape(0), dtype=torch.float32, device="cuda")]
    fmt.rebuild(dec, [plane], np.ones(4, np.uint8), dense)
    torch.cuda.synchronize()
    d = dense[0].cpu().numpy()
    assert d[0, 0, 0] == 10.0 and d[0, 1, 1] == 10.0
    assert np.count_nonzero(d) == 2


def test_rebuild_errors():
    wv, fmt = _wv()
    dec = wv.Decoder(128, 128, 64, 2, wv.W97, wv.GRAY8)
    enc = {"block_end": np.zeros(16, np.uint32), "values": np.zeros(0, np.uint8),
           "index": np.zeros(0, np.uint16), "bounds": np.zeros(4, np.float32)}
    plane = fmt.DevicePlane(enc)
    dense = [torch.zeros(dec.plane_shape(0), dtype=torch.float32, device="cuda")]
    with pytest.raises(wv.WvError) as e:
        fmt.rebuild(dec, [plane], np.ones(4, np.uint8), dense, np.full(4, 3, np.uint8))
    assert e.value.status == wv.EINVAL


# --- asynchronous prefetch of inter-frame sets (Section 3.5, Fig. 4) ---------

from oracle import interframe


def _set_store(W, H, tile, levels, wavelet, seed, alpha):
    """Oracle-encoded bands of one set of 4 frames: each frame's forward
    transform, the Haar transform across the set (Section 3.2), every band
    encoded in the format (Sections 3.3, 3.4).  Returns [band][plane] records."""
    frames = []
    for f in range(4):
        spec = wvinputs.FrameSpec(W, H, tile, seed * 10 + f)
        src = wvinputs.source_planes(spec)
        frames.append([fwd2d(s.numpy().reshape(-1, *s.shape[2:]).astype(np.float64), levels, wavelet)
                       for s in src])
    store = [[None] * 3 for _ in range(4)]
    for p in range(3):
        bands = interframe.haar_forward(np.stack([frames[f][p] for f in range(4)]))
        ph = H if p == 0 else H // 2
        for b in range(4):
            store[b][p] = pf.encode_plane(bands[b].astype(np.float32), levels, W // tile, ph, alpha, True)
    return store


def _oracle_set(store, edges, mask, levels, wavelet, lc):
    """Rebuilt visible bands and the 4 decoded frames, by the oracle."""
    n_tiles = mask.size
    vis = np.nonzero(mask)[0]
    planes, dense = [], []
    for p in range(3):
        dt = np.int16 if wavelet == W53 else np.float32
        full = np.zeros((4, n_tiles, edges[p], edges[p]), dt)
        for b in range(4):
            full[b][vis] = pf.rebuild_plane(store[b][p], edges[p], levels, vis, lc, wavelet)
        planes.append(full)
    outs = [interframe.decode_set_viewport(planes, t, mask, levels, wavelet, (1, 1, 1, 1), lc)[1]
            for t in range(4)]
    return planes, outs


@pytest.mark.parametrize("wavelet,levels,direct", [(W97, 4, False), (W53, 5, True)])
def test_prefetch_pipeline_equals_oracle(wavelet, levels, direct):
    """Three sets of four frames at 2048 x 1024 (4 x 2 tiles of 512) staged
    from a pinned host store, each while the previous set is rebuilt and
    decoded: ragged viewports, one foveated, one empty.  Rebuilt bands are
    exact; decoded frames bit-exact (5/3) or within 1e-3 (9/7)."""
    wv, fmt = _wv()
    W, H, tile = 2048, 1024, 512
    wl = wv.W53 if wavelet == W53 else wv.W97
    dec = wv.Decoder(W, H, tile, levels, wl, wv.YUV420)
    edges = [tile, tile // 2, tile // 2]
    masks = [np.array([1, 1, 0, 1, 0, 1, 1, 0], np.uint8), np.array([0, 1, 1, 0, 1, 1, 1, 1], np.uint8),
             np.zeros(8, np.uint8), np.array([1, 0, 0, 0, 0, 0, 0, 1], np.uint8)]
    lcs = [np.full(8, levels, np.uint8) for _ in masks]
    lcs[1][[2, 4]] = levels - 1
    lcs[1][6] = levels - 3
    stores = [_set_store(W, H, tile, levels, wavelet, 70 + s, 0.05 if s % 2 else 0.0) for s in range(2)]
    host = [[[fmt.HostPlane(e) for e in band] for band in st] for st in stores]
    n_sets = len(masks)
    pfch = fmt.Prefetcher(dec, 4, 64 << 20)
    bufs = [[torch.zeros(dec.set_shape(4, p), dtype=dec.coef_dtype, device="cuda") for p in range(3)]
            for _ in range(2)]
    outs = [[torch.full(dec.out_shape(max(1, int(m.sum()))), 7, dtype=dec.sample_dtype, device="cuda")
             for _ in range(4)] for m in masks]
    up = [pfch.stage(host[0], masks[0], lcs[0], direct)]
    for s in range(n_sets):
        if s + 1 < n_sets:      # staged while set s is rebuilt and decoded
            up.append(pfch.stage(host[(s + 1) % 2], masks[s + 1], lcs[s + 1], direct))
        b = bufs[s % 2]
        pfch.rebuild([b[p][f] for f in range(4) for p in range(3)])
        nvis = int(masks[s].sum())
        if nvis:
            dec.decode_set(b, 4, (1, 1, 1, 1), 0, masks[s], [o[:nvis] for o in outs[s]], lcs[s])
        if s == 1:
            torch.cuda.synchronize()   # a set kept for the band check below
            kept = [x.cpu().numpy() for x in b]
    torch.cuda.synchronize()
    pfch.close()
    assert up[2] == 0
    for s in range(n_sets):
        st = stores[s % 2]
        vis = np.nonzero(masks[s])[0]
        # uploaded bytes: staged block ends plus three bytes per record of the runs
        rec = sum(fmt.visible_runs(dec._desc, p, st[b][p], masks[s], lcs[s])[2] for b in range(4) for p in range(3))
        nb = [fmt.blocks_per_tile(dec._desc, p) for p in range(3)]
        if direct:
            assert up[s] == 3 * rec + 4 * 4 * len(vis) * sum(nb)
        else:
            assert up[s] >= 3 * rec + 4 * 4 * len(vis) * sum(nb)
        if not vis.size:
            continue
        want_planes, want_outs = _oracle_set(st, edges, masks[s], levels, wavelet, lcs[s])
        if s == 1:
            for p in range(3):
                assert np.array_equal(kept[p][:, vis], want_planes[p][:, vis]), f"set 1 plane {p} bands"
        for t in range(4):
            got = outs[s][t][:len(vis)].cpu().numpy()
            if wavelet == W53:
                assert np.array_equal(got, want_outs[t]), f"set {s} frame {t}"
            else:
                assert float(np.max(np.abs(got.astype(np.float64) - want_outs[t]))) <= TOL97, f"set {s} frame {t}"


def test_prefetch_errors():
    wv, fmt = _wv()
    dec = wv.Decoder(1024, 512, 512, 3, wv.W97, wv.GRAY8)
    enc = {"block_end": np.zeros(512, np.uint32), "values": np.zeros(0, np.uint8),
           "index": np.zeros(0, np.uint16), "bounds": np.zeros(4, np.float32)}
    hp = fmt.HostPlane(enc)
    with pytest.raises(wv.WvError):
        fmt.Prefetcher(dec, 0, 1 << 20)
    pfch = fmt.Prefetcher(dec, 2, 4096)
    dense = [torch.zeros(dec.plane_shape(0), dtype=torch.float32, device="cuda")]
    with pytest.raises(wv.WvError) as e:             # nothing staged
        pfch.rebuild(dense)
    assert e.value.status == wv.EINVAL
    with pytest.raises(wv.WvError):                  # three frames, at most two
        pfch.stage([[hp]] * 3, np.ones(2, np.uint8))
    with pytest.raises(wv.WvError):                  # 2 x 256 block ends = 2 KiB per frame: 3 frames do not fit 4 KiB
        pfch2 = fmt.Prefetcher(dec, 3, 4096)
        pfch2.stage([[hp]] * 3, np.ones(2, np.uint8))
    assert pfch.stage([[hp]], np.ones(2, np.uint8)) == 2048
    assert pfch.stage([[hp]], np.array([1, 0], np.uint8)) == 1024
    with pytest.raises(wv.WvError):                  # a third staged set
        pfch.stage([[hp]], np.ones(2, np.uint8))
    pfch.rebuild(dense)
    pfch.rebuild(dense)
    torch.cuda.synchronize()
    assert not dense[0].any()
    pfch.close()


def test_prefetch_from_store_file_equals_oracle(tmp_path):
    """The same pipeline with its store read from a file of the format
    (Section 3.4) into pinned memory: two sets, per-run copies straight from
    the store for the second."""
    wv, fmt = _wv()
    W, H, tile, levels = 2048, 1024, 512, 4
    dec = wv.Decoder(W, H, tile, levels, wv.W97, wv.YUV420)
    edges = [tile, tile // 2, tile // 2]
    stores = [_set_store(W, H, tile, levels, W97, 90 + s, 0.05) for s in range(2)]
    path = tmp_path / "sets.wvf"
    fmt.write_store(path, dec._desc, [band for st in stores for band in st])
    st = fmt.Store(path)
    assert st.n_frames == 8
    masks = [np.array([1, 1, 0, 1, 0, 1, 1, 0], np.uint8), np.array([0, 1, 1, 1, 1, 0, 0, 1], np.uint8)]
    lcs = [np.full(8, levels, np.uint8), np.array([4, 3, 4, 2, 4, 4, 4, 1], np.uint8)]
    pfch = fmt.Prefetcher(dec, 4, 64 << 20)
    for s in range(2):
        bufs = [torch.zeros(dec.set_shape(4, p), dtype=dec.coef_dtype, device="cuda") for p in range(3)]
        nvis = int(masks[s].sum())
        outs = [torch.empty(dec.out_shape(nvis), dtype=dec.sample_dtype, device="cuda") for _ in range(4)]
        pfch.stage([st.frame(4 * s + b) for b in range(4)], masks[s], lcs[s], direct=s == 1)
        pfch.rebuild([bufs[p][f] for f in range(4) for p in range(3)])
        dec.decode_set(bufs, 4, (1, 1, 1, 1), 0, masks[s], outs, lcs[s])
        torch.cuda.synchronize()
        want_planes, want_outs = _oracle_set(stores[s], edges, masks[s], levels, W97, lcs[s])
        vis = np.nonzero(masks[s])[0]
        for p in range(3):
            assert np.array_equal(bufs[p].cpu().numpy()[:, vis], want_planes[p][:, vis]), (s, p)
        for t in range(4):
            err = float(np.max(np.abs(outs[t].cpu().numpy().astype(np.float64) - want_outs[t])))
            assert err <= TOL97, (s, t, err)
    pfch.close()
    st.close()


@pytest.mark.parametrize("tile,levels,tx,ty,wavelet", [
    (16, 3, 20, 20, W53),     # 389 visible tiles: more than one launch's; luma blocks of 16, chroma of 8
    (16, 1, 5, 4, W97),
    (32, 4, 5, 4, W97),       # blocks of 32 and 16, one per plane tile
    (64, 5, 5, 4, W53),
    (128, 2, 3, 2, W97),
    (256, 6, 3, 2, W53),
])
def test_rebuild_of_yuv_tiles_of_every_size(tile, levels, tx, ty, wavelet):
    """One launch rebuilds all planes of a frame, whose block edges and block
    counts differ: every tile size with mixed level counts, and a viewport of
    more tiles than a launch takes."""
    wv, _ = _wv()
    W, H, n = tx * tile, ty * tile, tx * ty
    rng = np.random.default_rng(tile + levels)
    mask = np.ones(n, np.uint8)
    mask[rng.choice(n, 11 if n > 360 else 2, replace=False)] = 0
    vis = np.nonzero(mask)[0]
    lc = rng.integers(0, levels + 1, n).astype(np.uint8)
    lc[vis[0]] = levels
    enc, edges = _frame(W, H, tile, levels, wavelet, vis, 500 + tile, 0.05, True)
    dec = wv.Decoder(W, H, tile, levels, wv.W53 if wavelet == W53 else wv.W97, wv.YUV420)
    dense, out = _run(dec, enc, mask, lc)
    _, want, _, want_dense = pf.decode_viewport(enc, edges, mask, levels, wavelet, lc)
    for p in range(3):
        assert np.array_equal(dense[p][vis], want_dense[p]), f"plane {p}: rebuilt coefficients differ"
        assert not dense[p][mask == 0].any(), "tiles outside the mask were written"
    if wavelet == W53:
        assert np.array_equal(out, want)
    else:
        assert float(np.max(np.abs(out.astype(np.float64) - want))) <= TOL97
